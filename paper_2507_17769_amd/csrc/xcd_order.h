// Which block takes which piece of work, for kernels whose pieces share cache lines: consecutive blocks run on different XCDs,
// each with an L2 of its own, eight of them.  Host and device, without HIP, so that it can be checked on its own.
#pragma once

namespace ps {

// Token rows and the L2s.  A 128-byte line of an operand-order matrix holds 16 bytes of eight consecutive rows, and a line of
// the KV cache up to 16 tokens, while consecutive blocks run on different XCDs, each with an L2 of its own: with a block per
// row a line would be written in pieces by eight L2s and put together in memory, byte-masked.  So the row kernels give every
// XCD octets of rows: block b takes row row_of_block(b), and the grid is rounded up to whole rounds of eight octets.  Below
// 64 rows, where the octets would not reach all XCDs and launch latency is what counts, blocks are rows.
// (2048 tokens, 8B shape, us, rows in order / octets: reduce_add_norm 30.1 / 25.5, rmsnorm 17.8 / 13.9, rope_append 20.9 / 19.9,
// whole step of four layers 3437 / 3349; 271 tokens 958 / 938; 64 tokens 834 / 832.)
constexpr int ROW_ROUND = 64;
__host__ __device__ inline int row_blocks(int n_rows) { return n_rows < ROW_ROUND ? n_rows : (n_rows + ROW_ROUND - 1) / ROW_ROUND * ROW_ROUND; }
__host__ __device__ inline int row_of_block(int b, int n_rows) { return n_rows < ROW_ROUND ? b : (b & ~63) | ((b & 7) << 3) | ((b >> 3) & 7); }

// Merge groups (one 16-row query tile of one sequence and KV head each) are listed KV head by KV head, the tiles of prefill
// chunks before the decodes.  Four consecutive groups go to an XCD in rounds of 32: for a chunk they are tiles of consecutive
// rows, which share lines of the output, and every XCD gets the same mixture of a chunk's tiles and of decodes.  Fewer than 128
// groups, with which the rounds would not reach all XCDs evenly, are dealt out as contiguous eighths: the eight KV heads of a few
// decodes one to each XCD, which is also where the attention kernel wrote their partials.  (8B shape, four layers, step in us,
// in order / eighths / rounds: one decode behind 1024 tokens, 8 groups, 401.3 / 401.4 / 403.2; behind 8192 415.6 / 415.4 / 418.6;
// eight decodes, 64 groups, 441.0 / 440.4 / 442.6; 128 tokens next to 16 decodes, some 380 groups, 721.1 / 724.4 / 719.4; 250
// tokens next to 21 940.0 / 937.8 / 939.2; 64 decodes, 512 groups, the same each way.)
constexpr int MERGE_ROUNDS_FROM = 128;
__host__ __device__ inline int merge_blocks(int n_groups) { return n_groups < MERGE_ROUNDS_FROM ? (n_groups + 7) / 8 * 8 : (n_groups + 31) / 32 * 32; }
__host__ __device__ inline int merge_group_of_block(int b, int n_groups) {
    return n_groups < MERGE_ROUNDS_FROM ? (b & 7) * ((n_groups + 7) >> 3) + (b >> 3) : (b & ~31) | ((b & 7) << 2) | ((b >> 3) & 3);
}

}  // namespace ps
