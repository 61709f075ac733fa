// Order of the 64-slot tile's workgroups (gemm_mid.hpp): plain integer arithmetic, also compiled for the host.
#pragma once

namespace moe {

// The block and which of its nwork pieces (tile group, reduction range) a workgroup takes; false: none.  A block costs by its
// live parts, and experts with many rows may follow one another, so an equal number of consecutive blocks for each XCD is no
// equal share of the work.  So lanes of G = 8 / D XCDs take every D-th block, and the XCDs of a lane an equal share of
// the pieces of each of its blocks.  More XCDs on a block read its activations that many times (256 experts of 2048
// columns, even routing: 3 to 10 % with G = 8), fewer blocks in a lane even out less: 16 at least.
// Layer, time of the tiles that ran before this one over its time, runs of blocks -> this order: 8 experts (K 4096, N 14336, fp16),
// 20 rows an expert on average, power-law routing 0.85 -> 1.09, even 1.05 -> 1.04; 256 experts (K 7168, N 2048), 10 rows, weights of
// the experts as 1 / rank 0.96 -> 1.35, even 1.15 -> 1.15; 128 experts (K = N = 2048), 14 rows, 1 / rank 0.86 -> 1.11, even 1.01 -> 1.00.
__host__ __device__ __forceinline__ bool mid_work(int pid, int nblk, int nwork, int& blk, int& work) {
  const int xcd = pid & 7, D = nblk < 32 ? 1 : nblk < 64 ? 2 : nblk < 128 ? 4 : 8, G = 8 / D;
  const int nb = nblk / D, c = xcd % G, per = nb * nwork / G, rem = nb * nwork % G, len = per + (c < rem ? 1 : 0);
  int idx = pid >> 3;
  if (idx < len) {
    // the pieces of a block in G ranges, a range of all blocks before the next range
    const int L = c * per + (c < rem ? c : rem) + idx, range = (G * (L / nb) + G - 1) / nwork;
    const int first = range * nwork / G, width = (range + 1) * nwork / G - first, at = L - nb * first;
    blk = at / width * D + xcd / G;
    work = first + at % width;
    return true;
  }
  idx -= len;                  // the up to D - 1 blocks that are left: all XCDs
  const int left = (nblk - nb * D) * nwork, each = left / 8, more = left % 8;
  if (idx >= each + (xcd < more ? 1 : 0)) return false;
  const int L = xcd * each + (xcd < more ? xcd : more) + idx;
  blk = nb * D + L / nwork;
  work = L % nwork;
  return true;
}

// Workgroups to launch for up to nblk blocks (the kernel knows their number): the shares of an XCD differ by two at most.
__host__ inline long long mid_grid(long long nblk, int nwork) { return 8 * ((nblk * nwork + 7) / 8 + 2); }

}  // namespace moe
