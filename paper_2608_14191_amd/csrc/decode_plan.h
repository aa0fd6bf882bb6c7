// Shape decisions of the matrix-core decode kernel: on the host, before anything is launched,
// query heads and tokens per workgroup, the dynamic LDS layout and the grid; in every workgroup,
// from the lengths, the runs of a ragged batch.  Plain C++.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <algorithm>

#include "params.h"

#if defined(__HIPCC__)
#define AATC_PLAN_HD __host__ __device__
#else
#define AATC_PLAN_HD
#endif

namespace aatc {

constexpr int kMaxNH = 8;                        // most query heads of a workgroup
constexpr int kMfmaThreads = 512;                // eight waves
constexpr int kMfmaRecord = 128;                 // widest record of the matrix-core kernel
constexpr int kComputeUnits = 256;
constexpr size_t kMfmaLdsMax = 160 * 1024 - 2 * 1024;   // (static LDS: under 2 KiB)
constexpr size_t kAppendScratchBytes = 1104;     // AppendScratch, rounded to 16 bytes

// The LDS floats of the merge (see WideMerge): T_V operands, two batches of split weights and
// rescales, (M, L, bad) per head, and one float4 per thread.
constexpr size_t wide_merge_floats(int nh) {
  const int ng = kMfmaThreads / (nh * (kD / 4)), sb = 8 * ng;
  const int fin = 3 * (4 * 64 * 8) / 2 + 2 * nh * sb + 2 * nh;
  return (size_t)((fin + 4 * nh + 3) / 4 * 4 + 4 * kMfmaThreads);
}

// Dynamic LDS: key records | value tiles | alpha^K | alpha^V   (front, also the merge scratch) |
// query limb planes | channel weights | value operands | [O' if it does not fit over the key
// records] | [append scratch].  The cache streams into LDS while the query planes are built, so
// the planes' scratch shares the value-operand region (written only after the planes).  The
// transfers write whole 1 KiB blocks of the cache regions.
struct MfmaLds {
  int off_v, off_ak, off_av, off_ql, off_qc, off_pb, off_ob, ob_stride, off_es;
  size_t total;
  bool fits() const { return total <= kMfmaLdsMax; }
};

inline MfmaLds mfma_lds(int nt, int ntile, int np, int rk, int rv, bool append) {
  const int nh = 4 * nt, s = 128 * ntile;
  const size_t qc_bytes = (size_t)nh * kD * sizeof(float);
  MfmaLds l;
  l.off_v = s * rk;
  l.off_ak = l.off_v + s * rv;
  l.off_av = l.off_ak + 2 * s;
  const size_t front = std::max((size_t)l.off_av + 2 * s, wide_merge_floats(nh) * sizeof(float));
  l.off_ql = (int)((front + 255) / 256 * 256);
  l.off_qc = l.off_ql + 4 * nh * 2 * np * 64;
  l.off_pb = l.off_qc + (int)qc_bytes;
  size_t off = (size_t)l.off_pb + std::max((size_t)(s / 64) * nt * 64 * 16, qc_bytes);
  l.ob_stride = 8 * rv;
  const size_t ob_bytes = (size_t)2 * nh * l.ob_stride * 4;    // O' per (half, head, value bit)
  l.off_ob = ob_bytes <= (size_t)s * rk ? 0 : (int)off;
  if (l.off_ob) off += ob_bytes;
  l.off_es = (int)off;
  l.total = off + (append ? kAppendScratchBytes : 0);
  return l;
}

// How a call runs on the matrix-core kernel (records of at most kMfmaRecord bytes).
struct MfmaPlan {
  int nt;         // workgroups take 4 nt query heads of a KV head ...
  int hg;         // ... in hg groups
  int ntile;      // 128 ntile tokens per chunk
  int np;         // record dwords per lane group of the key operands (16 np bytes of record)
  bool fused;     // an append runs inside the decode launch (one workgroup row per KV head)
};

// Heads: eight per workgroup when there are more than four, records are at most 96 bytes and LDS
// holds them, else four (over 96 bytes LDS holds four; and so with values much wider than the
// keys, where the value sums find no room over the key records: 64-byte keys with 96-byte values
// need 172 KiB for eight heads, 118 for four).  Four heads and 512 tokens fit every pair of records.
// Tokens: 512 per chunk while the capacity's chunks all find a compute unit of their own and a row
// has at most 64 of them, else 1024 (a chunk's products take as long as its tokens are many: 16384
// tokens, 8 KV heads, 12.8 us against 14.5; but runs of two 512-token chunks take longer than one of
// 1024, 24000 tokens 16.4 against 14.5, and one workgroup merges a row's partials, 131072 tokens of
// one KV head with 8 query heads 35.5 against 27.6); records over 96 bytes in all take 512 (LDS).
inline MfmaPlan mfma_plan(int rk, int rv, int G, int64_t kv_rows, int64_t cap, bool append) {
  MfmaPlan p;
  const int wide = std::max(rk, rv);
  p.np = wide > 96 ? 8 : wide > 64 ? 6 : (rk / 4 + 3) / 4;
  p.nt = G > 4 && wide <= 96 &&
         mfma_lds(2, 4, p.np, rk, rv, append && G <= kMaxNH).fits() ? 2 : 1;
  p.hg = (G + 4 * p.nt - 1) / (4 * p.nt);
  p.fused = append && p.hg == 1;
  const bool few = kv_rows * p.hg * ((cap + 511) / 512) <= kComputeUnits && cap <= 32 * 1024;
  p.ntile = p.np <= 4 && rk + rv <= 96 && !few &&
            mfma_lds(p.nt, 8, p.np, rk, rv, p.fused).fits() ? 8 : 4;
  return p;
}

// Whether the launch deals every row the same number of workgroups, which need no length for it:
// when every chunk of the capacity can have one on its own compute unit, the batch is one sequence
// (its rows are equally long), or a row is one chunk.  (Dealt by the lengths, one-chunk rows wait
// for them before their first other load: 64 sequences of 512 tokens, 8 KV heads, capacity 1024,
// 29.9 us against 27.7.)  And when the rows alone take four rounds of the chip or more and no row
// can be longer than that in chunks: one run per row balances then within the last row's length,
// and reading the lengths of a thousand sequences in every workgroup costs more (2048 sequences of
// 300 tokens, 8 KV heads, capacity 2048: 2397 us, 799 now).
inline bool evenly_dealt(int batch, int64_t rows, int64_t chunks) {
  return batch == 1 || chunks == 1 || rows * chunks <= kComputeUnits ||
         (rows >= 4 * kComputeUnits && kComputeUnits * chunks <= rows);
}

// ceil(n / q) for 0 <= n < 2^20, 1 <= q < 2^20, rq = 1 / q within a few ulps: the product is within
// one of the quotient (2^21 (2^-23 + 2^-22)), the remainder says which way.
AATC_PLAN_HD inline int runs_of_row(int n, int q, float rq) {
  const int a = n + q - 1;
  const int t = (int)((float)a * rq), r = a - t * q;
  return t + (r >= q ? 1 : 0) - (r < 0 ? 1 : 0);
}

// Ragged batches: a row's chunks go in runs of q, a workgroup each, q chosen by every workgroup
// from the lengths.  A compute unit holds one workgroup at a time, so runs that take r rounds of
// the chip last about r (q + 1) chunk times (building a run's query planes and merging it cost
// about a chunk's time).  The smallest q whose runs fit the grid of r rounds is taken for the
// cheapest r: a run longer than needed costs every compute unit, and with more rows than half the
// compute units two rounds of long runs can cost more than one (17 sequences of 16384 down to
// 5800 tokens, 8 KV heads: 8 chunks a run, 59 us; 12 by a closed form over two rounds, 146).
struct RunPlan {
  int q, runs;                          // chunks per run, runs of the batch
};

// count(q): the runs of at most q chunks that the batch takes (falling in q).  tot: chunks of
// all rows, longest: of one row, limit: workgroups, at least as many as rows.
template <class Count>
AATC_PLAN_HD inline RunPlan smallest_runs(int tot, int rows, int longest, int limit, Count count) {
  int lo = (tot + limit - 1) / limit;   // (the average: no smaller one fits)
  RunPlan p{lo, count(lo)};
  if (p.runs <= limit) return p;
  // sum ceil(n / q) <= tot / q + rows
  const int closed = limit > rows ? (tot + limit - rows - 1) / (limit - rows) : longest;
  int hi = closed < longest ? closed : longest;
  p.runs = -1;
  while (hi - lo > 1) {
    const int mid = (lo + hi) / 2, n = count(mid);
    if (n <= limit) hi = mid, p.runs = n;
    else lo = mid;
  }
  p.q = hi;
  if (p.runs < 0) p.runs = count(hi);
  return p;
}

template <class Count>
AATC_PLAN_HD inline RunPlan choose_runs(int tot, int rows, int longest, int grid, Count count) {
  RunPlan best{1, 0};
  int64_t cost = INT64_MAX;
  for (int r = (rows + kComputeUnits - 1) / kComputeUnits; kComputeUnits * (r - 1) < grid; ++r) {
    const int limit = grid < kComputeUnits * r ? grid : kComputeUnits * r;
    if (cost <= (int64_t)r * ((tot + limit - 1) / limit + 1)) break;   // (more rounds cost no less)
    const RunPlan p = smallest_runs(tot, rows, longest, limit, count);
    if ((int64_t)r * (p.q + 1) < cost) {
      cost = (int64_t)r * (p.q + 1);
      best = p;
    }
  }
  return best;
}

// Workgroups of a ragged launch (a multiple of 8): one round while that gives every row two runs,
// else one round more than the rows need, for choose_runs to take or leave (workgroups without a
// run exit).
inline int64_t ragged_grid(int64_t rows, int64_t chunks) {
  const int64_t rounds = 2 * rows <= kComputeUnits ? 1 : (rows + kComputeUnits - 1) / kComputeUnits + 1;
  return (std::min(rows * chunks, kComputeUnits * rounds) + 7) / 8 * 8;
}

// The run of a workgroup, -1 for none.  Workgroups are dealt to the 8 XCDs round robin:
// consecutive runs (of one row, mostly) go to one XCD, and every XCD gets the same share of the
// runs (dealt by the grid instead, the workgroups without a run were those of the last XCDs, and
// the others took two rounds).
AATC_PLAN_HD inline int run_of_block(int block, int runs) {
  const int share = (runs + 7) / 8, i = block >> 3, run = (block & 7) * share + i;
  return i < share && run < runs ? run : -1;
}

}  // namespace aatc
