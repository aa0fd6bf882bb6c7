// Host build of the decode's shape decisions (decode_plan.h) for the CPU tests.
#include <cmath>
#include <cstdlib>

#include "decode_plan.h"

using namespace aatc;

// Pairs of record sizes for which the plan does not fit the kernel: LDS over the limit, the value
// sums or the regions out of place, or heads and records that its instances do not take.
extern "C" int plan_misfits(int G, int64_t kv_rows, int64_t cap, int append) {
  int bad = 0;
  for (int rk = 4; rk <= kMfmaRecord; rk += 4)
    for (int rv = 4; rv <= kMfmaRecord; rv += 4) {
      const MfmaPlan p = mfma_plan(rk, rv, G, kv_rows, cap, append != 0);
      const MfmaLds l = mfma_lds(p.nt, p.ntile, p.np, rk, rv, p.fused);
      const int nh = 4 * p.nt, s = 128 * p.ntile;
      bool ok = l.fits() && (p.nt == 1 || p.nt == 2) && (p.ntile == 4 || p.ntile == 8);
      ok = ok && nh * p.hg >= G && nh * (p.hg - 1) < G;              // every head, no empty group
      ok = ok && (!p.fused || (append && p.hg == 1));
      ok = ok && 16 * p.np >= rk && (p.np <= 4 || p.ntile == 4) && (p.np < 8 || p.nt == 1);
      ok = ok && l.off_v >= s * rk && l.off_ak >= l.off_v + s * rv && l.off_ql >= l.off_av + 2 * s;
      const size_t ob = (size_t)2 * nh * 8 * rv * 4;
      ok = ok && (l.off_ob == 0 ? ob <= (size_t)s * rk : l.off_ob + ob <= l.total);
      ok = ok && (!p.fused || l.off_es + kAppendScratchBytes <= l.total);
      bad += !ok;
    }
  return bad;
}

// The plan of one call: nt | hg << 8 | ntile << 16 | np << 24.
extern "C" int plan_of(int rk, int rv, int G, int64_t kv_rows, int64_t cap, int append, int* fused) {
  const MfmaPlan p = mfma_plan(rk, rv, G, kv_rows, cap, append != 0);
  *fused = p.fused;
  return p.nt | p.hg << 8 | p.ntile << 16 | p.np << 24;
}

// The runs of a ragged batch: rows of nch[i] chunks (rps rows of each), `chunks` of capacity.
// Returns the run length; *grid and *runs as launched and as dealt.
extern "C" int runs_of(const int* nch, int batch, int rps, int64_t chunks, int64_t* grid, int* runs) {
  const int rows = batch * rps;
  *grid = ragged_grid(rows, chunks);
  int tot = 0, longest = 0;
  for (int i = 0; i < batch; ++i) tot += nch[i] * rps, longest = std::max(longest, nch[i]);
  const RunPlan p = choose_runs(tot, rows, longest, (int)*grid, [&](int q) {
    int n = 0;
    for (int i = 0; i < batch; ++i) n += (nch[i] + q - 1) / q;
    return n * rps;
  });
  *runs = p.runs;
  return p.q;
}

extern "C" int block_run(int block, int runs) { return run_of_block(block, runs); }

extern "C" int dealt_evenly(int batch, int64_t rows, int64_t chunks) { return evenly_dealt(batch, rows, chunks); }

// Pairs (n, q) for which runs_of_row is not ceil(n / q), with 1 / q off by ulps either way.
extern "C" int64_t wrong_quotients(int n_max, int q_max, int step_n, int step_q, int ulps) {
  int64_t bad = 0;
  for (int q = 1; q < q_max; q += q < 64 ? 1 : step_q)
    for (int e = -ulps; e <= ulps; ++e) {
      float rq = 1.f / (float)q;
      for (int k = 0; k < std::abs(e); ++k) rq = std::nextafterf(rq, e > 0 ? 2.f : 0.f);
      for (int n = 0; n < n_max; n += step_n)
        for (int m = n; m < n + 2; ++m) bad += runs_of_row(m, q, rq) != (m + q - 1) / q;
      for (int k = 1; (int64_t)k * q < n_max && k < 2000; ++k)
        for (int m = k * q - 1; m <= k * q + 1; ++m) bad += runs_of_row(m, q, rq) != (m + q - 1) / q;
    }
  return bad;
}
