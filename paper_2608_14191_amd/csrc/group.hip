// AATC under head-group transforms (Sec. 5.1, the remark on head groups; Sec. 5.2, one
// token scale per head group; Sec. 6: G = 2 groups for Llama's 8 KV heads, 1 for Qwen's 4).
//
// A group is gkv consecutive KV heads; its token is the concatenation of their vectors
// (d = 128 gkv elements, KV head kk of the group at [128 kk, 128 kk + 128)).  Encode and
// decode follow Alg. 1 on those d-element vectors with the group's transform:
//   - group_encode_mfma_kernel: h = T^T x exactly rounded (the integer products of the
//     per-head path, over d elements), one alpha per (token, group), codes packed into
//     one token-major record per (token, group); group_encode_exact_kernel redoes the few
//     tokens it cannot certify;
//   - group_query_kernel: per query head, the channel weights W_c = q~_c s_c 2^(1-b_c)
//     scale log2(e) of q~ = T[block]^T q (App. B's effective query; the query of KV head k
//     lives in block k % gkv of its group);
//   - group_split_mfma_kernel: per (sequence, group, 256-token split) the scores of every
//     query head of the group, the split's softmax and the transformed-domain value sums,
//     on the matrix cores (fp16 operands) with the records staged in LDS; the VALU kernels
//     group_split_wide_kernel and group_split_kernel (64-token chunks, an online softmax)
//     take wider codes, or records too long for LDS;
//   - group_merge_kernel: per (sequence, query head) the merge of the split partials and the
//     inverse transform o = T[block] o~, by 64-channel chunks.
#include <algorithm>
#include <atomic>
#include <type_traits>

#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include "encode_core.h"
#include "group.h"
#include "group_launch.h"

namespace aatc {
namespace {

constexpr int kGThreads = 256;
constexpr int kGQThreads = 1024;                  // query kernel: sixteen waves of 8 rows
constexpr int kGChunk = 64;                       // tokens staged per chunk (one per lane)

__device__ inline float g_wave_max(float v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  return v;
}
__device__ inline float g_wave_sum(float v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// The signed code of a channel at record bit `off`, width b (1..16), from the record's
// dwords in LDS (the row has one padding dword after the record).
__device__ inline int record_code(const uint32_t* row, int off, int b) {
  const uint32_t w0 = row[off >> 5], w1 = row[(off >> 5) + 1];
  const uint32_t v = __builtin_amdgcn_alignbit(w1, w0, (uint32_t)(off & 31));   // (w1:w0) >> off
  return __builtin_amdgcn_sbfe((int)v, 0, b);                                   // sign-extended
}

// ---------------------------------------------------------------------------------------
// Encode on the matrix cores: the integer product of the per-head bulk encode (token in fixed
// point X = x 2^S, transform as the integers T 2^22, int8 limbs of both, int32 sums by weight,
// H = sum_j X_j Tq_jc) over d = 128 gkv elements.  bf16: three limbs of X (max |X| in
// [2^21, 2^22)), fp32: four ([2^29, 2^30)).  |H| can reach 2^53 (bf16) or 2^61 (fp32): it is
// formed in fp64 within 2^9, and E = sum_j |x_j 2^S - X_j| bounds |H - H_exact| by E 2^22 (plus
// those roundings).  A token whose E is 0 (bf16) has its exact H; for the others the scale and
// every code are certified against the bound, and the few that fail (0.2 % of key tokens at
// d = 512, bf16) get the scale mark kGRedo, which group_encode_exact_kernel, launched next,
// redoes exactly.
//
// A workgroup of eight waves takes 16 TT tokens against all channels: the X limbs in LDS in
// operand order (96 KiB at d = 512 and 64 tokens), shared by the waves; a wave owns every
// eighth tile of 16 channels and reads their transform columns straight from the parameter
// block into operands (nothing to share, and the limbs take a few byte permutes per 64
// products), so the transform is read once per 16 TT tokens.  What bounds it: the products
// (bf16: 9 x 8 per 16 x 16 outputs, 18 us per 8192 tokens and two groups).  Measured, 8192
// tokens, two groups of 512 channels, K and V: 5890 us before (fp64 VALU products, a wave per
// two tokens).
// ---------------------------------------------------------------------------------------
typedef int gi4 __attribute__((ext_vector_type(4)));
constexpr uint16_t kGRedo = 0xFFFFu;             // (an fp16 NaN: no token scale has it)
constexpr int kGEncWaves = 8;

__device__ inline float g_cross_row_max(float v) {      // over lanes l, l ^ 16, l ^ 32, l ^ 48
  auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
  r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ inline float g_cross_row_sum(float v) {
  auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Sixteen consecutive elements of a token as fp32.
__device__ inline void g_load16(const void* x, int dtype, int64_t at, bool vec, float (&v)[16]) {
  if (vec && dtype == AATC_BF16) {
    const uint4* p = reinterpret_cast<const uint4*>(static_cast<const uint16_t*>(x) + at);
    const uint4 a = p[0], b = p[1];
    const uint32_t w[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      v[2 * i] = __uint_as_float(w[i] << 16);
      v[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
    }
  } else if (vec) {
    const float4* p = reinterpret_cast<const float4*>(static_cast<const float*>(x) + at);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float4 a = p[i];
      v[4 * i] = a.x, v[4 * i + 1] = a.y, v[4 * i + 2] = a.z, v[4 * i + 3] = a.w;
    }
  } else {
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = load_elem(x, dtype, at + i);
  }
}

// The limbs (balanced int8 digits, lowest first) of four integers |v| <= 2^30 as one dword per
// limb: byte e of limb a of v_e.
template <int XL>
__device__ inline void g_limbs4(const int (&v)[4], uint32_t (&out)[XL]) {
  uint32_t y[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) y[e] = (uint32_t)v[e] + (XL == 3 ? 0x8080u : 0x808080u);
  const uint32_t l01 = __builtin_amdgcn_perm(y[1], y[0], 0x05010400u);
  const uint32_t l23 = __builtin_amdgcn_perm(y[3], y[2], 0x05010400u);
  const uint32_t h01 = __builtin_amdgcn_perm(y[1], y[0], 0x07030602u);
  const uint32_t h23 = __builtin_amdgcn_perm(y[3], y[2], 0x07030602u);
  out[0] = __builtin_amdgcn_perm(l23, l01, 0x05040100u) ^ 0x80808080u;
  out[1] = __builtin_amdgcn_perm(l23, l01, 0x07060302u) ^ 0x80808080u;
  out[2] = __builtin_amdgcn_perm(h23, h01, 0x05040100u) ^ (XL == 3 ? 0u : 0x80808080u);
  if constexpr (XL == 4) out[3] = __builtin_amdgcn_perm(h23, h01, 0x07060302u);
}

template <int NC, bool BF16, int TT>
__global__ __launch_bounds__(64 * kGEncWaves) __attribute__((amdgpu_waves_per_eu(2, 2)))
void group_encode_mfma_kernel(const void* __restrict__ params, const void* __restrict__ x,
                              int64_t n_tok, int64_t x_stride, int vec,
                              uint8_t* __restrict__ codes, uint16_t* __restrict__ alpha,
                              int64_t cap, int64_t pos) {
  constexpr int D = 64 * NC;
  constexpr int XL = BF16 ? 3 : 4, NS = XL + 2;     // limbs of X, limb-product sums
  constexpr int NT = 64 * kGEncWaves;
  constexpr int TOK = 16 * TT;                      // tokens of the workgroup
  constexpr int NCT = D / 16 / kGEncWaves;          // channel tiles per wave
  constexpr int WPT = kGEncWaves / TT;              // waves that stage one token tile
  constexpr int KPW = (NC + WPT - 1) / WPT;         // 64-element pieces each of them stages
  constexpr int DT = BF16 ? AATC_BF16 : AATC_F32;
  extern __shared__ __align__(16) uint8_t smem[];   // X limbs [XL][NC][TT][64 lanes][16], then
                                                    // the record rows [TOK][R / 4 + 1]
  __shared__ float sx[TOK][WPT];                    // per token: the pieces' max |x|, then E
  __shared__ float se[TOK][WPT];
  __shared__ float sm[3][TOK][kGEncWaves];          // per token and wave: max |u| and its bounds
  __shared__ unsigned sbad[TOK];
  __shared__ uint16_t sa[TOK];                      // the scales
  const int g = blockIdx.y, tid = threadIdx.x, lane = tid & 63, n = lane & 15, kg = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t t0 = (int64_t)blockIdx.x * TOK;
  const GroupParams* gp = group_params(params, g);
  if (gp->max_bits > 8) {
    // Codes wider than 8 bits need not fit a four-channel field: every token to the exact
    // kernel (uniform over the grid).
    if (tid < TOK && t0 + tid < n_tok) alpha[(int64_t)g * cap + pos + t0 + tid] = kGRedo;
    return;
  }
  const int rw = gp->record_bytes >> 2, rs = rw + 1;
  // (1) Stage X: wave (tile tt, piece wk) holds its token's pieces kc = wk + WPT i in registers
  //     until the token's maximum is known.
  {
    const int tt = wave % TT, wk = wave / TT, t = 16 * tt + n;
    const bool ok = t0 + t < n_tok;
    const int64_t at = (t0 + (ok ? t : 0)) * x_stride + (int64_t)g * D + 16 * kg;
    float xv[KPW][16], m = 0.f;
#pragma unroll
    for (int i = 0; i < KPW; ++i) {
      const int kc = wk + WPT * i;
      if (kc < NC) g_load16(x, DT, at + 64 * kc, vec != 0, xv[i]);      // (uniform)
    }
#pragma unroll
    for (int i = 0; i < KPW; ++i)
      if (wk + WPT * i < NC) {
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          xv[i][e] = ok ? xv[i][e] : 0.f;
          m = fmaxf(m, fabsf(xv[i][e]));
        }
      }
    m = g_cross_row_max(m);
    if (kg == 0) sx[t][wk] = m;
    if (tid < TOK) sbad[tid] = 0u;
    __syncthreads();
    m = sx[t][0];
#pragma unroll
    for (int w = 1; w < WPT; ++w) m = fmaxf(m, sx[t][w]);
    const int S = token_shift(m) + 8 * (XL - 3);
    const float sc = ldexpf(1.f, min(max(S, -kTFrac), 100 - kTFrac));
    float E = 0.f;
#pragma unroll
    for (int i = 0; i < KPW; ++i) {
      const int kc = wk + WPT * i;
      if (kc >= NC) break;
      uint32_t lb[XL][4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        int v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float xe = xv[i][4 * q + e], r = rintf(xe * sc);
          E += fabsf(fmaf(xe, sc, -r));            // (exact: at most 24 significant bits)
          v[e] = (int)r;
        }
        uint32_t o[XL];
        g_limbs4<XL>(v, o);
#pragma unroll
        for (int a = 0; a < XL; ++a) lb[a][q] = o[a];
      }
#pragma unroll
      for (int a = 0; a < XL; ++a)
        *reinterpret_cast<uint4*>(smem + (((size_t)(a * NC + kc) * TT + tt) * 64 + lane) * 16) =
            make_uint4(lb[a][0], lb[a][1], lb[a][2], lb[a][3]);
    }
    E = g_cross_row_sum(E);
    if (kg == 0) se[t][wk] = E;
  }
  __syncthreads();
  // (2) Products, channel tile by channel tile: u_c = fl32(fl32(H) / s_c) (r_c 2^(S + 22)) of
  //     channels 16 ct + 4 kg + i of tokens 16 tt + n stays in registers.
  float uv[NCT][TT][4];
  {
    const int4* tq = reinterpret_cast<const int4*>(gp->Tqt);
    int4 raw[4];
    auto fetch = [&](int step, int4 (&r)[4]) {     // columns of tile step / NC, piece step % NC
      const int ct = wave + kGEncWaves * (step / NC), kc = step % NC;
      const int4* p = tq + ((size_t)(16 * ct + n) * D + 64 * kc + 16 * kg) / 4;
#pragma unroll
      for (int q = 0; q < 4; ++q) r[q] = p[q];
    };
    fetch(0, raw);
#pragma unroll
    for (int it = 0; it < NCT; ++it) {
      gi4 acc[TT][NS];
#pragma unroll
      for (int tt = 0; tt < TT; ++tt)
#pragma unroll
        for (int k = 0; k < NS; ++k) acc[tt][k] = (gi4){0, 0, 0, 0};
#pragma unroll 1
      for (int kc = 0; kc < NC; ++kc) {
        const int step = it * NC + kc;
        gi4 a[3];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int v[4] = {raw[q].x, raw[q].y, raw[q].z, raw[q].w};
          uint32_t o[3];
          g_limbs4<3>(v, o);
#pragma unroll
          for (int l = 0; l < 3; ++l) a[l][q] = (int)o[l];
        }
        __builtin_amdgcn_sched_barrier(0);          // (the next step's loads go out now)
        if (step + 1 < NCT * NC) fetch(step + 1, raw);
        gi4 b[2][XL];
        auto load_b = [&](int tt, gi4 (&bt)[XL]) {
#pragma unroll
          for (int l = 0; l < XL; ++l)
            bt[l] = *reinterpret_cast<const gi4*>(smem + (((size_t)(l * NC + kc) * TT + tt) * 64 + lane) * 16);
        };
        load_b(0, b[0]);
#pragma unroll
        for (int tt = 0; tt < TT; ++tt) {
          if (tt + 1 < TT) load_b(tt + 1, b[(tt + 1) & 1]);
          __builtin_amdgcn_sched_barrier(0);
          const gi4 (&bt)[XL] = b[tt & 1];
          auto mac = [&](int t, int xa) {
            acc[tt][xa + t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[t], bt[xa], acc[tt][xa + t], 0, 0, 0);
          };
          // (a product's sum is never the previous product's)
#pragma unroll
          for (int xa = XL - 1; xa >= 0; --xa) mac(2, xa);
          mac(1, 0);
          mac(0, 0);
#pragma unroll
          for (int xa = XL - 1; xa >= 1; --xa) mac(1, xa);
#pragma unroll
          for (int xa = 1; xa < XL; ++xa) mac(0, xa);
        }
      }
      const int c0 = 16 * (wave + kGEncWaves * it) + 4 * kg;
      const float4 is4 = *reinterpret_cast<const float4*>(gp->inv_s + c0);
      const float is[4] = {is4.x, is4.y, is4.z, is4.w};
#pragma unroll
      for (int tt = 0; tt < TT; ++tt)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          // (one sum at a time: two do not fit 32 bits at d = 512)
          double H = (double)acc[tt][NS - 1][i];
#pragma unroll
          for (int k = NS - 2; k >= 0; --k) H = fma(H, 256.0, (double)acc[tt][k][i]);
          // (kept here: sunk to its uses, the five sums lived on instead of u, 137 registers
          // spilled at d = 512, 290 MB of scratch writes per 32768 tokens, 171 us instead of 147
          // for 8192 tokens, K and V)
          float u = (float)H * is[i];
          asm volatile("" : "+v"(u));
          uv[it][tt][i] = u;
        }
    }
  }
  // (3) Per token: the largest |u| and, for tokens with an error bound, the range of the exact
  //     one, over this wave's channels, then over the waves.
  float eH[TT];                                     // bound of |H - H_exact|, 0 when exact
#pragma unroll
  for (int tt = 0; tt < TT; ++tt) {
    float E = se[16 * tt + n][0];
#pragma unroll
    for (int w = 1; w < WPT; ++w) E += se[16 * tt + n][w];
    // (2^-13 in units of 2^22: the fp64 roundings of H, which pass 2^53 only with E > 0 or
    // fp32 input; the factor covers E's own rounding and the fp32 products below)
    eH[tt] = (BF16 && E == 0.f) ? 0.f : (E + 0x1p-13f) * (1.f + 0x1p-14f) * 0x1p22f;
    float am = 0.f, lo = 0.f, hi = 0.f;
#pragma unroll
    for (int it = 0; it < NCT; ++it) {
      const int c0 = 16 * (wave + kGEncWaves * it) + 4 * kg;
      const float4 is4 = *reinterpret_cast<const float4*>(gp->inv_s + c0);
      const float is[4] = {is4.x, is4.y, is4.z, is4.w};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float u = fabsf(uv[it][tt][i]);       // (0 on dropped channels)
        am = fmaxf(am, u);
        hi = fmaxf(hi, fmaf(eH[tt], is[i], u));
        lo = fmaxf(lo, fmaf(-eH[tt], is[i], u));
      }
    }
    am = g_cross_row_max(am);
    lo = g_cross_row_max(lo);
    hi = g_cross_row_max(hi);
    if (kg == 0) {
      sm[0][16 * tt + n][wave] = am;
      sm[1][16 * tt + n][wave] = lo;
      sm[2][16 * tt + n][wave] = hi;
    }
  }
  __syncthreads();                                  // (the X limbs are consumed too)
  uint32_t* rec = reinterpret_cast<uint32_t*>(smem);
  for (int i = tid; i < TOK * rs; i += NT) rec[i] = 0u;
  // (4) Scale and codes; channels 16 ct + 4 kg .. + 3 are one bit field of <= 32 bits.
  const bool midrise = gp->quantizer == AATC_QUANT_MIDRISE;
  uint32_t field[NCT][TT];
#pragma unroll
  for (int tt = 0; tt < TT; ++tt) {
    const int t = 16 * tt + n;
    float mx = sx[t][0], am = 0.f, lo = 0.f, hi = 0.f;
#pragma unroll
    for (int w = 1; w < WPT; ++w) mx = fmaxf(mx, sx[t][w]);
#pragma unroll
    for (int w = 0; w < kGEncWaves; ++w) {
      am = fmaxf(am, sm[0][t][w]);
      lo = fmaxf(lo, sm[1][t][w]);
      hi = fmaxf(hi, sm[2][t][w]);
    }
    // With k = S + 22 in [0, 100] every value here is r 2^k of the canonical sequence, a normal
    // fp32 number or zero; other tokens are redone.
    const int k = token_shift(mx) + 8 * (XL - 3) + kTFrac;
    const float amax_r = ldexpf(am, -k);
    const __half a16 = token_alpha(amax_r);
    const float inv_ak = ldexpf(inverse_alpha(a16), -k);
    // (below 22 the scale 2^S is below 1 and E could underflow; eH is NaN with a NaN or infinite
    // element)
    bool bad = !(mx < INFINITY && k >= kTFrac && k <= 100 && eH[tt] < INFINITY);
    if (eH[tt] > 0.f) {
      const float lo_r = ldexpf(lo, -k) - 0x1p-21f * amax_r;
      const float hi_r = ldexpf(hi, -k) + 0x1p-21f * amax_r + 0x1p-140f;
      bad |= __half_as_ushort(token_alpha(fmaxf(lo_r, 0.f))) != __half_as_ushort(token_alpha(hi_r));
    }
    const float ea = eH[tt] * inv_ak;
    auto codes_of = [&](auto certify, auto mid_rise) {
      constexpr bool CERT = decltype(certify)::value, MR = decltype(mid_rise)::value;
#pragma unroll
      for (int it = 0; it < NCT; ++it) {
        const int c0 = 16 * (wave + kGEncWaves * it) + 4 * kg;
        uint32_t b4 = *reinterpret_cast<const uint32_t*>(gp->bits + c0);
        const float4 is4 = *reinterpret_cast<const float4*>(gp->inv_s + c0);
        const float is[4] = {is4.x, is4.y, is4.z, is4.w};
        uint32_t f = 0u, sh = 0u;
#pragma unroll
        for (int i = 0; i < 4; ++i, b4 >>= 8) {
          const uint32_t b = b4 & 255u;
          const float p2 = __uint_as_float((126u + max(b, 1u)) << 23);       // 2^(b - 1)
          const float xq = (uv[it][tt][i] * inv_ak) * p2;
          const float xc = __builtin_amdgcn_fmed3f(xq, -p2, p2 - 1.f);
          int code;
          if constexpr (MR) asm("v_cvt_flr_i32_f32 %0, %1" : "=v"(code) : "v"(xc));
          else asm("v_cvt_rpi_i32_f32 %0, %1" : "=v"(code) : "v"(xc));
          f |= ((uint32_t)code & ((1u << b) - 1u)) << sh;                    // (b = 0: nothing)
          sh += b;
          if constexpr (CERT) {
            // the bound in x units plus both evaluations' fp32 roundings, against the distance
            // to the nearest decision boundary (dropped channels: u = 0, 1 / s = 0)
            const float kf = p2 * is[i] * (1.f + 0x1p-20f);
            const float mg = fmaf(kf, ea, fmaf(0x1p-21f, fabsf(xq), 0x1p-22f));
            const float d = fabsf(__builtin_amdgcn_fractf(xq) - 0.5f);
            bad |= eH[tt] > 0.f && (MR ? (kf > 0.f && d >= 0.5f - mg) : (d <= mg));
          }
        }
        field[it][tt] = f;
      }
    };
    const bool cert = __builtin_amdgcn_ballot_w64(eH[tt] > 0.f) != 0ull;
    if (midrise) {
      if (cert) codes_of(std::true_type{}, std::true_type{});
      else codes_of(std::false_type{}, std::true_type{});
    } else {
      if (cert) codes_of(std::true_type{}, std::false_type{});
      else codes_of(std::false_type{}, std::false_type{});
    }
    if (bad) atomicOr(&sbad[t], 1u);
    if (wave == 0 && kg == 0) sa[t] = __half_as_ushort(a16);
  }
  __syncthreads();                                  // (rows cleared)
#pragma unroll
  for (int it = 0; it < NCT; ++it) {
    const int off = gp->bit_off[16 * (wave + kGEncWaves * it) + 4 * kg];
#pragma unroll
    for (int tt = 0; tt < TT; ++tt) {
      uint32_t* w0 = rec + (16 * tt + n) * rs + (off >> 5);
      const uint64_t v = (uint64_t)field[it][tt] << (off & 31);
      if ((uint32_t)v) atomicOr(w0, (uint32_t)v);
      if ((uint32_t)(v >> 32)) atomicOr(w0 + 1, (uint32_t)(v >> 32));
    }
  }
  __syncthreads();
  const int nt = (int)min<int64_t>(TOK, n_tok - t0);
  uint32_t* out = reinterpret_cast<uint32_t*>(codes) + ((int64_t)g * cap + pos + t0) * rw;
  const uint32_t mk = rw > 1 ? (uint32_t)((0x100000000ull + (uint32_t)rw - 1u) / (uint32_t)rw) : 0u;
  for (int i = tid; i < nt * rw; i += NT) {
    const int t = rw > 1 ? (int)__umulhi((uint32_t)i, mk) : i;
    if (!sbad[t]) out[i] = rec[t * rs + (i - t * rw)];
  }
  if (tid < nt)
    alpha[(int64_t)g * cap + pos + t0 + tid] = sbad[tid] ? kGRedo : sa[tid];
}

// The tokens left with the mark kGRedo, exactly: h_c = fl32(sum_j x_j T_jc) from fp64 sums of
// the exact products x_j T_jc, exact while |x|_1 stays below 2^(31 + g) (every product, hence
// every partial sum, is a multiple of 2^(g - 22), g the lowest set bit of the token's elements,
// and |T| <= 1); otherwise an interval test, and the exact accumulator where the interval
// straddles an fp32 rounding boundary.  A workgroup scans `share` marks and takes its
// marked tokens one at a time: thread (part, channel) sums a share of the elements (rows of T
// coalesced over the channels, sixteen in flight), the shares meet in LDS.  (A wave per token
// walked 512 rows in sequence, over 100 us.)
constexpr int kGFixThreads = 1024;
constexpr int kGFixTokens = 64;                    // most marks of a workgroup
template <int NC>
__global__ __launch_bounds__(kGFixThreads) void group_encode_exact_kernel(
    const void* __restrict__ params, const void* __restrict__ x, int dtype, int64_t n_tok,
    int64_t x_stride, uint8_t* __restrict__ codes, uint16_t* __restrict__ alpha, int64_t cap,
    int64_t pos, int share) {
  constexpr int D = 64 * NC;
  constexpr int NP = kGFixThreads / D;              // element shares
  constexpr int JP = (D + NP - 1) / NP;             // elements per share
  constexpr int kRow = D * kMaxBits / 32 + 1;
  static_assert(JP % 16 == 0 || D % NP == 0, "whole shares");
  __shared__ uint16_t list[kGFixTokens];
  __shared__ int n_list, glsb_s;
  __shared__ float xs[D];
  __shared__ double part[NP][D];
  __shared__ float red[kGFixThreads / 64], redl[kGFixThreads / 64];
  __shared__ uint32_t row[kRow];
  __shared__ float hx[D];
  __shared__ uint16_t open_c[D];
  __shared__ int n_open;
  const int g = blockIdx.y, tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const GroupParams* gp = group_params(params, g);
  const int64_t base = (int64_t)blockIdx.x * share;
  if (tid == 0) n_list = 0;
  __syncthreads();
  if (tid < share && base + tid < n_tok &&
      alpha[(int64_t)g * cap + pos + base + tid] == kGRedo)
    list[atomicAdd(&n_list, 1)] = (uint16_t)tid;
  __syncthreads();
  const int cnt = n_list;
  const int rw = gp->record_bytes >> 2;
  const size_t esize = dtype == AATC_BF16 ? 2 : 4;
  for (int li = 0; li < cnt; ++li) {
    const int64_t t = base + list[li];
    const void* xrow = static_cast<const char*>(x) + (t * x_stride + (int64_t)g * D) * esize;
    // The token, its lowest set bit (4096 for a zero token) and |x|_1; the channel's table
    // entries, so that no load is left after the sums.
    int glsb = 4096;
    float l1 = 0.f;
    int b = 0, off = 0;
    float is = 0.f;
    if (tid < D) {
      const float xe = load_elem(xrow, dtype, tid);
      b = gp->bits[tid];
      off = gp->bit_off[tid];
      is = gp->inv_s[tid];
      xs[tid] = xe;
      l1 = fabsf(xe);
      const uint32_t bv = __float_as_uint(xe) & 0x7fffffffu;
      if (bv != 0u) {
        const int ef = (int)(bv >> 23), m = (int)(bv & 0x7fffffu);
        glsb = ef ? ef - 150 + __builtin_ctz((uint32_t)m | 0x800000u) : -149 + __builtin_ctz((uint32_t)m);
      }
    }
    if (tid == 0) {
      glsb_s = 4096;
      n_open = 0;
    }
    for (int i = tid; i < kRow; i += kGFixThreads) row[i] = 0u;
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) glsb = min(glsb, __shfl_xor(glsb, o, 64));
    l1 = g_wave_sum(l1);
    if (lane == 0) redl[wave] = l1;
    __syncthreads();
    if (lane == 0) atomicMin(&glsb_s, glsb);
    const int c = tid % D, pt = tid / D;
    if (pt < NP) {
      double s0 = 0.0, s1 = 0.0;
      const float* tr = gp->T + c;
#pragma unroll 1
      for (int j0 = pt * JP; j0 < (pt + 1) * JP; j0 += 16) {
        float tv[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) tv[k] = tr[(size_t)(j0 + k) * D];
#pragma unroll
        for (int k = 0; k < 16; k += 2) {
          s0 = fma((double)xs[j0 + k], (double)tv[k], s0);
          s1 = fma((double)xs[j0 + k + 1], (double)tv[k + 1], s1);
        }
      }
      part[pt][c] = s0 + s1;
    }
    __syncthreads();
    float h = 0.f;
    bool open = false;                              // not decided by the interval
    if (tid < D) {
      double sv = part[0][tid];
#pragma unroll
      for (int p = 1; p < NP; ++p) sv += part[p][tid];
      l1 = redl[0];
      for (int w = 1; w < kGFixThreads / 64; ++w) l1 += redl[w];
      // The float sum l1 is within 2^-14 relative of |x|_1.
      const double l1d = (double)l1 * (1.0 + 0x1p-14);
      h = (float)sv;
      if (!(l1d < ldexp(1.0, 31 + min(glsb_s, 900)))) {
        // fp64 sum of D exact products: |error| <= D 2^-53 sum |p| <= D 2^-53 |x|_1
        const double bb = l1d * (D * 0x1p-52) + fabs(sv) * 0x1p-51 + 0x1p-1060;
        const float lo = (float)(sv - bb), hi = (float)(sv + bb);
        h = lo;
        open = lo != hi && b > 0;
      }
    }
    if (open) open_c[atomicAdd(&n_open, 1)] = (uint16_t)tid;
    __syncthreads();
    // The open channels by the exact accumulator, one per wave at a time (it holds any sum of
    // up to 512 such products: each is below 2^46 units of its lsb, so 512 of them stay below
    // 2^137, inside its 320 bits).
    for (int k = wave; k < n_open; k += kGFixThreads / 64) {
      const int oc = open_c[k];
      float xl[NC];
#pragma unroll
      for (int i = 0; i < NC; ++i) xl[i] = xs[lane + 64 * i];
      const float e = exact_dot_wave<NC>(xl, gp->Tqt + (size_t)oc * D);
      if (lane == 0) hx[oc] = e;
    }
    __syncthreads();
    if (open) h = hx[tid];
    const float r = h * is;
    const float m = g_wave_max(b > 0 ? fabsf(r) : 0.f);
    if (lane == 0) red[wave] = m;
    __syncthreads();
    float am = red[0];
    for (int w = 1; w < kGFixThreads / 64; ++w) am = fmaxf(am, red[w]);
    const __half a16 = token_alpha(am);
    if (b > 0) {
      const uint32_t q = quantize_code(r, inverse_alpha(a16), b, gp->quantizer == AATC_QUANT_MIDRISE);
      atomicOr(&row[off >> 5], q << (off & 31));
      if ((off & 31) + b > 32) atomicOr(&row[(off >> 5) + 1], q >> (32 - (off & 31)));
    }
    __syncthreads();
    uint32_t* out = reinterpret_cast<uint32_t*>(codes + ((int64_t)g * cap + pos + t) * gp->record_bytes);
    for (int i = tid; i < rw; i += kGFixThreads) out[i] = row[i];
    if (tid == 0) alpha[(int64_t)g * cap + pos + t] = __half_as_ushort(a16);
    __syncthreads();                                // (the row and sums before the next token)
  }
}

// ---------------------------------------------------------------------------------------
// Decode.
// ---------------------------------------------------------------------------------------
struct GroupDecodeArgs {
  const void* params_k;
  const void* params_v;
  const void* q;
  int q_dtype;
  const uint8_t* k_codes;
  const uint16_t* k_alpha;
  const uint8_t* v_codes;
  const uint16_t* v_alpha;
  const int32_t* seq_len;
  int64_t cap;
  int n_q_heads, n_kv_heads, gkv, n_groups, heads;   // heads: query heads per group
  int n_splits;
  int rwk, rwv;                  // record dwords of the key and value caches
  float scale_log2e;
  float* w;                      // workspace regions
  float* cst;
  float* part;
  float* out;
  uint16_t* wop;                 // the weights as fp16 operands of the matrix-core split
  int32_t* wexp;                 //   and their per-head exponents (written when wops)
  int wops;
  float* otl;                    // the region `ot`: second head tile's operands, output shares
};

// The fp16 operands and exponents of a head tile (16 query heads) of one (sequence, group).
// The second tile (more than 16 heads) lies in the output shares' region, which the merge writes,
// after the split: 64 d bytes and 16 exponents of the 4 d heads >= 68 d bytes there.
__device__ inline uint16_t* wop_tile(const GroupDecodeArgs& a, size_t gset, int d, int tile) {
  return tile == 0 ? a.wop + gset * (d / 32) * (2 * 64 * 8)
                   : reinterpret_cast<uint16_t*>(a.otl + gset * a.heads * d);
}
__device__ inline int32_t* wexp_tile(const GroupDecodeArgs& a, size_t gset, int d, int tile) {
  return tile == 0 ? a.wexp + gset * 16
                   : reinterpret_cast<int32_t*>(a.otl + gset * a.heads * d + 16 * d);
}

// The split partial row of (split 0, head), and the merge's arrival count in its header.
__device__ inline float* first_partial_row(const GroupDecodeArgs& a, size_t gset, int hl, int d) {
  return a.part + (gset * a.n_splits * a.heads + hl) * (size_t)(d + kGPH);
}
__device__ inline unsigned* merge_count(const GroupDecodeArgs& a, size_t gset, int hl, int d) {
  return reinterpret_cast<unsigned*>(first_partial_row(a, gset, hl, d)) + 2;
}

// One workgroup per (sequence, query head): W_c for the head's group channels.  Wave w of
// sixteen sums the query against rows 8 w .. 8 w + 7 of the head's block of T (lane l:
// channels l + 64 m, coalesced rows; every load of the wave in flight at once), and the
// sixteen partial sums meet in LDS.
template <int NC>
__global__ __launch_bounds__(kGQThreads) void group_query_kernel(GroupDecodeArgs a) {
  constexpr int D = 64 * NC;
  constexpr int NW = kGQThreads / 64;
  constexpr int RW = 128 / NW;                      // rows of the block per wave
  __shared__ float qs[128];
  __shared__ float part[NW][D];
  __shared__ float red[NW], redm[NW];
  const int h = blockIdx.x, b = blockIdx.y, tid = threadIdx.x, lane = tid & 63;
  const int wave = tid >> 6;
  const int gq = a.n_q_heads / a.n_kv_heads;
  const int k = h / gq, g = k / a.gkv, kk = k % a.gkv, hl = h - g * a.heads;
  const GroupParams* gp = group_params(a.params_k, g);
  if (tid < 128) qs[tid] = load_elem(a.q, a.q_dtype, ((int64_t)b * a.n_q_heads + h) * 128 + tid);
  __syncthreads();
  float acc[NC];
#pragma unroll
  for (int m = 0; m < NC; ++m) acc[m] = 0.f;
  const float* trow = gp->T + (size_t)(kk * 128 + RW * wave) * D + lane;
#pragma unroll
  for (int j = 0; j < RW; ++j) {
    const float qj = qs[RW * wave + j];
#pragma unroll
    for (int m = 0; m < NC; ++m) acc[m] = fmaf(qj, trow[(size_t)j * D + 64 * m], acc[m]);
  }
#pragma unroll
  for (int m = 0; m < NC; ++m) part[wave][lane + 64 * m] = acc[m];
  __syncthreads();
  const bool midrise = gp->quantizer == AATC_QUANT_MIDRISE;
  const size_t rowi = ((size_t)b * a.n_groups + g) * a.heads + hl;
  constexpr int CPT = (D + kGQThreads - 1) / kGQThreads;
  float wvs[CPT];
  float csum = 0.f, wmax = 0.f;
#pragma unroll
  for (int i = 0; i < CPT; ++i) {
    const int c = tid + kGQThreads * i;
    wvs[i] = 0.f;
    if (c < D) {
      float qt = part[0][c];
#pragma unroll
      for (int w = 1; w < NW; ++w) qt += part[w][c];
      const int bc = gp->bits[c];
      const float wv = bc > 0 ? ldexpf(qt * gp->s[c] * a.scale_log2e, 1 - bc) : 0.f;
      a.w[rowi * D + c] = wv;
      csum += midrise ? 0.5f * wv : 0.f;
      wvs[i] = wv;
      wmax = fmaxf(wmax, fabsf(wv));
    }
  }
  csum = g_wave_sum(csum);
  wmax = g_wave_max(wmax);
  if (lane == 0) {
    red[wave] = csum;
    redm[wave] = wmax;
  }
  __syncthreads();
  if (tid == 0) {
    float cs = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) cs += red[w];
    a.cst[rowi] = cs;
    *merge_count(a, (size_t)b * a.n_groups + g, hl, D) = 0u;
  }
  if (a.wops) {
    // The matrix-core split's operands: W 2^e (largest |W| in [2^14, 2^15)) as fp16
    // Wh + Wl, channel c of this head (slot hl % 16 of head tile hl / 16) at block c / 32, lane
    // 16 ((c % 32) / 8) + hl % 16, element c % 8.
    float m = redm[0];
#pragma unroll
    for (int w = 1; w < NW; ++w) m = fmaxf(m, redm[w]);
    int e = 0;
    if (m > 0.f) (void)frexpf(m, &e);
    e = m > 0.f ? 15 - e : 0;
    const size_t gset = (size_t)b * a.n_groups + g;
    uint16_t* wop = wop_tile(a, gset, D, hl >> 4);
    if (tid == 0) wexp_tile(a, gset, D, hl >> 4)[hl & 15] = e;
#pragma unroll
    for (int i = 0; i < CPT; ++i) {
      const int c = tid + kGQThreads * i;
      if (c < D) {
        const float w = ldexpf(wvs[i], e);
        const _Float16 wh = (_Float16)w, wl = (_Float16)(w - (float)wh);
        const int l = 16 * ((c & 31) >> 3) + (hl & 15);
        uint16_t* o = wop + (c >> 5) * (2 * 64 * 8);
        o[l * 8 + (c & 7)] = __builtin_bit_cast(uint16_t, wh);
        o[(64 + l) * 8 + (c & 7)] = __builtin_bit_cast(uint16_t, wl);
      }
    }
  }
}

// One workgroup per (sequence, group, split of kGSplit tokens).  NQ: query heads of a group
// rounded up to a multiple of 4 (the unused ones have zero weights and are not stored).
template <int NC, int NQ>
__global__ __launch_bounds__(kGThreads) void group_split_kernel(GroupDecodeArgs a) {
  constexpr int D = 64 * NC;
  constexpr int HW = NQ / 4;                        // heads scored by each wave
  constexpr int CPT = (D + kGThreads - 1) / kGThreads;   // value channels per thread
  extern __shared__ __align__(16) uint8_t smem[];
  __shared__ float ak[kGChunk], av[kGChunk];
  __shared__ float m_run[NQ], l_run[NQ], fac[NQ], cst[NQ];
  const int split = blockIdx.x, g = blockIdx.y, b = blockIdx.z;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int len = (int)min((int64_t)max(a.seq_len[b], 0), a.cap);
  const int s0 = split * kGSplit;
  if (s0 >= len) return;                            // (whole workgroup, before any barrier)
  const int s1 = min(len, s0 + kGSplit);
  const GroupParams* pk = group_params(a.params_k, g);
  const GroupParams* pv = group_params(a.params_v, g);
  // (partial rows are [(sequence, group)][split][head])
  float* pbase = a.part + ((((size_t)b * a.n_groups + g) * a.n_splits + split) * a.heads) * (D + kGPH);
  const int rwk = a.rwk, rwv = a.rwv;
  if (pk->record_bytes != 4 * rwk || pv->record_bytes != 4 * rwv || pk->d != D || pv->d != D) {
    // caches of another record size than the parameter blocks: NaN outputs
    if (tid < a.heads) pbase[(size_t)tid * (D + kGPH)] = NAN;
    return;
  }
  const int rsk = rwk + 1, rsv = rwv + 1;           // LDS row strides (one padding dword)
  float* wl = reinterpret_cast<float*>(smem);                    // [D][NQ]
  uint32_t* kc = reinterpret_cast<uint32_t*>(wl + D * NQ);       // [kGChunk][rsk]
  uint32_t* vc = kc + kGChunk * rsk;                             // [kGChunk][rsv]
  float* pl = reinterpret_cast<float*>(vc + kGChunk * rsv);      // [kGChunk][NQ]
  uint32_t* kdesc = reinterpret_cast<uint32_t*>(pl + kGChunk * NQ);   // [D]: off | b << 16
  const size_t row0 = ((size_t)b * a.n_groups + g) * a.heads;
  for (int c = tid; c < D; c += kGThreads)
    kdesc[c] = (uint32_t)pk->bit_off[c] | ((uint32_t)pk->bits[c] << 16);
  for (int i = tid; i < D * NQ; i += kGThreads) {
    const int c = i / NQ, h = i % NQ;
    wl[i] = h < a.heads ? a.w[(row0 + h) * D + c] : 0.f;
  }
  if (tid < NQ) {
    m_run[tid] = -INFINITY;
    l_run[tid] = 0.f;
    cst[tid] = tid < a.heads ? a.cst[row0 + tid] : 0.f;
  }
  const int dak = pk->d_active;
  const bool mr_v = pv->quantizer == AATC_QUANT_MIDRISE;
  // This thread's value channels.
  int vb[CPT], vo[CPT];
  float acc[NQ][CPT];
#pragma unroll
  for (int i = 0; i < CPT; ++i) {
    const int c = tid + kGThreads * i;
    vb[i] = c < D ? pv->bits[c] : 0;
    vo[i] = c < D ? pv->bit_off[c] : 0;
#pragma unroll
    for (int h = 0; h < NQ; ++h) acc[h][i] = 0.f;
  }
  const size_t tok0 = ((size_t)b * a.n_groups + g) * (size_t)a.cap;
  const uint32_t* kw = reinterpret_cast<const uint32_t*>(a.k_codes + tok0 * pk->record_bytes);
  const uint32_t* vw = reinterpret_cast<const uint32_t*>(a.v_codes + tok0 * pv->record_bytes);
  for (int c0 = s0; c0 < s1; c0 += kGChunk) {
    const int nc = min(kGChunk, s1 - c0);
    __syncthreads();                                // the previous chunk's LDS is consumed
    for (int i = tid; i < nc * rwk; i += kGThreads) {
      const int t = i / rwk, w = i - t * rwk;
      kc[t * rsk + w] = kw[(size_t)(c0 + t) * rwk + w];
    }
    for (int i = tid; i < nc * rwv; i += kGThreads) {
      const int t = i / rwv, w = i - t * rwv;
      vc[t * rsv + w] = vw[(size_t)(c0 + t) * rwv + w];
    }
    if (tid < kGChunk) {
      kc[tid * rsk + rwk] = 0u;
      vc[tid * rsv + rwv] = 0u;
      float fk = 0.f, fv = 0.f;
      if (tid < nc) {
        fk = __half2float(__ushort_as_half(a.k_alpha[tok0 + c0 + tid]));
        fv = __half2float(__ushort_as_half(a.v_alpha[tok0 + c0 + tid]));
      }
      ak[tid] = fk;
      av[tid] = fv;
    }
    __syncthreads();
    // Scores: lane = token of the chunk, wave w = heads w HW .. w HW + HW - 1.
    {
      const bool ok = lane < nc;
      const uint32_t* krow = kc + (ok ? lane : 0) * rsk;
      float z[HW];
#pragma unroll
      for (int m = 0; m < HW; ++m) z[m] = 0.f;
#pragma unroll 4
      for (int c = 0; c < dak; ++c) {
        const uint32_t dsc = kdesc[c];
        const float cf = (float)record_code(krow, (int)(dsc & 0xffffu), (int)(dsc >> 16));
        const float* wr = wl + c * NQ + wave * HW;
#pragma unroll
        for (int m = 0; m < HW; ++m) z[m] = fmaf(wr[m], cf, z[m]);
      }
#pragma unroll
      for (int m = 0; m < HW; ++m) {
        const int h = wave * HW + m;
        const float zf = ok ? ak[lane] * (z[m] + cst[h]) : -INFINITY;
        const float mold = m_run[h];
        const float mnew = fmaxf(mold, g_wave_max(zf));
        const bool any = mnew > -INFINITY;
        const float p = (ok && any) ? __builtin_amdgcn_exp2f(zf - mnew) : 0.f;
        const float f = (any && mold > -INFINITY) ? __builtin_amdgcn_exp2f(mold - mnew) : (any ? 0.f : 1.f);
        const float ps = g_wave_sum(p);
        pl[lane * NQ + h] = p * av[lane];
        if (lane == 0) {
          m_run[h] = mnew;
          l_run[h] = l_run[h] * f + ps;
          fac[h] = f;
        }
      }
    }
    __syncthreads();
    // Values: thread = value channels tid + 256 i; every token of the chunk.
#pragma unroll
    for (int h = 0; h < NQ; ++h) {
      const float f = fac[h];
#pragma unroll
      for (int i = 0; i < CPT; ++i) acc[h][i] *= f;
    }
#pragma unroll 1
    for (int t = 0; t < nc; ++t) {
      const uint32_t* vrow = vc + t * rsv;
      float cf[CPT];
#pragma unroll
      for (int i = 0; i < CPT; ++i)
        cf[i] = vb[i] > 0 ? (float)record_code(vrow, vo[i], vb[i]) + (mr_v ? 0.5f : 0.f) : 0.f;
      const float* pr = pl + t * NQ;
#pragma unroll
      for (int h = 0; h < NQ; ++h) {
        const float p = pr[h];
#pragma unroll
        for (int i = 0; i < CPT; ++i) acc[h][i] = fmaf(p, cf[i], acc[h][i]);
      }
    }
  }
  __syncthreads();
  // Partial: (m, l) per head, o~_c = s_c 2^(1-b_c) sum_i P_i alpha_i level_ic.
#pragma unroll
  for (int i = 0; i < CPT; ++i) {
    const int c = tid + kGThreads * i;
    if (c < D) {
      const float sc = vb[i] > 0 ? ldexpf(pv->s[c], 1 - vb[i]) : 0.f;
#pragma unroll
      for (int h = 0; h < NQ; ++h)
        if (h < a.heads) pbase[(size_t)h * (D + kGPH) + kGPH + c] = acc[h][i] * sc;
    }
  }
  if (tid < a.heads) {
    pbase[(size_t)tid * (D + kGPH)] = m_run[tid];
    pbase[(size_t)tid * (D + kGPH) + 1] = l_run[tid];
  }
}

// The same split with the records of all 256 tokens in LDS (key records first, then the
// value records in the same rows) and eight waves: lane = token, waves 0-3 score the first
// half of the group's query heads for tokens 0..255 and waves 4-7 the second half (each code
// feeds NQ / 2 independent products), and thread = value channel.  Used when its LDS fits.
constexpr int kGWideThreads = 512;
template <int NC, int NQ>
__device__ inline void group_split_wide_body(const GroupDecodeArgs& a) {
  constexpr int D = 64 * NC;
  constexpr int NT = kGWideThreads;
  constexpr int HH = NQ / 2;                        // heads scored by each half
  constexpr int CPT = (D + NT - 1) / NT;
  static_assert(kGSplit == 256, "four waves of tokens");
  extern __shared__ __align__(16) uint8_t smem[];
  __shared__ float ak[kGSplit], av[kGSplit];
  __shared__ float wred[4][NQ];
  __shared__ float mh[NQ], lh[NQ], cst[NQ];
  const int split = blockIdx.x, g = blockIdx.y, b = blockIdx.z;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int tok = tid & (kGSplit - 1), half = wave >> 2;
  const int len = (int)min((int64_t)max(a.seq_len[b], 0), a.cap);
  const int s0 = split * kGSplit;
  if (s0 >= len) return;                            // (whole workgroup, before any barrier)
  const int nt = min(len, s0 + kGSplit) - s0;
  const GroupParams* pk = group_params(a.params_k, g);
  const GroupParams* pv = group_params(a.params_v, g);
  float* pbase = a.part + ((((size_t)b * a.n_groups + g) * a.n_splits + split) * a.heads) * (D + kGPH);
  const int rwk = a.rwk, rwv = a.rwv;
  if (pk->record_bytes != 4 * rwk || pv->record_bytes != 4 * rwv || pk->d != D || pv->d != D) {
    if (tid < a.heads) pbase[(size_t)tid * (D + kGPH)] = NAN;
    return;
  }
  const int rs = max(rwk, rwv) + 1;                 // LDS row stride (one padding dword)
  float* wl = reinterpret_cast<float*>(smem);                      // [D][NQ]
  uint32_t* rb = reinterpret_cast<uint32_t*>(wl + D * NQ);         // [kGSplit][rs]
  float* pl = reinterpret_cast<float*>(rb + kGSplit * rs);         // [kGSplit][NQ]
  uint32_t* kdesc = reinterpret_cast<uint32_t*>(pl + kGSplit * NQ);   // [D]: off | b << 16
  const size_t row0 = ((size_t)b * a.n_groups + g) * a.heads;
  for (int i = tid; i < D * NQ; i += NT) {
    const int c = i / NQ, h = i % NQ;
    wl[i] = h < a.heads ? a.w[(row0 + h) * D + c] : 0.f;
  }
  for (int c = tid; c < D; c += NT)
    kdesc[c] = (uint32_t)pk->bit_off[c] | ((uint32_t)pk->bits[c] << 16);
  if (tid < NQ) cst[tid] = tid < a.heads ? a.cst[row0 + tid] : 0.f;
  const size_t tok0 = ((size_t)b * a.n_groups + g) * (size_t)a.cap + s0;
  const uint32_t* kw = reinterpret_cast<const uint32_t*>(a.k_codes + tok0 * pk->record_bytes);
  const uint32_t* vw = reinterpret_cast<const uint32_t*>(a.v_codes + tok0 * pv->record_bytes);
  for (int i = tid; i < nt * rwk; i += NT) {
    const int t = i / rwk, w = i - t * rwk;
    rb[t * rs + w] = kw[i];
  }
  if (tid < kGSplit) {
    rb[tid * rs + rwk] = 0u;
    float fk = 0.f, fv = 0.f;
    if (tid < nt) {
      fk = __half2float(__ushort_as_half(a.k_alpha[tok0 + tid]));
      fv = __half2float(__ushort_as_half(a.v_alpha[tok0 + tid]));
    }
    ak[tid] = fk;
    av[tid] = fv;
  }
  __syncthreads();
  // Scores of token `tok` for heads half HH .. half HH + HH - 1.
  const bool ok = tok < nt;
  float z[HH];
  {
    const uint32_t* krow = rb + (ok ? tok : 0) * rs;
#pragma unroll
    for (int h = 0; h < HH; ++h) z[h] = 0.f;
    const int dak = pk->d_active;
    const float* wh = wl + half * HH;
#pragma unroll 2
    for (int c = 0; c < dak; ++c) {
      const uint32_t dsc = kdesc[c];
      const float cf = (float)record_code(krow, (int)(dsc & 0xffffu), (int)(dsc >> 16));
      const float* wc = wh + c * NQ;
      if constexpr (HH % 4 == 0) {
#pragma unroll
        for (int q = 0; q < HH / 4; ++q) {
          const float4 w4 = reinterpret_cast<const float4*>(wc)[q];
          z[4 * q] = fmaf(w4.x, cf, z[4 * q]);
          z[4 * q + 1] = fmaf(w4.y, cf, z[4 * q + 1]);
          z[4 * q + 2] = fmaf(w4.z, cf, z[4 * q + 2]);
          z[4 * q + 3] = fmaf(w4.w, cf, z[4 * q + 3]);
        }
      } else {
#pragma unroll
        for (int h = 0; h < HH; ++h) z[h] = fmaf(wc[h], cf, z[h]);
      }
    }
    const float akt = ak[tok];
#pragma unroll
    for (int i = 0; i < HH; ++i) {
      z[i] = ok ? akt * (z[i] + cst[half * HH + i]) : -INFINITY;
      const float m = g_wave_max(z[i]);
      if (lane == 0) wred[wave & 3][half * HH + i] = m;
    }
  }
  __syncthreads();                                  // (every key record read, maxima in)
  if (tid < NQ) mh[tid] = fmaxf(fmaxf(wred[0][tid], wred[1][tid]), fmaxf(wred[2][tid], wred[3][tid]));
  for (int i = tid; i < nt * rwv; i += NT) {
    const int t = i / rwv, w = i - t * rwv;
    rb[t * rs + w] = vw[i];
  }
  if (tid < kGSplit) rb[tid * rs + rwv] = 0u;
  __syncthreads();
  {
    const float avt = av[tok];
#pragma unroll
    for (int i = 0; i < HH; ++i) {
      const int h = half * HH + i;
      const float p = ok ? __builtin_amdgcn_exp2f(z[i] - mh[h]) : 0.f;
      pl[tok * NQ + h] = p * avt;
      const float ps = g_wave_sum(p);
      if (lane == 0) wred[wave & 3][h] = ps;
    }
  }
  __syncthreads();
  if (tid < NQ) lh[tid] = (wred[0][tid] + wred[1][tid]) + (wred[2][tid] + wred[3][tid]);
  // Values: thread = channels tid + 512 i, every token, every head.
  const bool mr_v = pv->quantizer == AATC_QUANT_MIDRISE;
  int vb[CPT], vo[CPT];
  float acc[NQ][CPT];
#pragma unroll
  for (int i = 0; i < CPT; ++i) {
    const int c = tid + NT * i;
    vb[i] = c < D ? pv->bits[c] : 0;
    vo[i] = c < D ? pv->bit_off[c] : 0;
#pragma unroll
    for (int h = 0; h < NQ; ++h) acc[h][i] = 0.f;
  }
  bool any = false;
#pragma unroll
  for (int i = 0; i < CPT; ++i) any = any || vb[i] > 0;
  if (any) {
#pragma unroll 2
    for (int t = 0; t < nt; ++t) {
      const uint32_t* vrow = rb + t * rs;
      float cf[CPT];
#pragma unroll
      for (int i = 0; i < CPT; ++i)
        cf[i] = vb[i] > 0 ? (float)record_code(vrow, vo[i], vb[i]) + (mr_v ? 0.5f : 0.f) : 0.f;
      const float4* pr = reinterpret_cast<const float4*>(pl + t * NQ);
#pragma unroll
      for (int q = 0; q < NQ / 4; ++q) {
        const float4 p4 = pr[q];
#pragma unroll
        for (int i = 0; i < CPT; ++i) {
          acc[4 * q][i] = fmaf(p4.x, cf[i], acc[4 * q][i]);
          acc[4 * q + 1][i] = fmaf(p4.y, cf[i], acc[4 * q + 1][i]);
          acc[4 * q + 2][i] = fmaf(p4.z, cf[i], acc[4 * q + 2][i]);
          acc[4 * q + 3][i] = fmaf(p4.w, cf[i], acc[4 * q + 3][i]);
        }
      }
    }
  }
  __syncthreads();                                  // (mh, lh written)
#pragma unroll
  for (int i = 0; i < CPT; ++i) {
    const int c = tid + NT * i;
    if (c < D) {
      const float sc = vb[i] > 0 ? ldexpf(pv->s[c], 1 - vb[i]) : 0.f;
#pragma unroll
      for (int h = 0; h < NQ; ++h)
        if (h < a.heads) pbase[(size_t)h * (D + kGPH) + kGPH + c] = acc[h][i] * sc;
    }
  }
  if (tid < a.heads) {
    pbase[(size_t)tid * (D + kGPH)] = mh[tid];
    pbase[(size_t)tid * (D + kGPH) + 1] = lh[tid];
  }
}

template <int NC, int NQ>
__global__ __launch_bounds__(kGWideThreads) void group_split_wide_kernel(GroupDecodeArgs a) {
  group_split_wide_body<NC, NQ>(a);
}

// Loads of one staging pass: dwords i0 + u NT (u < kGStageU) of the records (the index past
// the end clamped to the last dword), all issued before any is used.
constexpr int kGStageU = 24;
template <int NT>
__device__ inline void stage_load(const uint32_t* src, int total, int i0, uint32_t (&v)[kGStageU]) {
#pragma unroll
  for (int u = 0; u < kGStageU; ++u) v[u] = src[min(i0 + u * NT, total - 1)];
}
// Their stores into LDS rows of rs dwords (token t = i / rw as the high half of
// i ceil(2^32 / rw): exact for i < 2^32 / rw).
template <int NT>
__device__ inline void stage_store(uint32_t* rb, int rs, int total, int rw, int i0,
                                   const uint32_t (&v)[kGStageU]) {
  const uint32_t mk = rw > 1 ? (uint32_t)((0x100000000ull + (uint32_t)rw - 1u) / (uint32_t)rw) : 0u;
#pragma unroll
  for (int u = 0; u < kGStageU; ++u) {
    const int i = i0 + u * NT;
    if (i < total) {
      const int t = rw > 1 ? (int)__umulhi((uint32_t)i, mk) : i;
      rb[t * rs + (i - t * rw)] = v[u];
    }
  }
}
// The records of tokens 0 .. nt-1 (rw dwords each, contiguous at src) into LDS rows, one
// round trip per pass of kGStageU dwords per thread.
template <int NT>
__device__ inline void stage_records(uint32_t* rb, int rs, const uint32_t* src, int nt, int rw) {
  const int total = nt * rw;
  for (int i0 = threadIdx.x; i0 < total; i0 += NT * kGStageU) {
    uint32_t v[kGStageU];
    stage_load<NT>(src, total, i0, v);
    stage_store<NT>(rb, rs, total, rw, i0, v);
  }
}

// The same with 16-byte loads (src 16-byte aligned, total >= 4): the whole uint4s of the
// records, the last total % 4 dwords by single loads; kGStage4 uint4 per thread and pass.
constexpr int kGStage4 = 6;
template <int NT>
__device__ inline void stage4_load(const uint32_t* src, int total, int j0, uint4 (&v)[kGStage4],
                                   uint32_t& tail) {
  const uint4* s4 = reinterpret_cast<const uint4*>(src);
  const int n4 = total >> 2;
#pragma unroll
  for (int u = 0; u < kGStage4; ++u) v[u] = s4[min(j0 + u * NT, n4 - 1)];   // (n4 >= 1)
  const int it = 4 * n4 + (int)threadIdx.x;
  tail = it < total ? src[it] : 0u;
}
template <int NT>
__device__ inline void stage4_store(uint32_t* rb, int rs, int total, int rw, int j0,
                                    const uint4 (&v)[kGStage4], uint32_t tail, bool first) {
  const uint32_t mk = rw > 1 ? (uint32_t)((0x100000000ull + (uint32_t)rw - 1u) / (uint32_t)rw) : 0u;
  auto put = [&](int i, uint32_t x) {
    const int t = rw > 1 ? (int)__umulhi((uint32_t)i, mk) : i;
    rb[t * rs + (i - t * rw)] = x;
  };
  const int n4 = total >> 2;
#pragma unroll
  for (int u = 0; u < kGStage4; ++u) {
    const int j = j0 + u * NT;
    if (j < n4) {
      put(4 * j, v[u].x);
      put(4 * j + 1, v[u].y);
      put(4 * j + 2, v[u].z);
      put(4 * j + 3, v[u].w);
    }
  }
  const int it = 4 * n4 + (int)threadIdx.x;
  if (first && it < total) put(it, tail);
}
// The records into LDS rows: 16-byte loads when src is aligned, one round trip per pass.
template <int NT>
__device__ inline void stage_records_any(uint32_t* rb, int rs, const uint32_t* src, int nt, int rw) {
  const int total = nt * rw;
  if (total <= 0) return;
  if ((reinterpret_cast<uintptr_t>(src) & 15u) == 0u && total >= 4) {
    // (every thread takes the first pass: it also carries the tail dwords)
    for (int j0 = threadIdx.x; j0 == (int)threadIdx.x || j0 < (total >> 2); j0 += NT * kGStage4) {
      uint4 v[kGStage4];
      uint32_t tail;
      stage4_load<NT>(src, total, j0, v, tail);
      stage4_store<NT>(rb, rs, total, rw, j0, v, tail, j0 == (int)threadIdx.x);
    }
  } else {
    stage_records<NT>(rb, rs, src, nt, rw);
  }
}

// The same split on the matrix cores (up to 32 query heads per group in NHT tiles of 16, codes
// of at most 12 bits, which fp16 holds exactly): eight waves, the records of all 256 tokens in
// LDS.  The extraction of the codes bounds both product phases, so a second head tile costs
// little (28 heads, batch 4 ragged to 8000 tokens: 136 us on the VALU before).
//   - Scores: v_mfma_f32_16x16x32_f16 with A = the query weights (16 heads x 32 channels)
//     and B = the codes of 16 tokens (32 channels x 16 tokens).  Each head's weights come
//     scaled by a power of two (largest |W| in [2^14, 2^15)) and split into fp16 parts
//     W' = Wh + Wl (written by group_query_kernel), both multiplied with the same codes into
//     one fp32 sum (products exact, |W' - Wh - Wl| <= 2^-22 |W'|).
//   - Values: A = P (16 heads x 32 tokens), P = p alpha^V scaled by a power of two (largest
//     alpha^V of the split in [2^13, 2^14)) and split the same way, B = the codes of 16
//     channels over those 32 tokens.  The midrise half step is 1/2 sum_t P, added once.
// Operand layouts (lane 16 kg + n): A row n, k = 8 kg .. 8 kg + 7; B column n, the same k;
// the 16 x 16 result row 4 kg + i, column n in element i.
// DUAL: key and value records in LDS together; otherwise the value records replace the key
// records after the scores, held in registers until then where their loads are vectors (every
// load of the split is issued at the start either way).  P reuses the weight operands'
// region.  A workgroup whose codes are wider takes the VALU body above (uniform).
typedef _Float16 gh8 __attribute__((ext_vector_type(8)));
typedef float gf4 __attribute__((ext_vector_type(4)));
constexpr int kGPRow = kGSplit + 8;              // halves per head row of P (rows 4 banks
                                                 // apart: conflict-free operand reads)
constexpr size_t kGMfmaLdsCap = 150 * 1024;       // dynamic LDS of the matrix-core split

// The weight operands, later P (both parts, 16 NHT head rows).
template <int NC, int NHT>
inline constexpr size_t kGWopBytes = std::max((size_t)NHT * (64 * NC / 32) * 2 * 64 * 16,
                                              (size_t)2 * 16 * NHT * kGPRow * 2);
template <int NC, int NHT>
inline constexpr size_t group_mfma_lds(int rw_max, bool dual) {
  const size_t rows = (size_t)kGSplit * (rw_max + 1) * 4;
  return kGWopBytes<NC, NHT> + (size_t)2 * 64 * NC * 4 +        // key and value descriptors
         (dual ? 2 * rows : rows);
}

template <int NC, int NHT, bool DUAL>
__global__ __launch_bounds__(kGWideThreads) void group_split_mfma_kernel(GroupDecodeArgs a) {
  constexpr int D = 64 * NC;
  constexpr int NT = kGWideThreads;
  constexpr int NKB = D / 32;                       // channel blocks of the score products
  constexpr int NCB = D / 16;                       // channel blocks of the value products
  constexpr int NQ = 16 * NHT;                      // head slots
  constexpr int W4 = NKB * 128 / NT;                // 16-byte operand loads per thread and tile
  static_assert(kGSplit == 256, "eight waves of 32 tokens");
  static_assert(NKB * 128 % NT == 0, "whole operand loads");
  extern __shared__ __align__(16) uint8_t smem[];
  __shared__ float ak[kGSplit], av[kGSplit];
  __shared__ float wred[8][NQ], wred2[8][NQ];
  __shared__ float mh[NQ], lh[NQ], ph_sum[NQ], cst[NQ];
  __shared__ int wexp[NQ];
  __shared__ int pexp;
  const int split = blockIdx.x, g = blockIdx.y, b = blockIdx.z;
  const int tid = threadIdx.x, lane = tid & 63, n = lane & 15, kg = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int len = (int)min((int64_t)max(a.seq_len[b], 0), a.cap);
  const int s0 = split * kGSplit;
  if (s0 >= len) return;                            // (whole workgroup, before any barrier)
  const GroupParams* pk = group_params(a.params_k, g);
  const GroupParams* pv = group_params(a.params_v, g);
  if (pk->max_bits > 12 || pv->max_bits > 12) {
    group_split_wide_body<NC, NQ>(a);
    return;
  }
  const int nt = min(len, s0 + kGSplit) - s0;
  float* pbase = a.part + ((((size_t)b * a.n_groups + g) * a.n_splits + split) * a.heads) * (D + kGPH);
  const int rwk = a.rwk, rwv = a.rwv;
  if (pk->record_bytes != 4 * rwk || pv->record_bytes != 4 * rwv || pk->d != D || pv->d != D) {
    if (tid < a.heads) pbase[(size_t)tid * (D + kGPH)] = NAN;
    return;
  }
  const int rs = max(rwk, rwv) + 1;                 // LDS row stride (one padding dword)
  const size_t rows_b = (size_t)kGSplit * rs * 4;
  gh8* wop = reinterpret_cast<gh8*>(smem);                                  // [NHT][NKB][2][64]
  _Float16* pl = reinterpret_cast<_Float16*>(smem);                         // [2][NQ][kGPRow]
  uint32_t* kdesc = reinterpret_cast<uint32_t*>(smem + kGWopBytes<NC, NHT>);   // [D]: off | b << 16
  uint32_t* vdesc = kdesc + D;
  uint32_t* rbk = vdesc + D;                                                // [kGSplit][rs]
  uint32_t* rbv = DUAL ? rbk + rows_b / 4 : rbk;
  const size_t gset = (size_t)b * a.n_groups + g;
  const size_t row0 = gset * a.heads;
  const size_t tok0 = gset * (size_t)a.cap + s0;
  const uint32_t* kw = reinterpret_cast<const uint32_t*>(a.k_codes + tok0 * pk->record_bytes);
  const uint32_t* vw = reinterpret_cast<const uint32_t*>(a.v_codes + tok0 * pv->record_bytes);
  // (1) Every load first: the weight operands, the records (the first pass of each, 16-byte
  //     loads where the records are aligned), the scales, descriptors and constants; then
  //     the stores.
  const int totk = nt * rwk, totv = nt * rwv;
  const bool vec = ((reinterpret_cast<uintptr_t>(kw) | reinterpret_cast<uintptr_t>(vw)) & 15u) == 0u &&
                   totk >= 4 && totv >= 4 && totk <= 4 * NT * kGStage4 && totv <= 4 * NT * kGStage4;
  uint4 vv[kGStage4];                               // (vec: the value records until stored)
  uint32_t tv = 0u;
  auto stage_all = [&]() {
    uint4 wv4[NHT][W4];
    auto load_w = [&]() {
#pragma unroll
      for (int ht = 0; ht < NHT; ++ht) {
        const uint4* wsrc = reinterpret_cast<const uint4*>(wop_tile(a, gset, D, ht));
#pragma unroll
        for (int i = 0; i < W4; ++i) wv4[ht][i] = wsrc[tid + NT * i];
      }
    };
    auto store_w = [&]() {
#pragma unroll
      for (int ht = 0; ht < NHT; ++ht)
#pragma unroll
        for (int i = 0; i < W4; ++i)
          reinterpret_cast<uint4*>(wop)[ht * NKB * 128 + tid + NT * i] = wv4[ht][i];
    };
    if (vec) {                                      // (uniform; no branch among the loads)
      uint4 vk[kGStage4];
      uint32_t tk;
      load_w();
      stage4_load<NT>(kw, totk, tid, vk, tk);
      stage4_load<NT>(vw, totv, tid, vv, tv);
      store_w();
      stage4_store<NT>(rbk, rs, totk, rwk, tid, vk, tk, true);
      if constexpr (DUAL) stage4_store<NT>(rbv, rs, totv, rwv, tid, vv, tv, true);
    } else {
      load_w();
      store_w();
      stage_records_any<NT>(rbk, rs, kw, nt, rwk);
      if constexpr (DUAL) stage_records_any<NT>(rbv, rs, vw, nt, rwv);
    }
  };
  {
    // (the small loads of step (1), issued before the records' and stored after them)
    constexpr int CPT = (D + NT - 1) / NT;
    uint32_t kbits[CPT], koff[CPT], vbits[CPT], voff[CPT];
#pragma unroll
    for (int i = 0; i < CPT; ++i) {
      const int c = min(tid + NT * i, D - 1);
      kbits[i] = pk->bits[c];
      koff[i] = pk->bit_off[c];
      vbits[i] = pv->bits[c];
      voff[i] = pv->bit_off[c];
    }
    const int ti = min(tid, nt - 1);
    const uint16_t ka16 = a.k_alpha[tok0 + ti], va16 = a.v_alpha[tok0 + ti];
    const int hi = min(tid & (NQ - 1), a.heads - 1);
    const float cst_v = a.cst[row0 + hi];
    const int wexp_v = wexp_tile(a, gset, D, hi >> 4)[hi & 15];
    stage_all();
#pragma unroll
    for (int i = 0; i < CPT; ++i) {
      const int c = tid + NT * i;
      // (a dropped channel: offset 0, width 0; its code is selected to 0)
      if (c < D) {
        kdesc[c] = kbits[i] ? koff[i] | (kbits[i] << 16) : 0u;
        vdesc[c] = vbits[i] ? voff[i] | (vbits[i] << 16) : 0u;
      }
    }
    if (tid < kGSplit) {
      rbk[tid * rs + rwk] = 0u;
      if constexpr (DUAL) rbv[tid * rs + rwv] = 0u;
      ak[tid] = tid < nt ? __half2float(__ushort_as_half(ka16)) : 0.f;
      av[tid] = tid < nt ? __half2float(__ushort_as_half(va16)) : 0.f;
    }
    if (tid < NQ) {
      cst[tid] = tid < a.heads ? cst_v : 0.f;
      wexp[tid] = tid < a.heads ? wexp_v : 0;
    }
  }
  __syncthreads();
  if (tid < kGSplit) {
    // the largest value scale of the split, for the exponent of P's scaling
    const float m = g_wave_max(av[tid]);
    if (lane == 0) wred2[wave][0] = m;
  }
  // (2) Scores of tokens 32 wave + 16 tb + n, heads 16 ht + 4 kg + i (slots past the group's heads
  //     hold other data: their operand rows are zeroed).
  // (the extract is made for every channel and a dropped one, width 0, selected to 0:
  // no branch around the LDS reads)
  auto code_of = [&](const uint32_t* row, uint32_t dsc) -> _Float16 {
    const int bw = (int)(dsc >> 16);
    const int code = record_code(row, (int)(dsc & 0xffffu), bw);
    return (_Float16)(float)(bw ? code : 0);
  };
  gf4 zs[NHT][2] = {};
  {
    const uint32_t* krow[2] = {rbk + (32 * wave + n) * rs, rbk + (32 * wave + 16 + n) * rs};
    const gh8 zero8 = {};
#pragma unroll 2
    for (int kb = 0; kb < NKB; ++kb) {
      gh8 whi[NHT], wlo[NHT];
#pragma unroll
      for (int ht = 0; ht < NHT; ++ht) {
        const bool head_ok = 16 * ht + n < a.heads;
        whi[ht] = head_ok ? wop[(ht * NKB + kb) * 128 + lane] : zero8;
        wlo[ht] = head_ok ? wop[(ht * NKB + kb) * 128 + 64 + lane] : zero8;
      }
      const int c0 = 32 * kb + 8 * kg;
      const uint4 d0 = *reinterpret_cast<const uint4*>(kdesc + c0);
      const uint4 d1 = *reinterpret_cast<const uint4*>(kdesc + c0 + 4);
      const uint32_t dk[8] = {d0.x, d0.y, d0.z, d0.w, d1.x, d1.y, d1.z, d1.w};
#pragma unroll
      for (int tb = 0; tb < 2; ++tb) {
        gh8 cb;
#pragma unroll
        for (int e = 0; e < 8; ++e) cb[e] = code_of(krow[tb], dk[e]);
#pragma unroll
        for (int ht = 0; ht < NHT; ++ht) {
          zs[ht][tb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(whi[ht], cb, zs[ht][tb], 0, 0, 0);
          zs[ht][tb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(wlo[ht], cb, zs[ht][tb], 0, 0, 0);
        }
      }
    }
  }
  float z[NHT][2][4];
#pragma unroll
  for (int hi = 0; hi < 4 * NHT; ++hi) {
    const int ht = hi >> 2, i = hi & 3, h = 16 * ht + 4 * kg + i;
    float m = -INFINITY;
#pragma unroll
    for (int tb = 0; tb < 2; ++tb) {
      const int t = 32 * wave + 16 * tb + n;
      z[ht][tb][i] = t < nt ? ak[t] * (ldexpf(zs[ht][tb][i], -wexp[h]) + cst[h]) : -INFINITY;
      m = fmaxf(m, z[ht][tb][i]);
    }
#pragma unroll
    for (int o = 8; o >= 1; o >>= 1) m = fmaxf(m, __shfl_xor(m, o, 64));
    if (n == 0) wred[wave][h] = m;
  }
  __syncthreads();                                  // (every key record read, maxima in)
  if (tid < NQ) {
    float m = wred[0][tid];
#pragma unroll
    for (int w = 1; w < 8; ++w) m = fmaxf(m, wred[w][tid]);
    mh[tid] = m;
  }
  if (tid == 0) {
    const float m = fmaxf(fmaxf(wred2[0][0], wred2[1][0]), fmaxf(wred2[2][0], wred2[3][0]));
    int e = 0;
    if (m > 0.f) (void)frexpf(m, &e);
    pexp = m > 0.f ? 14 - e : 0;                    // max alpha^V 2^pexp in [2^13, 2^14)
  }
  if constexpr (!DUAL) {
    if (vec) stage4_store<NT>(rbv, rs, totv, rwv, tid, vv, tv, true);
    else stage_records_any<NT>(rbv, rs, vw, nt, rwv);
    if (tid < kGSplit) rbv[tid * rs + rwv] = 0u;
  }
  __syncthreads();
  // (3) p = 2^(z - m), P = p alpha^V: the sums of p (the softmax denominator) and of P (the
  //     midrise half step), and P 2^pexp as fp16 parts in [head][token] rows.
  {
    const int pe = pexp;
#pragma unroll
    for (int hi = 0; hi < 4 * NHT; ++hi) {
      const int ht = hi >> 2, i = hi & 3, h = 16 * ht + 4 * kg + i;
      float ps = 0.f, qs = 0.f;
#pragma unroll
      for (int tb = 0; tb < 2; ++tb) {
        const int t = 32 * wave + 16 * tb + n;
        const float p = t < nt ? __builtin_amdgcn_exp2f(z[ht][tb][i] - mh[h]) : 0.f;
        const float pv_ = p * av[t];
        ps += p;
        qs += pv_;
        const float sp = ldexpf(pv_, pe);
        const _Float16 hh = (_Float16)sp;
        pl[h * kGPRow + t] = hh;
        pl[(NQ + h) * kGPRow + t] = (_Float16)(sp - (float)hh);
      }
#pragma unroll
      for (int o = 8; o >= 1; o >>= 1) {
        ps += __shfl_xor(ps, o, 64);
        qs += __shfl_xor(qs, o, 64);
      }
      if (n == 0) {
        wred[wave][h] = ps;
        wred2[wave][h] = qs;
      }
    }
  }
  __syncthreads();
  if (tid < NQ) {
    float ps = 0.f, qs = 0.f;
#pragma unroll
    for (int w = 0; w < 8; ++w) {
      ps += wred[w][tid];
      qs += wred2[w][tid];
    }
    lh[tid] = ps;
    ph_sum[tid] = qs;
  }
  __syncthreads();
  // (4) Values: wave w takes channel blocks w, w + 8, ...; lane 16 kg + n ends with heads
  //     16 ht + 4 kg + i of channel 16 cb + n.
  const bool mr_v = pv->quantizer == AATC_QUANT_MIDRISE;
  const int pe = pexp;
  for (int cb = wave; cb < NCB; cb += 8) {
    const int c = 16 * cb + n;
    const uint32_t dsc = vdesc[c];
    gf4 acc[NHT] = {};
#pragma unroll 2
    for (int tk = 0; tk < kGSplit / 32; ++tk) {
      const int t0 = 32 * tk + 8 * kg;
      gh8 cv;
#pragma unroll
      for (int e = 0; e < 8; ++e) cv[e] = code_of(rbv + (t0 + e) * rs, dsc);
#pragma unroll
      for (int ht = 0; ht < NHT; ++ht) {
        const gh8 phi = *reinterpret_cast<const gh8*>(pl + (16 * ht + n) * kGPRow + t0);
        const gh8 plo = *reinterpret_cast<const gh8*>(pl + (NQ + 16 * ht + n) * kGPRow + t0);
        acc[ht] = __builtin_amdgcn_mfma_f32_16x16x32_f16(phi, cv, acc[ht], 0, 0, 0);
        acc[ht] = __builtin_amdgcn_mfma_f32_16x16x32_f16(plo, cv, acc[ht], 0, 0, 0);
      }
    }
    const int bc = (int)(dsc >> 16);
    const float sc = bc > 0 ? ldexpf(pv->s[c], 1 - bc) : 0.f;
#pragma unroll
    for (int hi = 0; hi < 4 * NHT; ++hi) {
      const int h = 16 * (hi >> 2) + 4 * kg + (hi & 3);
      if (h < a.heads) {
        const float o = ldexpf(acc[hi >> 2][hi & 3], -pe) + (mr_v ? 0.5f * ph_sum[h] : 0.f);
        pbase[(size_t)h * (D + kGPH) + kGPH + c] = o * sc;
      }
    }
  }
  if (tid < a.heads) {
    pbase[(size_t)tid * (D + kGPH)] = mh[tid];
    pbase[(size_t)tid * (D + kGPH) + 1] = lh[tid];
  }
}

// The merge: one workgroup per (sequence, query head, 64 channels of o~), so that every compute
// unit reads a share of the split partials and of T_V.  Every chunk recomputes the splits'
// maximum M and weights 2^(m_s - M) (a few hundred floats); thread (range, channel) sums one
// quarter of the splits with eight loads in flight; o~ = sum_s w_s o~_s / sum_s w_s l_s (NaN if
// a split reported mismatched records, 0 for an empty sequence).  The chunk's share of the
// inverse transform, sum over its channels of T_V[128 kk + j][c] o~_c (its part of T_V loaded at
// the start), goes out with device-coherent stores, and the last chunk of a head to arrive
// adds the shares in order.  (Coherent accesses and a relaxed count need no cache write-back: a
// release before each arrival had made this 31 us.  Two launches, sums then transform, took
// 5.8 + 5.8 us, 6.0 + 9.6 for 112 heads.)
// A share's 128 outputs lie in the chunk's 64 floats of the head's rows of `ot` and of the
// weight region (read last by the split kernel, so no line of theirs is cached here); the
// arrival count in the header of the head's first partial row, cleared by the query kernel.
constexpr int kGMergeThreads = 256;
constexpr int kGMergeSplits = 1024;              // splits weighted per pass
template <int NC>
__global__ __launch_bounds__(kGMergeThreads) void group_merge_kernel(GroupDecodeArgs a) {
  constexpr int D = 64 * NC;
  constexpr int NT = kGMergeThreads;
  constexpr int NSUB = NT / 64;                    // split ranges per channel
  constexpr int NW = NT / 64;
  __shared__ float ot[NSUB][64];
  __shared__ __align__(16) float oc[64];
  __shared__ float wsp[kGMergeSplits];
  __shared__ float red[NW];
  __shared__ int last_s;
  const int h = blockIdx.x / NC, ci = blockIdx.x % NC, b = blockIdx.y;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int gq = a.n_q_heads / a.n_kv_heads;
  const int k = h / gq, g = k / a.gkv, kk = k % a.gkv, hl = h - g * a.heads;
  // Row j = tid / 2 of the head's block of T_V, half of the chunk's columns.
  float4 tv[8];
  {
    const float4* tr = reinterpret_cast<const float4*>(
        group_params(a.params_v, g)->T + (size_t)(kk * 128 + (tid >> 1)) * D + 64 * ci + 32 * (tid & 1));
#pragma unroll
    for (int q = 0; q < 8; ++q) tv[q] = tr[q];
  }
  float* out = a.out + ((int64_t)b * a.n_q_heads + h) * 128;
  const int len = (int)min((int64_t)max(a.seq_len[b], 0), a.cap);
  if (len == 0) {                                  // (uniform over the head's workgroups)
    if (ci == 0 && tid < 128) out[tid] = 0.f;
    return;
  }
  const int ns = (len + kGSplit - 1) / kGSplit;
  const size_t gset = (size_t)b * a.n_groups + g;
  float* pb = first_partial_row(a, gset, hl, D);
  const size_t sstride = (size_t)a.heads * (D + kGPH);
  float mx = -INFINITY;
  for (int s = tid; s < ns; s += NT) {
    const float ms = pb[s * sstride];
    mx = (mx != mx || ms != ms) ? NAN : fmaxf(mx, ms);   // (a NaN mark is kept)
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    const float y = __shfl_xor(mx, o, 64);
    mx = (mx != mx || y != y) ? NAN : fmaxf(mx, y);
  }
  if (lane == 0) red[wave] = mx;
  __syncthreads();
  float M = red[0];
  for (int w = 1; w < NW; ++w) M = (M != M || red[w] != red[w]) ? NAN : fmaxf(M, red[w]);
  if (M != M) {                                    // (uniform over the head's workgroups)
    if (ci == 0 && tid < 128) out[tid] = NAN;
    return;
  }
  const int c = tid & 63, sub = tid >> 6;
  float L = 0.f, acc = 0.f;
  for (int s0 = 0; s0 < ns; s0 += kGMergeSplits) {
    const int n = min(kGMergeSplits, ns - s0);
    __syncthreads();                                // (the previous pass's weights are read)
    float lsum = 0.f;
    for (int s = tid; s < n; s += NT) {
      const float* p = pb + (size_t)(s0 + s) * sstride;
      const float w = __builtin_amdgcn_exp2f(p[0] - M);
      wsp[s] = w;
      lsum = fmaf(w, p[1], lsum);
    }
    lsum = g_wave_sum(lsum);
    __syncthreads();
    if (lane == 0) red[wave] = lsum;
    __syncthreads();
    for (int w = 0; w < NW; ++w) L += red[w];
    const int lo = n * sub / NSUB, hi = n * (sub + 1) / NSUB;
    const float* p = pb + kGPH + 64 * ci + c + (size_t)s0 * sstride;
    float a0 = 0.f, a1 = 0.f;
    int s = lo;
    for (; s + 8 <= hi; s += 8) {
      float v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = p[(size_t)(s + u) * sstride];
#pragma unroll
      for (int u = 0; u < 8; u += 2) {
        a0 = fmaf(wsp[s + u], v[u], a0);
        a1 = fmaf(wsp[s + u + 1], v[u + 1], a1);
      }
    }
    for (; s < hi; ++s) a0 = fmaf(wsp[s], p[(size_t)s * sstride], a0);
    acc += a0 + a1;
  }
  ot[sub][c] = acc;
  __syncthreads();
  if (tid < 64) {
    float v = 0.f;
#pragma unroll
    for (int u = 0; u < NSUB; ++u) v += ot[u][tid];
    oc[tid] = v * (L > 0.f ? 1.f / L : 0.f);
  }
  __syncthreads();
  float o = 0.f;
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    const float4 x = *reinterpret_cast<const float4*>(&oc[32 * (tid & 1) + 4 * q]);
    o = fmaf(tv[q].x, x.x, o);
    o = fmaf(tv[q].y, x.y, o);
    o = fmaf(tv[q].z, x.z, o);
    o = fmaf(tv[q].w, x.w, o);
  }
  o += __shfl_xor(o, 1, 64);
  const size_t row = ((size_t)b * a.n_q_heads + h) * D;
  auto share = [&](int x, int j) { return (j < 64 ? a.otl : a.w) + row + 64 * x + (j & 63); };
  if ((tid & 1) == 0)
    __hip_atomic_store(share(ci, tid >> 1), o, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __builtin_amdgcn_s_waitcnt(0);                    // this thread's store has completed
  __syncthreads();
  if (tid == 0)
    last_s = __hip_atomic_fetch_add(merge_count(a, gset, hl, D), 1u, __ATOMIC_RELAXED,
                                    __HIP_MEMORY_SCOPE_AGENT) == (unsigned)(NC - 1);
  __syncthreads();
  if (!last_s || tid >= 128) return;
  float v[NC];
#pragma unroll
  for (int x = 0; x < NC; ++x)
    v[x] = __hip_atomic_load(share(x, tid), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  float r = v[0];
#pragma unroll
  for (int x = 1; x < NC; ++x) r += v[x];
  out[tid] = r;
}

// The dynamic LDS limit of one kernel on the current device, raised once per device when a
// launch first needs more (an idempotent attribute call; the recorded limit only grows).
struct GroupLds {
  std::atomic<size_t> set[64] = {};
  bool ensure(const void* kernel, size_t lds) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return false;
    if (dev < 0 || dev >= 64)
      return hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                                 (int)lds) == hipSuccess;
    size_t cur = set[dev].load(std::memory_order_acquire);
    if (lds <= cur) return true;
    if (hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) !=
        hipSuccess)
      return false;
    while (cur < lds && !set[dev].compare_exchange_weak(cur, lds, std::memory_order_acq_rel)) {
    }
    return true;
  }
};

// Whether the matrix-core split fits: its LDS, and that of the VALU body which a workgroup of the
// same launch takes for codes over 12 bits (the widths lie on the device), with 16 NHT head slots.
// At 512 channels the VALU body ends it at records of 99 dwords with one tile (6.19 bits per channel)
// and 51 with two (3.19); the operands alone would hold 113 and 81.  *lds gets the size, and the
// result is true when both record sets fit at once (DUAL).
template <int NC, int NHT>
bool group_mfma_fit(int rwk, int rwv, size_t* lds) {
  constexpr int D = 64 * NC, NQ = 16 * NHT;
  const int rwm = std::max(rwk, rwv);
  const size_t wide = sizeof(float) * (size_t)D * NQ + sizeof(uint32_t) * (size_t)kGSplit * (rwm + 1) +
                      sizeof(float) * (size_t)kGSplit * NQ + sizeof(uint32_t) * D;
  const size_t m2 = std::max(wide, group_mfma_lds<NC, NHT>(rwm, true));
  const size_t m1 = std::max(wide, group_mfma_lds<NC, NHT>(rwm, false));
  *lds = m2 <= kGMfmaLdsCap ? m2 : m1 <= kGMfmaLdsCap ? m1 : 0;
  return m2 <= kGMfmaLdsCap;
}

template <int NC, int NHT, bool DUAL>
aatc_status launch_split_mfma(const GroupDecodeArgs& a, dim3 grid, size_t lds, hipStream_t st) {
  static GroupLds limit;
  if (!limit.ensure((const void*)group_split_mfma_kernel<NC, NHT, DUAL>, lds)) return AATC_E_DEVICE;
  hipLaunchKernelGGL((group_split_mfma_kernel<NC, NHT, DUAL>), grid, dim3(kGWideThreads), lds, st, a);
  return hipGetLastError() == hipSuccess ? AATC_OK : AATC_E_DEVICE;
}

template <int NC, int NQ>
aatc_status launch_split(const GroupDecodeArgs& a, int batch, int rwk, int rwv,
                         hipStream_t st) {
  constexpr int D = 64 * NC;
  const size_t lds_wide = sizeof(float) * (size_t)D * NQ +
                          sizeof(uint32_t) * (size_t)kGSplit * (std::max(rwk, rwv) + 1) +
                          sizeof(float) * (size_t)kGSplit * NQ + sizeof(uint32_t) * D;
  const dim3 grid((unsigned)a.n_splits, (unsigned)a.n_groups, (unsigned)batch);
  if (a.wops) {
    constexpr int NHT = NQ <= 16 ? 1 : 2;
    size_t lds = 0;
    if (group_mfma_fit<NC, NHT>(rwk, rwv, &lds)) return launch_split_mfma<NC, NHT, true>(a, grid, lds, st);
    return launch_split_mfma<NC, NHT, false>(a, grid, lds, st);
  }
  if (lds_wide <= 144 * 1024) {
    static GroupLds limit_wide;
    if (!limit_wide.ensure((const void*)group_split_wide_kernel<NC, NQ>, lds_wide))
      return AATC_E_DEVICE;
    hipLaunchKernelGGL((group_split_wide_kernel<NC, NQ>), grid, dim3(kGWideThreads), lds_wide,
                       st, a);
    return hipGetLastError() == hipSuccess ? AATC_OK : AATC_E_DEVICE;
  }
  const size_t lds = sizeof(float) * (size_t)D * NQ +
                     sizeof(uint32_t) * (size_t)kGChunk * (rwk + 1 + rwv + 1) +
                     sizeof(float) * (size_t)kGChunk * NQ + sizeof(uint32_t) * D;
  if (lds > 150 * 1024) return AATC_E_UNSUPPORTED;
  static GroupLds limit;
  if (!limit.ensure((const void*)group_split_kernel<NC, NQ>, lds)) return AATC_E_DEVICE;
  hipLaunchKernelGGL((group_split_kernel<NC, NQ>),
                     dim3((unsigned)a.n_splits, (unsigned)a.n_groups, (unsigned)batch),
                     dim3(kGThreads), lds, st, a);
  return hipGetLastError() == hipSuccess ? AATC_OK : AATC_E_DEVICE;
}

template <int NC>
aatc_status launch_decode_nc(GroupDecodeArgs a, int batch, int rwk, int rwv, hipStream_t st) {
  size_t lds_m = 0;
  if (a.heads <= 16) (void)group_mfma_fit<NC, 1>(rwk, rwv, &lds_m);
  else (void)group_mfma_fit<NC, 2>(rwk, rwv, &lds_m);
  a.wops = lds_m > 0 ? 1 : 0;                       // the query kernel writes the operands
  hipLaunchKernelGGL((group_query_kernel<NC>), dim3((unsigned)a.n_q_heads, (unsigned)batch),
                     dim3(kGQThreads), 0, st, a);
  if (hipGetLastError() != hipSuccess) return AATC_E_DEVICE;
  aatc_status s;
  if (a.heads <= 4) s = launch_split<NC, 4>(a, batch, rwk, rwv, st);
  else if (a.heads <= 8) s = launch_split<NC, 8>(a, batch, rwk, rwv, st);
  else if (a.heads <= 16) s = launch_split<NC, 16>(a, batch, rwk, rwv, st);
  else s = launch_split<NC, 32>(a, batch, rwk, rwv, st);
  if (s != AATC_OK) return s;
  hipLaunchKernelGGL((group_merge_kernel<NC>), dim3((unsigned)(a.n_q_heads * NC), (unsigned)batch),
                     dim3(kGMergeThreads), 0, st, a);
  return hipGetLastError() == hipSuccess ? AATC_OK : AATC_E_DEVICE;
}

template <int NC, bool BF16, int TT>
aatc_status launch_group_encode_tt(const void* params, int n_groups, const void* x, int64_t n_tok,
                                   int64_t x_tok_stride, int vec, uint8_t* codes, uint16_t* alpha,
                                   int64_t cap, int64_t pos, hipStream_t st) {
  constexpr int D = 64 * NC;
  // X limbs, or the record rows (codes of at most 8 bits: R <= D bytes).
  constexpr size_t lds = std::max((size_t)(BF16 ? 3 : 4) * D * 16 * TT, (size_t)16 * TT * (D / 4 + 1) * 4);
  static GroupLds limit;
  if (!limit.ensure((const void*)group_encode_mfma_kernel<NC, BF16, TT>, lds)) return AATC_E_DEVICE;
  const int64_t blocks = (n_tok + 16 * TT - 1) / (16 * TT);
  if (blocks > 0x7fffffff) return AATC_E_UNSUPPORTED;
  hipLaunchKernelGGL((group_encode_mfma_kernel<NC, BF16, TT>),
                     dim3((unsigned)blocks, (unsigned)n_groups), dim3(64 * kGEncWaves), lds, st,
                     params, x, n_tok, x_tok_stride, vec, codes, alpha, cap, pos);
  return hipGetLastError() == hipSuccess ? AATC_OK : AATC_E_DEVICE;
}

template <int NC>
aatc_status launch_group_encode_nc(const void* params, int n_groups, const void* x,
                                   aatc_dtype x_dtype, int64_t n_tok, int64_t x_tok_stride,
                                   uint8_t* codes, uint16_t* alpha, int64_t cap, int64_t pos,
                                   hipStream_t st) {
  const int vec = (reinterpret_cast<uintptr_t>(x) % 16 == 0 &&
                   (size_t)x_tok_stride * (x_dtype == AATC_BF16 ? 2 : 4) % 16 == 0) ? 1 : 0;
  // Tokens per workgroup: as many as leave the chip a workgroup per compute unit (each reads
  // the whole transform), fp32 at most 32 (registers).
  auto fills = [&](int tt) { return (n_tok / (16 * tt)) * n_groups >= 192; };
  aatc_status s;
  if (x_dtype == AATC_BF16) {
    if (fills(4)) s = launch_group_encode_tt<NC, true, 4>(params, n_groups, x, n_tok, x_tok_stride, vec, codes, alpha, cap, pos, st);
    else if (fills(2)) s = launch_group_encode_tt<NC, true, 2>(params, n_groups, x, n_tok, x_tok_stride, vec, codes, alpha, cap, pos, st);
    else s = launch_group_encode_tt<NC, true, 1>(params, n_groups, x, n_tok, x_tok_stride, vec, codes, alpha, cap, pos, st);
  } else {
    if (fills(2)) s = launch_group_encode_tt<NC, false, 2>(params, n_groups, x, n_tok, x_tok_stride, vec, codes, alpha, cap, pos, st);
    else s = launch_group_encode_tt<NC, false, 1>(params, n_groups, x, n_tok, x_tok_stride, vec, codes, alpha, cap, pos, st);
  }
  if (s != AATC_OK) return s;
  // The tokens whose certificate failed (stream order: after the kernel above).  Each costs its
  // workgroup about 20 us at d = 512, so they are spread over four workgroups per compute unit
  // (8192 tokens, two groups, K and V: 162 us with 16 marks each, 169 with 64, 170 with 4); past
  // that the scans of unmarked shares would add up.
  const int share = (n_tok / 16) * n_groups <= 1024 ? 16 : kGFixTokens;
  hipLaunchKernelGGL((group_encode_exact_kernel<NC>),
                     dim3((unsigned)((n_tok + share - 1) / share), (unsigned)n_groups),
                     dim3(kGFixThreads), 0, st, params, x, (int)x_dtype, n_tok, x_tok_stride, codes,
                     alpha, cap, pos, share);
  return hipGetLastError() == hipSuccess ? AATC_OK : AATC_E_DEVICE;
}

}  // namespace

aatc_status launch_group_encode(const void* params, int n_groups, int gkv, const void* x,
                                aatc_dtype x_dtype, int64_t n_tok, int64_t x_tok_stride,
                                void* codes, uint16_t* alpha, int64_t cap, int64_t pos,
                                void* stream) {
  if (n_tok == 0) return AATC_OK;
  const hipStream_t st = static_cast<hipStream_t>(stream);
  auto* c8 = static_cast<uint8_t*>(codes);
  switch (gkv) {
    case 1: return launch_group_encode_nc<2>(params, n_groups, x, x_dtype, n_tok, x_tok_stride, c8, alpha, cap, pos, st);
    case 2: return launch_group_encode_nc<4>(params, n_groups, x, x_dtype, n_tok, x_tok_stride, c8, alpha, cap, pos, st);
    case 3: return launch_group_encode_nc<6>(params, n_groups, x, x_dtype, n_tok, x_tok_stride, c8, alpha, cap, pos, st);
    case 4: return launch_group_encode_nc<8>(params, n_groups, x, x_dtype, n_tok, x_tok_stride, c8, alpha, cap, pos, st);
  }
  return AATC_E_UNSUPPORTED;
}

size_t group_decode_workspace_bytes(int batch, int n_q_heads, int n_kv_heads, int gkv,
                                    int64_t cap) {
  const int n_groups = n_kv_heads / gkv;
  const int heads = n_q_heads / n_groups;
  return group_ws_layout(batch, n_groups, heads, 128 * gkv, cap).total;
}

aatc_status launch_group_decode(const void* params_k, const void* params_v, int batch,
                                int n_q_heads, int n_kv_heads, int gkv, const void* q,
                                aatc_dtype q_dtype, const void* k_codes,
                                const uint16_t* k_alpha, const void* v_codes,
                                const uint16_t* v_alpha, const int32_t* seq_len, int64_t cap,
                                int k_record_bytes, int v_record_bytes, float softmax_scale,
                                float* out, void* workspace, void* stream) {
  const hipStream_t st = static_cast<hipStream_t>(stream);
  GroupDecodeArgs a{};
  a.params_k = params_k;
  a.params_v = params_v;
  a.q = q;
  a.q_dtype = (int)q_dtype;
  a.k_codes = static_cast<const uint8_t*>(k_codes);
  a.k_alpha = k_alpha;
  a.v_codes = static_cast<const uint8_t*>(v_codes);
  a.v_alpha = v_alpha;
  a.seq_len = seq_len;
  a.cap = cap;
  a.n_q_heads = n_q_heads;
  a.n_kv_heads = n_kv_heads;
  a.gkv = gkv;
  a.n_groups = n_kv_heads / gkv;
  a.heads = n_q_heads / a.n_groups;
  a.scale_log2e = softmax_scale * 1.4426950408889634f;
  const GroupWs l = group_ws_layout(batch, a.n_groups, a.heads, 128 * gkv, cap);
  a.n_splits = l.n_splits;
  if ((int64_t)l.n_splits > 0xffff || batch > 0xffff) return AATC_E_UNSUPPORTED;
  char* ws = static_cast<char*>(workspace);
  a.w = reinterpret_cast<float*>(ws + l.w);
  a.cst = reinterpret_cast<float*>(ws + l.c);
  a.part = reinterpret_cast<float*>(ws + l.partials);
  a.wop = reinterpret_cast<uint16_t*>(ws + l.wop);
  a.wexp = reinterpret_cast<int32_t*>(ws + l.wexp);
  a.otl = reinterpret_cast<float*>(ws + l.ot);
  a.out = out;
  const int rwk = k_record_bytes / 4, rwv = v_record_bytes / 4;
  a.rwk = rwk;
  a.rwv = rwv;
  switch (gkv) {
    case 1: return launch_decode_nc<2>(a, batch, rwk, rwv, st);
    case 2: return launch_decode_nc<4>(a, batch, rwk, rwv, st);
    case 3: return launch_decode_nc<6>(a, batch, rwk, rwv, st);
    case 4: return launch_decode_nc<8>(a, batch, rwk, rwv, st);
  }
  return AATC_E_UNSUPPORTED;
}

}  // namespace aatc
