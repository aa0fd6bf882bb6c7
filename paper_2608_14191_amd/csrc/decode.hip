// AATC decode attention on gfx950 (Algorithm 1, inference part, evaluated in the
// transformed domain of App. B: q~ = T_K^T q; the inverse transform T_V is applied once
// to each output).
//
// Each workgroup scores a share of one (sequence, KV head)'s tokens for the query heads of
// that KV head, runs a softmax over the share and accumulates the value codes into a partial
// (m, l, o~) in the workspace.  The last workgroup of each (sequence, KV head) to finish
// merges the partials and applies T_V.
//
// Two kernels share that structure:
//  * decode_mfma_kernel: records of at most 128 bytes (budgets <= 1024 bits), any G <= 16;
//    both contractions run on int8 MFMA over the bits of the packed codes; a workgroup's
//    share is a run of 512- or 1024-token chunks;
//  * decode_split_kernel: wider records; plain VALU over 512-token splits.
//
// Codes are b-bit two's complement patterns, code = sum_{k < b-1} 2^k bit_k -
// 2^(b-1) bit_(b-1): every record bit is a virtual channel whose weight is its
// channel's weight times +-2^k, and sums over bits need no offset term.
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>

#include "decode_plan.h"
#include "encode_core.h"
#include "launch.h"
#include "params.h"
#include "workspace.h"

namespace aatc {
namespace {

constexpr int kThreads = 256;                    // generic kernel: four waves
constexpr int kSplit = 512;                      // tokens per workgroup, generic kernel
constexpr float kLog2e = 1.4426950408889634f;
constexpr int kRsrcWord3 = 0x00020000;           // raw buffer descriptor word 3 (gfx950)
constexpr int kCoherent = 16;                    // cache policy sc1: device-coherent access
constexpr int kMergeU = 8;                       // split partials in flight per merging thread

typedef int v4i __attribute__((ext_vector_type(4)));
typedef const __attribute__((address_space(1))) uint32_t* gdword;   // global-memory dword
typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v2f __attribute__((ext_vector_type(2)));

struct DecodeArgs {
  const void* params_k;
  const void* params_v;
  const void* q;
  uint8_t* k_codes;               // written only by the fused append
  uint16_t* k_alpha;
  uint8_t* v_codes;
  uint16_t* v_alpha;
  const int32_t* seq_len;
  const void* x_k;                // fused append: new token [batch][n_kv_heads][d], or null
  const void* x_v;
  int x_dtype;
  float* out;
  unsigned* counters;
  Partial* partials;
  float* append_r;                // fused append: [rows][kAppStride] coefficients, bounds
  const Partial* seg;             // full-precision segment partials [rows][G], or null
  int64_t cap;
  int batch, n_q_heads, n_kv_heads, G, q_dtype;
  int hg;                         // groups of query heads per KV head, a workgroup row each
  int max_splits;                 // partial slots per row
  int rk, rv;                     // record bytes
  float scale_log2e;
  int off_v, off_ak, off_av, off_ql, off_qc, off_pb, off_ob, ob_stride, off_es;   // dynamic LDS
};

__device__ inline float load_q(const void* q, int dtype, int64_t idx) {
  if (dtype == AATC_BF16) {
    uint32_t b = static_cast<const uint16_t*>(q)[idx];
    return __uint_as_float(b << 16);
  }
  return static_cast<const float*>(q)[idx];
}

__device__ inline float half_bits_to_float(uint16_t h) {
  return __half2float(__ushort_as_half(h));
}

// Buffer descriptors: loads past `bytes` return 0, stores past it are dropped.
__device__ inline __amdgpu_buffer_rsrc_t make_rsrc(const void* base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, (int)bytes,
                                           kRsrcWord3);
}
__device__ inline v2f buf_load8_coherent(__amdgpu_buffer_rsrc_t r, uint32_t off) {
  return (v2f)__builtin_amdgcn_raw_buffer_load_b64(r, (int)off, 0, kCoherent);
}
__device__ inline v4f buf_load16_coherent(__amdgpu_buffer_rsrc_t r, uint32_t off) {
  return (v4f)__builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, kCoherent);
}
__device__ inline void buf_store16_coherent(v4f v, __amdgpu_buffer_rsrc_t r, uint32_t off) {
  __builtin_amdgcn_raw_buffer_store_b128((v4i)v, r, (int)off, 0, kCoherent);
}
__device__ inline void buf_store4_coherent(float v, __amdgpu_buffer_rsrc_t r, uint32_t off) {
  __builtin_amdgcn_raw_buffer_store_b32(__float_as_int(v), r, (int)off, 0, kCoherent);
}

// Device-coherent scalar store: a relaxed agent-scope atomic is performed where every
// compute unit of the device sees it (it bypasses the per-XCD caches).
__device__ inline void st_dev(float* p, float v) {
  __hip_atomic_store(reinterpret_cast<unsigned*>(p), __float_as_uint(v), __ATOMIC_RELAXED,
                     __HIP_MEMORY_SCOPE_AGENT);
}

// Wave-wide maximum and sum without LDS round trips: quad butterflies and row rotations
// (DPP), then the four row results read as scalars.
template <int CTRL>
__device__ inline float dpp_f(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, false));
}
// Lane l and lane l ^ 16 (l ^ 32) combined without LDS: the row swaps of gfx950 return
// both halves of the exchange, so op(r[0], r[1]) is op(v, partner) in every lane.
__device__ inline float xor16_max(float v) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ inline float xor32_max(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ inline float xor16_sum(float v) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ inline float xor32_sum(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ inline int xor16_sum(int v) {
  const auto r = __builtin_amdgcn_permlane16_swap((unsigned)v, (unsigned)v, false, false);
  return (int)r[0] + (int)r[1];
}
__device__ inline int xor32_sum(int v) {
  const auto r = __builtin_amdgcn_permlane32_swap((unsigned)v, (unsigned)v, false, false);
  return (int)r[0] + (int)r[1];
}

// Wave-wide maximum and sum without LDS round trips: quad butterflies and row rotations
// (DPP), then the row swaps; every lane ends with the result.
__device__ inline float wave_max_dpp(float v) {
  v = fmaxf(v, dpp_f<0xB1>(v));            // quad_perm [1,0,3,2]
  v = fmaxf(v, dpp_f<0x4E>(v));            // quad_perm [2,3,0,1]
  v = fmaxf(v, dpp_f<0x124>(v));           // row_ror:4
  v = fmaxf(v, dpp_f<0x128>(v));           // row_ror:8
  return xor32_max(xor16_max(v));
}
__device__ inline float wave_sum_dpp(float v) {
  v += dpp_f<0xB1>(v);
  v += dpp_f<0x4E>(v);
  v += dpp_f<0x124>(v);
  v += dpp_f<0x128>(v);
  return xor32_sum(xor16_sum(v));
}
// Maximum and sum over each row of 16 lanes (every lane of the row ends with it).
__device__ inline float row16_max(float v) {
  v = fmaxf(v, dpp_f<0xB1>(v));
  v = fmaxf(v, dpp_f<0x4E>(v));
  v = fmaxf(v, dpp_f<0x124>(v));
  return fmaxf(v, dpp_f<0x128>(v));
}
__device__ inline float row16_sum(float v) {
  v += dpp_f<0xB1>(v);
  v += dpp_f<0x4E>(v);
  v += dpp_f<0x124>(v);
  return v + dpp_f<0x128>(v);
}
template <int CTRL>
__device__ inline int dpp_i(int v) {
  return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xF, 0xF, false);
}
__device__ inline int wave_sum_i32(int v) {         // exact while the sum fits 32 bits
  v += dpp_i<0xB1>(v);
  v += dpp_i<0x4E>(v);
  v += dpp_i<0x124>(v);
  v += dpp_i<0x128>(v);
  return xor32_sum(xor16_sum(v));
}
// One step of a reduce-scatter across lanes l and l ^ BIT (BIT = 8, 16 or 32): the lane
// with that bit clear keeps the sums of the lower half of the C values, the other the
// upper half.  (The row swaps return the pair ordered by lane: lower lane's value first.)
template <int C, int BIT>
__device__ inline void reduce_scatter_step(const float (&in)[C], float (&out)[C / 2]) {
  const bool up = (threadIdx.x & BIT) != 0;
#pragma unroll
  for (int i = 0; i < C / 2; ++i) {
    const float k = up ? in[C / 2 + i] : in[i];
    const float s = up ? in[i] : in[C / 2 + i];
    float p;
    if constexpr (BIT == 32) {
      const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(s), __float_as_uint(s), false, false);
      p = __uint_as_float(up ? r[0] : r[1]);
    } else if constexpr (BIT == 16) {
      const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(s), __float_as_uint(s), false, false);
      p = __uint_as_float(up ? r[0] : r[1]);
    } else {
      static_assert(BIT == 8, "bits 3, 4, 5");
      p = dpp_f<0x128>(s);                     // row_ror:8 within rows of 16: lane l ^ 8
    }
    out[i] = k + p;
  }
}

// N independent reductions taken step by step together, so that each step's exchanges
// overlap (a single chain waits on every step).
template <int N>
__device__ inline void wave_max_n(float (&v)[N]) {
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] = fmaxf(v[i], dpp_f<0xB1>(v[i]));
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] = fmaxf(v[i], dpp_f<0x4E>(v[i]));
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] = fmaxf(v[i], dpp_f<0x124>(v[i]));
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] = fmaxf(v[i], dpp_f<0x128>(v[i]));
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] = xor16_max(v[i]);
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] = xor32_max(v[i]);
}
template <int N>
__device__ inline void wave_sum_n(float (&v)[N]) {
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] += dpp_f<0xB1>(v[i]);
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] += dpp_f<0x4E>(v[i]);
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] += dpp_f<0x124>(v[i]);
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] += dpp_f<0x128>(v[i]);
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] = xor16_sum(v[i]);
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] = xor32_sum(v[i]);
}
template <int N>
__device__ inline void wave_sum_i32_n(int (&v)[N]) {
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] += dpp_i<0xB1>(v[i]);
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] += dpp_i<0x4E>(v[i]);
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] += dpp_i<0x124>(v[i]);
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] += dpp_i<0x128>(v[i]);
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] = xor16_sum(v[i]);
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] = xor32_sum(v[i]);
}

__device__ inline float block_reduce(float v, bool is_max, float* scratch) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    float w = __shfl_xor(v, o, 64);
    v = is_max ? fmaxf(v, w) : v + w;
  }
  const int wave = threadIdx.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) scratch[wave] = v;
  __syncthreads();
  float r = scratch[0];
  for (int i = 1; i < kThreads / 64; ++i) r = is_max ? fmaxf(r, scratch[i]) : r + scratch[i];
  return r;
}

// Lane-quad data movement (lanes 4k .. 4k + 3): xor 1 and xor 2 within the quad.
__device__ inline uint32_t quad_xor1(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, false);
}
__device__ inline uint32_t quad_xor2(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, false);
}
__device__ inline float quad_xor1(float v) { return __uint_as_float(quad_xor1(__float_as_uint(v))); }
__device__ inline float quad_xor2(float v) { return __uint_as_float(quad_xor2(__float_as_uint(v))); }

// Four balanced int8 limbs of a 32-bit value |x| < 2^30, packed in one dword (limb L in
// byte L, two's complement): x = sum_L limb_L 256^L.
__device__ inline uint32_t pack_limbs(int x) {
  return ((uint32_t)x + 0x80808080u) ^ 0x80808080u;
}

// s_waitcnt immediates (gfx9 layout: vmcnt [3:0] and [15:14], expcnt [6:4], lgkmcnt [11:8]).
constexpr int kWaitVm0 = (0x7 << 4) | (0xF << 8);            // vmcnt(0) only
constexpr int kWaitLgkm0 = 0xF | (0x7 << 4) | (0x3 << 14);    // lgkmcnt(0) only

// s_barrier alone, with no wait on outstanding memory operations (unlike __syncthreads(),
// whose fence waits for every load of the wave, LDS transfers included).  The memory
// clobber keeps the compiler's memory accesses on their side; the scheduling barriers
// keep other instructions (and the waits they would bring) there too.
__device__ inline void plain_barrier() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_barrier" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

// s_waitcnt vmcnt(n) for a wave-uniform n known only at run time (0 <= n < 64).
__device__ inline void wait_vmcnt(int n) {
#define AATC_VMW(k)                                                                         \
  case k:                                                                                  \
    __builtin_amdgcn_s_waitcnt(((k) & 0xF) | (0x7 << 4) | (0xF << 8) | (((k) >> 4) << 14)); \
    break;
#define AATC_VMW4(k) AATC_VMW(k) AATC_VMW(k + 1) AATC_VMW(k + 2) AATC_VMW(k + 3)
  switch (__builtin_amdgcn_readfirstlane(n)) {
    AATC_VMW4(0) AATC_VMW4(4) AATC_VMW4(8) AATC_VMW4(12) AATC_VMW4(16) AATC_VMW4(20)
    AATC_VMW4(24) AATC_VMW4(28) AATC_VMW4(32) AATC_VMW4(36) AATC_VMW4(40) AATC_VMW4(44)
    AATC_VMW4(48) AATC_VMW4(52) AATC_VMW4(56) AATC_VMW4(60)
    default: __builtin_amdgcn_s_waitcnt(0); break;
  }
#undef AATC_VMW4
#undef AATC_VMW
}

// The same for small n (a larger one waits for all but the last 15).
__device__ inline void wait_vmcnt_small(int n) {
#define AATC_VMW(k)                                                                         \
  case k:                                                                                  \
    __builtin_amdgcn_s_waitcnt(((k) & 0xF) | (0x7 << 4) | (0xF << 8));                       \
    break;
  switch (__builtin_amdgcn_readfirstlane(n)) {
    AATC_VMW(0) AATC_VMW(1) AATC_VMW(2) AATC_VMW(3) AATC_VMW(4) AATC_VMW(5) AATC_VMW(6)
    AATC_VMW(7) AATC_VMW(8) AATC_VMW(9) AATC_VMW(10) AATC_VMW(11) AATC_VMW(12) AATC_VMW(13)
    AATC_VMW(14)
    default: __builtin_amdgcn_s_waitcnt(0xF | (0x7 << 4) | (0xF << 8)); break;
  }
#undef AATC_VMW
}

__device__ inline v4i mfma_i8(v4i a, v4i b, v4i c) {
  return __builtin_amdgcn_mfma_i32_16x16x64_i8(a, b, c, 0, 0, 0);
}

// Bytes of LDS the merge of an NTHR-thread workgroup needs (at the start of the dynamic
// LDS).
constexpr size_t merge_lds_bytes(int G, int NTHR) {
  return (size_t)(6 * NTHR + G * kD + (NTHR / 32) * G * kD) * sizeof(float);
}

// Inverse transform o = T_V o~ of G vectors with NTHR threads: thread (j4, cb) holds T_V
// rows 4 j4 .. 4 j4 + 3 at columns CW cb .. CW cb + CW - 1 (CW = 4096 / NTHR).
template <int NTHR>
struct TvBlock {
  static constexpr int NCB = NTHR / 32, CW = kD / NCB;
  v4f t[4][CW / 4];
  __device__ void load(const HeadParams* hv) {
    const int j4 = threadIdx.x & 31, cb = threadIdx.x >> 5;
#pragma unroll
    for (int jj = 0; jj < 4; ++jj)
#pragma unroll
      for (int k = 0; k < CW / 4; ++k)
        t[jj][k] = reinterpret_cast<const v4f*>(hv->T)[(4 * j4 + jj) * (kD / 4) + (CW / 4) * cb + k];
  }
  // osum: LDS [G][kD] input; ored: LDS [NCB][G][kD] scratch.  Calls sink(h, j, o_hj) once
  // per output, after a barrier; the caller synchronizes before osum is reused.
  template <class Sink>
  __device__ void apply(const float* osum, float* ored, int G, Sink sink) const {
    const int tid = threadIdx.x, j4 = tid & 31, cb = tid >> 5;
    for (int h = 0; h < G; ++h) {
      const v4f* oh = reinterpret_cast<const v4f*>(osum + h * kD) + (CW / 4) * cb;
      v4f ov4[CW / 4];
#pragma unroll
      for (int k = 0; k < CW / 4; ++k) ov4[k] = oh[k];
#pragma unroll
      for (int jj = 0; jj < 4; ++jj) {
        v4f p = t[jj][0] * ov4[0];
#pragma unroll
        for (int k = 1; k < CW / 4; ++k) p += t[jj][k] * ov4[k];
        ored[(cb * G + h) * kD + 4 * j4 + jj] = p.x + p.y + p.z + p.w;
      }
    }
    __syncthreads();
    for (int i = tid; i < G * kD; i += NTHR) {
      const int h = i / kD, j = i % kD;
      float acc = 0.f;
#pragma unroll
      for (int b = 0; b < NCB; ++b) acc += ored[(b * G + h) * kD + j];
      sink(h, j, acc);
    }
  }
};

// o = T_V o~ on the matrix cores (v_mfma_f32_16x16x32_bf16, fp32 sums), T and o~ as sums of bf16
// terms, each the remainder of those before: pairs (three products, 2^-16 relative), T's from
// the parameter block's operand-ordered copy; or triples (exact, the six products T_a o_b with
// a + b <= 2, the rest below 2^-24), T split here, for the shapes that had fp32 sums before
// (6 bits, 6001 tokens: 5.6e-6 of the output in pairs against 4.6e-6; triples cost 0.8 us, their
// row-wise loads and the split).  Wave w < 8 computes output rows 16 w .. + 15 for up to 16
// vectors: A = its 16-row block of T, lane 16 g + n row n at columns 32 kk + 8 g .. + 7, B
// column n = vector n.
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

struct TvMfma {
  bf16x8 a[4][3];                         // [k-step][term]
  v4f t[4][2];                            // triples: the lane's columns of T until split()
  __device__ void load(const HeadParams* hv, bool triple) {
    const int lane = threadIdx.x & 63, wave = (threadIdx.x >> 6) & 7;
    if (triple) {
      const v4f* tp = reinterpret_cast<const v4f*>(hv->T + (16 * wave + (lane & 15)) * kD + 8 * (lane >> 4));
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
        t[kk][0] = tp[8 * kk];
        t[kk][1] = tp[8 * kk + 1];
      }
    } else {
      const bf16x8* tp = reinterpret_cast<const bf16x8*>(hv->Tm);
#pragma unroll
      for (int kk = 0; kk < 4; ++kk)
#pragma unroll
        for (int u = 0; u < 2; ++u) a[kk][u] = tp[((wave * 4 + kk) * 2 + u) * 64 + lane];
    }
  }
  __device__ void split() {
#pragma unroll
    for (int kk = 0; kk < 4; ++kk)
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        float x = t[kk][e >> 2][e & 3];
#pragma unroll
        for (int u = 0; u < 3; ++u) {
          a[kk][u][e] = (__bf16)x;
          x -= (float)a[kk][u][e];
        }
      }
  }
  static constexpr int kOperand = 4 * 64 * 8;   // elements of one term's B operands in LDS
  // B operands in LDS: term t at ob + t kOperand holds [k-step][lane] 16-byte units, lane
  // 16 g + n: vector n at elements 32 kk + 8 g .. + 7 (put() writes one element).
  __device__ static void put(__bf16* ob, int n, int c, float x, bool triple) {
    const int i = ((c >> 5) * 64 + 16 * ((c >> 3) & 3) + n) * 8 + (c & 7);
    const __bf16 b0 = (__bf16)x;
    x -= (float)b0;
    const __bf16 b1 = (__bf16)x;
    ob[i] = b0;
    ob[kOperand + i] = b1;
    if (triple) ob[2 * kOperand + i] = (__bf16)(x - (float)b1);
  }
  // Calls sink(n, j0, o[j0 .. j0 + 3] of vector n) for n < G (triples: after split(); the
  // caller synchronizes after the puts); waves 0 .. 7.
  template <class Sink>
  __device__ void apply(const __bf16* ob, int G, bool triple, Sink sink) const {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, n = lane & 15;
    const bf16x8* b8 = reinterpret_cast<const bf16x8*>(ob);
    v4f acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = acc0, acc2 = acc0;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      const bf16x8 b0 = b8[kk * 64 + lane], b1 = b8[(4 + kk) * 64 + lane];
      acc0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[kk][0], b0, acc0, 0, 0, 0);
      acc1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[kk][0], b1, acc1, 0, 0, 0);
      acc2 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[kk][1], b0, acc2, 0, 0, 0);
    }
    if (triple) {
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
        const bf16x8 b0 = b8[kk * 64 + lane], b1 = b8[(4 + kk) * 64 + lane], b2 = b8[(8 + kk) * 64 + lane];
        acc1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[kk][0], b2, acc1, 0, 0, 0);
        acc2 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[kk][1], b1, acc2, 0, 0, 0);
        acc1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[kk][2], b0, acc1, 0, 0, 0);
      }
    }
    if (n < G) sink(n, 16 * wave + 4 * (lane >> 4), acc0 + acc1 + acc2);
  }
};

// Extra work of the merging workgroup (the segment and the fused append supply one, below).
struct NoHook {
  __device__ void prefetch() {}
  __device__ void encode() {}
  __device__ void fold(int, int, float&, float&, v4f&) const {}
  __device__ void fold1(int, int, float&, float&, float&) const {}
  __device__ float add1(int, int, float o) const { return o; }
  __device__ v4f add4(int, int, v4f o) const { return o; }
  __device__ void finish() {}
};

// Called by every workgroup of the generic kernel after it stored its partial with
// device-coherent stores.  The last of a (sequence, KV head) to arrive merges the split partials;
// the hook's fold() adds one more (score, value) term per output slot, add1() one more term after
// the inverse transform.
template <int NTHR, class Hook>
__device__ __forceinline__ void merge_if_last(const void* params_v, int kvh, int64_t row, int G,
                                              int n_splits, const Partial* partials,
                                              unsigned* counters, float* out_rows, float* lds,
                                              Hook& hook) {
  __shared__ unsigned last_s;
  const int tid = threadIdx.x;
  __builtin_amdgcn_s_waitcnt(0);          // this thread's partial stores have completed
  __syncthreads();
  // The arrival count goes out first; every workgroup then fetches T_V, which the merge
  // would need, under the count's round trip.
  unsigned prev = 0u;
  if (tid == 0)
    prev = __hip_atomic_fetch_add(&counters[row * kCtrStride], 1u, __ATOMIC_RELAXED,
                                  __HIP_MEMORY_SCOPE_AGENT);
  const HeadParams* hv = head_params(params_v, kvh);
  TvBlock<NTHR> tv;
  tv.load(hv);
  if (tid == 0) last_s = (prev == (unsigned)n_splits - 1u) ? 1u : 0u;
  __syncthreads();
  if (!last_s) return;
  float* cm = lds;                                         // [NTHR] group maxima
  float* cl = cm + NTHR;                                   // [NTHR] group sums
  v4f* cacc = reinterpret_cast<v4f*>(cl + NTHR);           // [NTHR]
  float* osum = reinterpret_cast<float*>(cacc + NTHR);     // [G][kD]
  float* ored = osum + G * kD;                             // [NTHR / 32][G][kD]
  const __amdgpu_buffer_rsrc_t prs =
      make_rsrc(partials + row * n_splits * G, (uint32_t)(n_splits * G * sizeof(Partial)));

  // (a) Online merge over the splits: slot (head, float4 column) per thread; groups of
  //     threads take interleaved splits and combine at the end.
  const int slots = G * (kD / 4);
  for (int base = 0; base < slots; base += NTHR) {
    const int width = min(slots - base, NTHR);
    const int ngroups = NTHR / width;
    const int slot = base + tid % width, grp = tid / width;
    const int h = slot >> 5, c4 = slot & 31;
    const bool active = grp < ngroups;
    float M = -INFINITY, Ls = 0.f;
    v4f acc = {0.f, 0.f, 0.f, 0.f};
    bool bad = false;
    v2f hd[kMergeU];
    v4f ov[kMergeU];
    auto issue = [&](int s0) {                     // past the last split the loads read 0
#pragma unroll
      for (int u = 0; u < kMergeU; ++u) {
        const uint32_t off = (uint32_t)(((s0 + u * ngroups) * G + h) * sizeof(Partial));
        hd[u] = buf_load8_coherent(prs, off);
        ov[u] = (v4f)__builtin_amdgcn_raw_buffer_load_b128(prs, (int)(off + 16 + 16 * c4), 0,
                                                          kCoherent);
      }
    };
    // Branch-free, so that every load of a batch is issued before the first wait (an
    // empty split has o~ = 0, and loads past the last split read 0).
    auto consume = [&](int s0) {
#pragma unroll
      for (int u = 0; u < kMergeU; ++u) {
        const float ms = (active && s0 + u * ngroups < n_splits) ? hd[u].x : -INFINITY;
        bad |= (ms != ms);
        const float mn = fmaxf(M, ms);
        const float sa = (mn == -INFINITY) ? 1.f : exp2f(M - mn);
        const float sb = (ms == -INFINITY) ? 0.f : exp2f(ms - mn);
        acc = acc * sa + ov[u] * sb;
        Ls = Ls * sa + hd[u].y * sb;
        M = mn;
      }
    };
    issue(grp);
    consume(grp);
    for (int s0 = grp + kMergeU * ngroups; s0 < n_splits; s0 += kMergeU * ngroups) {
      issue(s0);
      consume(s0);
    }
    cm[tid] = bad ? NAN : M;
    cl[tid] = Ls;
    cacc[tid] = acc;
    __syncthreads();
    if (tid < width) {
      M = cm[tid];
      Ls = cl[tid];
      acc = cacc[tid];
      bad = M != M;
      for (int q = 1; q < ngroups; ++q) {
        const float ms = cm[q * width + tid];
        bad |= (ms != ms);
        if (ms > -INFINITY) {
          const float mn = fmaxf(M, ms);
          const float sa = exp2f(M - mn), sb = exp2f(ms - mn);
          acc = acc * sa + cacc[q * width + tid] * sb;
          Ls = Ls * sa + cl[q * width + tid] * sb;
          M = mn;
        }
      }
      hook.fold(h, c4, M, Ls, acc);
      const float inv_l = bad ? NAN : (Ls > 0.f ? 1.f / Ls : 0.f);
      reinterpret_cast<v4f*>(osum)[h * (kD / 4) + c4] = acc * inv_l;
    }
    __syncthreads();
  }
  // (b) o = T_V o~.
  tv.apply(osum, ored, G, [&](int h, int j, float o) {
    out_rows[(int64_t)h * kD + j] = hook.add1(h, j, o);
  });
  if (tid == 0) counters[row * kCtrStride] = 0u;
}

// The merge of the MFMA kernel.  The partials go in batches of SB splits.  For each head
// one of waves 2.. (the table waves) keeps the running maximum M and sum L, and per batch
// writes the rescale 2^(M_old - M) and the splits' weights 2^(m_s - M) to LDS; every
// thread loads the partial vectors of one (head, channel quad) unit for its group's SU
// splits of the batch (16-byte loads) and adds them up with those weights after the
// batch's barrier.  Waves 0 and 1 run the hook's encode while their loads are in flight
// (the first barrier also publishes it).  The NG group sums of a unit meet in LDS; then
// each output element (head h, channel c) takes its one more hook term and goes into the
// B operands of o = T_V o~.
// LDS: T_V B operands (12 KiB) | weights [2][NH][SB] | rescales [2][NH] | (M, L, bad) [NH]
// | group sums [NG][NU] (16 B each).  Every run has loaded tv during its last value phase, so
// the merging one starts with T_V in registers.
template <int NTHR, int NH>
struct WideMerge {
  static constexpr int NW = NTHR / 64;
  static constexpr int NU = NH * (kD / 4);            // (head, channel quad) units
  static constexpr int NG = NTHR / NU;                // split groups
  static constexpr int SU = 8;                        // splits per thread and batch
  static constexpr int SB = SU * NG;                  // splits per batch
  static constexpr int NTW = NW - 2;                  // table waves
  static constexpr int NHW = (NH + NTW - 1) / NTW;    // heads per table wave
  static constexpr int NP = (NH * kD + NTHR - 1) / NTHR;   // output elements per thread
  static_assert(NG >= 1 && NG * NU == NTHR && SB <= 64 && NTW >= 1, "thread mapping");
  static constexpr int kWt = 3 * TvMfma::kOperand / 2;   // float offsets of the regions
  static constexpr int kSa = kWt + 2 * NH * SB;
  static constexpr int kFin = kSa + 2 * NH;
  static constexpr int kRed = (kFin + 4 * NH + 3) / 4 * 4;
  static_assert(NTHR == kMfmaThreads && kRed + 4 * NTHR == wide_merge_floats(NH), "merge scratch");
};

template <int NTHR, int NH, class Hook>
__device__ __forceinline__ void merge_if_last_wide(int G, int n_splits, const Partial* parts,
                                                   unsigned* counter, float* out_rows, float* lds,
                                                   TvMfma& tv, bool triple, Hook& hook) {
  using WM = WideMerge<NTHR, NH>;
  constexpr int SU = WM::SU, SB = WM::SB, NU = WM::NU, NTW = WM::NTW, NHW = WM::NHW;
  __shared__ unsigned last_s;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  __builtin_amdgcn_s_waitcnt(0);          // this thread's partial stores have completed
  __syncthreads();
  if (tid == 0) {
    const unsigned prev =
        __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    last_s = (prev == (unsigned)n_splits - 1u) ? 1u : 0u;
  }
  __syncthreads();
  if (!last_s) return;
  hook.prefetch();
  __builtin_amdgcn_sched_barrier(0);
  __bf16* ob = reinterpret_cast<__bf16*>(lds);
  float* wt = lds + WM::kWt;
  float* sat = lds + WM::kSa;
  v4f* fin = reinterpret_cast<v4f*>(lds + WM::kFin);
  v4f* red = reinterpret_cast<v4f*>(lds + WM::kRed);
  const __amdgpu_buffer_rsrc_t prs = make_rsrc(parts, (uint32_t)(n_splits * G * sizeof(Partial)));
  // 32-bit offsets: the descriptor covers less than 2^31 bytes.
  const uint32_t step = (uint32_t)G * (uint32_t)sizeof(Partial);
  const int u = tid % NU, q = tid / NU, h = u / (kD / 4), c4 = u % (kD / 4);
  const bool unit_on = h < G;
  const bool table = wave >= 2;
  float tM[NHW], tL[NHW];
  bool tbad[NHW];
#pragma unroll
  for (int i = 0; i < NHW; ++i) {
    tM[i] = -INFINITY;
    tL[i] = 0.f;
    tbad[i] = false;
  }
  v2f thd[NHW];
  v4f ov[SU];
  v4f acc = {0.f, 0.f, 0.f, 0.f};
  // A batch's loads (past the last split or head they read 0): the table waves' (m, l)
  // first, then every thread's vectors.
  auto issue = [&](int s0) {
    if (table) {
#pragma unroll
      for (int i = 0; i < NHW; ++i) {
        const int h2 = wave - 2 + NTW * i;
        const bool on = (h2 < G) & (lane < SB) & (s0 + lane < n_splits);
        thd[i] = buf_load8_coherent(
            prs, on ? (uint32_t)(s0 + lane) * step + (uint32_t)h2 * (uint32_t)sizeof(Partial)
                    : 0x80000000u);
      }
    }
#pragma unroll
    for (int k = 0; k < SU; ++k) {
      const int sp = s0 + q * SU + k;
      const bool on = unit_on & (sp < n_splits);
      ov[k] = buf_load16_coherent(
          prs, on ? (uint32_t)sp * step + (uint32_t)h * (uint32_t)sizeof(Partial) + 16u +
                        16u * (uint32_t)c4
                  : 0x80000000u);
    }
  };
  // The table waves' part of a batch (NaN maxima mark records that did not match).
  auto tables = [&](int s0, int b) {
    if (!table) return;
#pragma unroll
    for (int i = 0; i < NHW; ++i) {
      const int h2 = wave - 2 + NTW * i;
      if (h2 >= G) continue;                         // (uniform over the wave)
      const bool in = (lane < SB) & (s0 + lane < n_splits);
      const float ms = in ? thd[i].x : -INFINITY;
      tbad[i] |= __builtin_amdgcn_ballot_w64(ms != ms) != 0;
      const float mn = fmaxf(tM[i], wave_max_dpp(ms));    // (NaN lanes are ignored)
      // (the hardware exp2: weights below 2^-126 of the largest flush to 0)
      const float sa = (mn == -INFINITY) ? 1.f : __builtin_amdgcn_exp2f(tM[i] - mn);
      const float w = (ms == -INFINITY || ms != ms) ? 0.f : __builtin_amdgcn_exp2f(ms - mn);
      tL[i] = tL[i] * sa + wave_sum_dpp(w * thd[i].y);
      tM[i] = mn;
      if (lane < SB) wt[((b & 1) * NH + h2) * SB + lane] = w;
      if (lane == 0) sat[(b & 1) * NH + h2] = sa;
    }
  };
  auto accumulate = [&](int b) {
    if (!unit_on) return;
    const v4f* wv = reinterpret_cast<const v4f*>(wt + ((b & 1) * NH + h) * SB + q * SU);
    const float sa = sat[(b & 1) * NH + h];
    float w[SU];
#pragma unroll
    for (int k = 0; k < SU / 4; ++k) {
      const v4f x = wv[k];
      w[4 * k] = x[0], w[4 * k + 1] = x[1], w[4 * k + 2] = x[2], w[4 * k + 3] = x[3];
    }
    v4f a0 = acc * sa, a1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < SU; k += 2) {
      a0 += w[k] * ov[k];
      a1 += w[k + 1] * ov[k + 1];
    }
    acc = a0 + a1;
  };
  issue(0);
  // While the loads are in flight: the hook's encode in waves 0 and 1, the split of T_V in the
  // rest (theirs after the sums).
  if (triple && wave >= 2) tv.split();
  hook.encode();
  for (int s0 = 0, b = 0;; ++b) {
    tables(s0, b);
    __syncthreads();                      // the batch's weights (first: the hook's encode)
    accumulate(b);
    s0 += SB;
    if (s0 >= n_splits) break;
    issue(s0);
  }
  if (triple && wave < 2) tv.split();
  if (table && lane == 0) {
#pragma unroll
    for (int i = 0; i < NHW; ++i) {
      const int h2 = wave - 2 + NTW * i;
      if (h2 < G) fin[h2] = (v4f){tM[i], tL[i], tbad[i] ? 1.f : 0.f, 0.f};
    }
  }
  red[q * NU + u] = acc;
  __syncthreads();
#pragma unroll
  for (int p = 0; p < WM::NP; ++p) {
    const int slot = p * NTHR + tid, hh = slot / kD, c = slot % kD;
    if (hh < G) {
      float a = 0.f;
#pragma unroll
      for (int g = 0; g < WM::NG; ++g)
        a += reinterpret_cast<const float*>(red + g * NU + hh * (kD / 4))[c];
      const v4f f = fin[hh];
      float M = f[0], Ls = f[1];
      hook.fold1(hh, c, M, Ls, a);
      // (0 only for an empty row: a NaN among the scores, from a NaN or infinite query, leaves
      // the maximum and the integer sums without a trace, but not L)
      TvMfma::put(ob, hh, c, f[2] != 0.f || Ls != Ls ? NAN : (Ls > 0.f ? a / Ls : 0.f), triple);
    }
  }
  __syncthreads();
  // o = T_V o~ (the partials are in the transformed domain).
  tv.apply(ob, G, triple, [&](int hh, int j0, v4f o) {
    *reinterpret_cast<v4f*>(out_rows + (int64_t)hh * kD + j0) = hook.add4(hh, j0, o);
  });
  hook.finish();
  if (tid == 0) *counter = 0u;
}

// ---------------------------------------------------------------------------------------
// Full-precision segment (the first tokens and the recent window kept at input precision,
// Sec. 6 and App. E): exact softmax attention of each query head over the segment's tokens
// in the original domain, one workgroup per (sequence, KV head), written as one more split
// partial (log2-domain maximum and sum of its weights, sum_t p_t v_t in the original domain),
// which the merge of the compressed-cache splits folds in: its weight in the softmax before
// the inverse transform, its value sum after it.
//
// A few tens of KB per workgroup: the time is latency.  Sixteen waves, four tokens per wave at
// once (16 lanes x 8 elements a row, 16-byte loads), every key load of a wave in flight
// together; the value sums with a wave per (head, share of the tokens).  Batch 8, 8 KV heads,
// 132 tokens: 125 us before (a thread per token with scalar loads, and T_V^T applied here).
// ---------------------------------------------------------------------------------------
constexpr int kSegThreads = 1024;
constexpr int kSegWaves = kSegThreads / 64;
constexpr int kSegMax = 256;           // tokens of one segment
constexpr int kSegIt = kSegMax / (4 * kSegWaves);   // key rows per lane group

// Elements 8 e .. 8 e + 7 of a row as fp32 (vec: rows 16-byte aligned).
__device__ inline void load_row8(const void* base, int dtype, int64_t row, int e, bool vec,
                                 float (&v)[8]) {
  if (vec && dtype == AATC_BF16) {
    const uint4 u = *reinterpret_cast<const uint4*>(static_cast<const uint16_t*>(base) + row * kD + 8 * e);
    const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      v[2 * i] = __uint_as_float(w[i] << 16);
      v[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
    }
  } else if (vec) {
    const v4f* p = reinterpret_cast<const v4f*>(static_cast<const float*>(base) + row * kD + 8 * e);
    const v4f a = p[0], b = p[1];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      v[i] = a[i];
      v[4 + i] = b[i];
    }
  } else {
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = load_elem(base, dtype, row * kD + 8 * e + i);
  }
}

__global__ __launch_bounds__(kSegThreads) void segment_partial_kernel(
    int n_q_heads, int n_kv_heads, const void* __restrict__ q, int q_dtype,
    const void* __restrict__ seg_k, const void* __restrict__ seg_v, int seg_dtype,
    const int32_t* __restrict__ seg_len, int seg_cap, float scale_log2e,
    Partial* __restrict__ seg_out) {
  __shared__ __align__(16) float qs[kMaxGroup][kD];
  __shared__ float z[kMaxGroup][kSegMax];
  __shared__ __align__(16) float ored[kSegWaves][kD];
  const int row = blockIdx.x, kvh = row % n_kv_heads, seq = row / n_kv_heads;
  const int G = n_q_heads / n_kv_heads;
  const int tid = threadIdx.x, lane = tid & 63, e = lane & 15, tr = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = min(max(seg_len[seq], 0), seg_cap);
  Partial* out = seg_out + (int64_t)row * G;
  if (n == 0) {                                        // (uniform, before any barrier)
    for (int i = tid; i < G * kD; i += kSegThreads) out[i / kD].o[i % kD] = 0.f;
    if (tid < G) {
      out[tid].m = -INFINITY;
      out[tid].l = 0.f;
    }
    return;
  }
  const int64_t tok0 = (int64_t)row * seg_cap;         // [batch][n_kv_heads][seg_cap][d]
  const bool vec = ((reinterpret_cast<uintptr_t>(seg_k) | reinterpret_cast<uintptr_t>(seg_v)) & 15u) == 0u;
  // Key rows 64 i + 4 wave + tr (past the end clamped to the last row: their logits are
  // dropped), then the queries.
  float kr[kSegIt][8];
#pragma unroll
  for (int i = 0; i < kSegIt; ++i)
    if (64 * i < n)                                    // (uniform)
      load_row8(seg_k, seg_dtype, tok0 + min(64 * i + 4 * wave + tr, n - 1), e, vec, kr[i]);
  for (int i = tid; i < G * kD; i += kSegThreads)
    qs[i / kD][i % kD] =
        load_q(q, q_dtype, ((int64_t)seq * n_q_heads + kvh * G) * kD + i) * scale_log2e;
  __syncthreads();
#pragma unroll 1
  for (int h = 0; h < G; ++h) {
    const v4f q0 = *reinterpret_cast<const v4f*>(&qs[h][8 * e]), q1 = *reinterpret_cast<const v4f*>(&qs[h][8 * e + 4]);
#pragma unroll
    for (int i = 0; i < kSegIt; ++i) {
      if (64 * i >= n) break;                          // (uniform)
      float a = 0.f;
#pragma unroll
      for (int k = 0; k < 4; ++k) a = fmaf(q0[k], kr[i][k], fmaf(q1[k], kr[i][4 + k], a));
      a = row16_sum(a);
      if (e == 0) z[h][64 * i + 4 * wave + tr] = a;
    }
  }
  __syncthreads();
  // Maximum, weights 2^(z - m) and their sum: wave h takes head h.
  if (wave < G) {
    float zl[kSegMax / 64], m = -INFINITY, l = 0.f;
#pragma unroll
    for (int i = 0; i < kSegMax / 64; ++i) {
      zl[i] = lane + 64 * i < n ? z[wave][lane + 64 * i] : -INFINITY;
      m = fmaxf(m, zl[i]);
    }
    m = wave_max_dpp(m);
#pragma unroll
    for (int i = 0; i < kSegMax / 64; ++i) {
      const float p = lane + 64 * i < n ? exp2f(zl[i] - m) : 0.f;
      z[wave][lane + 64 * i] = p;
      l += p;
    }
    l = wave_sum_dpp(l);
    if (lane == 0) {
      out[wave].m = m;
      out[wave].l = l;
    }
  }
  __syncthreads();
  // Value sums: wave (share, head) of Gp = G rounded up to a power of two heads; a lane group
  // takes every fourth token of the share, four rows in flight.
  const int lg = G > 1 ? 32 - __builtin_clz((unsigned)(G - 1)) : 0;
  const int h = wave & ((1 << lg) - 1), step = 4 * (kSegWaves >> lg);
  float acc[8] = {};
  if (h < G) {
    for (int t0 = 4 * (wave >> lg) + tr; t0 < n + tr; t0 += 4 * step) {   // (uniform trip count)
      float vr[4][8], p[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int t = t0 + u * step;
        load_row8(seg_v, seg_dtype, tok0 + min(t, n - 1), e, vec, vr[u]);
        p[u] = t < n ? z[h][min(t, n - 1)] : 0.f;
      }
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int k = 0; k < 8; ++k) acc[k] = t0 + u * step < n ? fmaf(p[u], vr[u][k], acc[k]) : acc[k];
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) acc[k] = xor32_sum(xor16_sum(acc[k]));
    if (tr == 0) {
      *reinterpret_cast<v4f*>(&ored[wave][8 * e]) = (v4f){acc[0], acc[1], acc[2], acc[3]};
      *reinterpret_cast<v4f*>(&ored[wave][8 * e + 4]) = (v4f){acc[4], acc[5], acc[6], acc[7]};
    }
  }
  __syncthreads();
  for (int i = tid; i < G * kD; i += kSegThreads) {
    const int hh = i / kD, j = i % kD;
    float o = 0.f;
    for (int w = hh; w < kSegWaves; w += 1 << lg) o += ored[w][j];
    out[hh].o[j] = o;
  }
}

// The merging workgroup folds the segment's partial of its (sequence, KV head) (written by
// segment_partial_kernel, which ran before this launch): its weight enters the softmax of
// every output element, its value sum is added after the inverse transform.
struct SegHook {
  const Partial* seg;                  // this row's partials
  float* w;                            // LDS: the segment's final weight per head
  __device__ void prefetch() {}
  __device__ void encode() {}
  template <class V>
  __device__ void weigh(int h, bool first, float& M, float& Ls, V& acc) const {
    const float ms = seg[h].m;
    float f = 0.f;
    if (seg[h].l != 0.f) {             // (0 for an empty segment; NaN scores are kept)
      const float mn = fmaxf(M, ms);
      const float sa = exp2f(M - mn), sb = exp2f(ms - mn);
      acc = acc * sa;
      Ls = Ls * sa + seg[h].l * sb;
      M = mn;
      f = sb / Ls;
    }
    if (first) w[h] = f;
  }
  __device__ void fold1(int h, int c, float& M, float& Ls, float& acc) const {
    weigh(h, c == 0, M, Ls, acc);
  }
  __device__ void fold(int h, int c4, float& M, float& Ls, v4f& acc) const {
    weigh(h, c4 == 0, M, Ls, acc);
  }
  __device__ float add1(int h, int j, float o) const {
    return w[h] != 0.f ? fmaf(w[h], seg[h].o[j], o) : o;
  }
  __device__ v4f add4(int h, int j0, v4f o) const {
    return w[h] != 0.f ? o + w[h] * *reinterpret_cast<const v4f*>(seg[h].o + j0) : o;
  }
  __device__ void finish() {}
};

// ---------------------------------------------------------------------------------------
// Generic VALU kernel (any G <= 16, any budget).
// ---------------------------------------------------------------------------------------
// Fused append.  The splits stop short of the new token (position len - 1) and share its
// encode (exactly the encode kernels' arithmetic): split s computes the transformed
// coefficients r_c = h_c / s_c of the dot products d = s + n_splits (w + 8 i) of the
// 2 x 128 (key channels, then value channels), one per wave, and stores them in the
// workspace.  The merging workgroup loads the 256 coefficients ahead of the partials and,
// while those are in flight, takes the token scales, quantizes, and forms the token's score
// z = alpha^K sum_c Q_c 2^(1 - b_c) code_c per head (Q_c: the key phase's channel weights)
// and transformed value v~_c = alpha^V s_c 2^(1 - b_c) code_c; it folds them into the
// merge as one more term and writes the codes into both caches.  Every split has been read
// when the last one arrives, so nothing else touches the new slot.
// ---------------------------------------------------------------------------------------
struct AppendScratch {                 // LDS region of its own
  uint32_t erec[2][kMaxBudget / 32];   // key record, value record
  float vnew[kD];                      // transformed value of the token
  float znew[16];                      // the token's log2-domain score per head
  uint32_t ea16[2];                    // fp16 scales
};
static_assert((sizeof(AppendScratch) + 15) / 16 * 16 == kAppendScratchBytes, "append scratch");

// r = h~ / s of F transformed coefficients of the appended token (the encode kernels'
// arithmetic, reductions interleaved), from this lane's two elements of the token (raw
// dwords: bf16 halves or fp32) and of the coefficient's column of the integer transform:
// X_j = rint(x_j 2^S) with max |X| in [2^21, 2^22), H = sum_j X_j Tq_jc exact (each lane's
// two products below 2^45, the wave sums taken as 24-bit halves in int32), h~ =
// fl32(H 2^-(S+22)).  eh = E 2^-S (1 + 2^-16), E = sum_j |x_j 2^S - X_j|, bounds |h - h~|
// for the exact h (eh = 0: h~ is exact; NaN or infinite with a NaN or infinite element, and where
// 2^S is below 1 and E could underflow).
template <int F>
__device__ inline void append_coefficients(const uint32_t (&x)[F][2], const int (&t)[F][2],
                                           int x_dtype, const float (&inv_s)[F], float (&out)[F],
                                           float (&eh)[F]) {
  const int lane = threadIdx.x & 63;
  const bool bf = x_dtype == AATC_BF16;
  float xa[F], xb[F], m[F];
#pragma unroll
  for (int f = 0; f < F; ++f) {
    xa[f] = bf ? __uint_as_float(((lane & 1) ? (x[f][0] >> 16) : (x[f][0] & 0xffffu)) << 16)
               : __uint_as_float(x[f][0]);
    xb[f] = bf ? __uint_as_float(((lane & 1) ? (x[f][1] >> 16) : (x[f][1] & 0xffffu)) << 16)
               : __uint_as_float(x[f][1]);
    m[f] = fmaxf(fabsf(xa[f]), fabsf(xb[f]));
  }
  wave_max_n(m);
  int shift[F], hl[2 * F];
  float E[F];
#pragma unroll
  for (int f = 0; f < F; ++f) {
    shift[f] = token_shift(m[f]);
    const float va = ldexpf(xa[f], shift[f]), vb = ldexpf(xb[f], shift[f]);
    const float ra = rintf(va), rb = rintf(vb);
    E[f] = fabsf(va - ra) + fabsf(vb - rb);
    const long long p = (long long)(int)ra * t[f][0] + (long long)(int)rb * t[f][1];
    hl[2 * f] = (int)(p >> 24);
    hl[2 * f + 1] = (int)(p & 0xffffff);
  }
  wave_sum_i32_n(hl);
  wave_sum_n(E);
#pragma unroll
  for (int f = 0; f < F; ++f) {
    const double H = fma((double)hl[2 * f], 16777216.0, (double)hl[2 * f + 1]);
    out[f] = integer_result(H, shift[f]) * inv_s[f];
    eh[f] = shift[f] < 0 ? INFINITY : ldexpf(E[f] * (1.f + 0x1p-16f), -shift[f]);
  }
}

template <int NTHR, int NH>
struct AppendHook {
  static_assert(NTHR >= 2 * kD && NH <= 16, "thread mapping");
  uint8_t* k_codes;
  uint16_t* k_alpha;
  uint8_t* v_codes;
  uint16_t* v_alpha;
  const float* coeff;                  // this row's coefficients and bounds (workspace)
  const HeadParams* ehp[2];            // key and value parameters of this KV head
  const void* xrow[2];                 // the new key and value token of this row
  int x_dtype;
  int64_t row, cap;
  int len, G, rk, rv;
  bool on;                             // the sequence has a token to append
  // Wave 0 encodes the key token, wave 1 the value token, lane l channels l and l + 64:
  int e_b[2], e_off[2];                // their widths and first record bits
  bool e_mr;                           // the wave's tensor uses the midrise reading
  float e_s[2];                        // their scales s_c (value token)
  const float* qc;                     // Q_c of every head [NH][kD] (LDS; key token)
  AppendScratch* sc;
  float r2[2];                         // their coefficients r_c = h_c / s_c
  float eh;                            // the wave's token: fixed-point error bound

  __device__ void prefetch() {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const __amdgpu_buffer_rsrc_t rs =
        make_rsrc(coeff, (on && wave < 2) ? (uint32_t)(kAppStride * 4) : 0u);
#pragma unroll
    for (int i = 0; i < 2; ++i)
      r2[i] = __int_as_float(__builtin_amdgcn_raw_buffer_load_b32(
          rs, 4 * ((wave & 1) * kD + lane + 64 * i), 0, kCoherent));
    eh = __int_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, 4 * (2 * kD + (wave & 1)), 0,
                                                             kCoherent));
  }

  // The token's codes, scales, score per head and transformed value, each tensor by one
  // wave (wave reductions only); the merge's next barrier makes them visible.
  __device__ void encode() {
    if (!on) return;                   // uniform over the workgroup
    float qk[2][NH];                   // (read here: no LDS round trip behind a branch later)
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (wave < 2) {
      const int et = wave;
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int h = 0; h < NH; ++h) qk[i][h] = qc[h * kD + lane + 64 * i];
      if (lane < kMaxBudget / 32) sc->erec[et][lane] = 0u;
      // A token that is not exact in fixed point keeps its coefficients if the certificate
      // holds; otherwise (rarely) the exact routine recomputes them.
      const float ehw = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(eh)));
      const HeadParams* ep = et ? ehp[1] : ehp[0];
      if (!(ehw <= 0.f) && !wave_certify(ep, r2, ehw)) {
        const void* xr = et ? xrow[1] : xrow[0];
        float xl[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) xl[i] = load_elem(xr, x_dtype, lane + 64 * i);
        exact_r_wave(ep, xl, r2);
      }
      float m = 0.f;
#pragma unroll
      for (int i = 0; i < 2; ++i) m = fmaxf(m, e_b[i] > 0 ? fabsf(r2[i]) : 0.f);
      const __half a16 = token_alpha(wave_max_dpp(m));
      const float inv = inverse_alpha(a16);
      const bool midrise = e_mr;
      float code[2];                   // the level in steps: code, or code + 1/2 (midrise)
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        code[i] = 0.f;
        const int eb = e_b[i], eoff = e_off[i];
        if (eb > 0) {
          const uint32_t u = quantize_code(r2[i], inv, eb, midrise);
          atomicOr(&sc->erec[et][eoff >> 5], u << (eoff & 31));
          if ((eoff & 31) + eb > 32) atomicOr(&sc->erec[et][(eoff >> 5) + 1], u >> (32 - (eoff & 31)));
          code[i] = (float)((int)(u << (32 - eb)) >> (32 - eb)) + (midrise ? 0.5f : 0.f);
        }
      }
      const float af = __half2float(a16);
      if (et == 0) {
        float z[NH];
#pragma unroll
        for (int h = 0; h < NH; ++h) {
          z[h] = 0.f;
#pragma unroll
          for (int i = 0; i < 2; ++i)
            z[h] += e_b[i] ? qk[i][h] * ldexpf(code[i], 1 - e_b[i]) : 0.f;
        }
        wave_sum_n(z);
#pragma unroll
        for (int h = 0; h < NH; ++h)
          if (lane == 0) sc->znew[h] = af * z[h];
      } else {
#pragma unroll
        for (int i = 0; i < 2; ++i)
          sc->vnew[lane + 64 * i] = e_b[i] ? ldexpf(af * e_s[i] * code[i], 1 - e_b[i]) : 0.f;
      }
      if (lane == 0) sc->ea16[et] = __half_as_ushort(a16);
    }
  }
  // The token's log2-domain score for head h.
  __device__ float znew(int h) const { return sc->znew[h]; }

  __device__ v4f add4(int, int, v4f o) const { return o; }
  __device__ void fold1(int h, int c, float& M, float& Ls, float& acc) const {
    if (!on) return;
    const float ms = znew(h);
    const float mn = fmaxf(M, ms);
    const float sa = __builtin_amdgcn_exp2f(M - mn), sb = __builtin_amdgcn_exp2f(ms - mn);
    acc = acc * sa + sc->vnew[c] * sb;
    Ls = Ls * sa + sb;
    M = mn;
  }

  // The codes go to the caches last: the key record and both scales, and the token's
  // bits of its value tile (one atomic per record bit: the tile's other tokens share
  // those words).
  __device__ void finish() {
    if (!on) return;
    const int tid = threadIdx.x;
    const int64_t tg = row * cap + (len - 1);
    for (int i = tid; i < rk / 4; i += NTHR)
      reinterpret_cast<uint32_t*>(k_codes + tg * rk)[i] = sc->erec[0][i];
    if (tid == 0) {
      k_alpha[tg] = (uint16_t)sc->ea16[0];
      v_alpha[tg] = (uint16_t)sc->ea16[1];
    }
    const int p = len - 1, tp = p & (kTile - 1);
    const uint32_t bit = 1u << tile_bit(tp);
    uint32_t* gt = reinterpret_cast<uint32_t*>(v_codes + (row * cap + (p - tp)) * rv) + tile_word(tp);
    for (int v = tid; v < 8 * rv; v += NTHR) {
      if ((sc->erec[1][v >> 5] >> (v & 31)) & 1u)
        __hip_atomic_fetch_or(&gt[2 * v], bit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      else
        __hip_atomic_fetch_and(&gt[2 * v], ~bit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
};

// ---------------------------------------------------------------------------------------
__global__ __launch_bounds__(kThreads) void decode_split_kernel(
    const void* __restrict__ params_k, const void* __restrict__ params_v, int n_q_heads,
    int n_kv_heads, const void* __restrict__ q, int q_dtype,
    const uint8_t* __restrict__ k_codes, const uint16_t* __restrict__ k_alpha,
    const uint8_t* __restrict__ v_codes, const uint16_t* __restrict__ v_alpha,
    const int32_t* __restrict__ seq_len, int64_t cap, float scale, float* __restrict__ out,
    unsigned* __restrict__ counters, Partial* __restrict__ partials, int n_splits, int rk,
    int rv, const Partial* __restrict__ seg) {
  extern __shared__ float dyn[];
  __shared__ float qs[kMaxGroup][kD];
  __shared__ float qp[kMaxGroup][kD];
  __shared__ float red[kThreads / 64];
  __shared__ float mh[kMaxGroup], lh[kMaxGroup];
  __shared__ float chq[kMaxGroup];      // midrise: the half-step term of the scores
  __shared__ float wh[kMaxGroup];       // sum over the split of P alpha^V

  const int split = blockIdx.x, kvh = blockIdx.y, seq = blockIdx.z;
  const int G = n_q_heads / n_kv_heads;
  const int tid = threadIdx.x;
  const HeadParams* hk = head_params(params_k, kvh);
  const HeadParams* hv = head_params(params_v, kvh);
  const bool layout_ok = hk->record_bytes == rk && hv->record_bytes == rv;
  const int bk = hk->budget, bv = hv->budget;
  const int VS = 8 * max(rk, rv);                   // record bits of the wider tensor
  float* sc = dyn;                                  // [G][kSplit] logits, then weights
  float* vq = dyn + G * kSplit;                     // [G][VS] per-bit weights / sums

  const int len = (int)min<int64_t>(max(seq_len[seq], 0), cap);   // out-of-range lengths clamp
  const int t0 = split * kSplit;
  const int nt = layout_ok ? max(0, min(kSplit, len - t0)) : 0;

  // Queries of the group, then q'_c = (T_K^T q)_c * s_c * 2^(1-b_c) * scale * log2(e).
  for (int i = tid; i < G * kD; i += kThreads)
    qs[i / kD][i % kD] = load_q(q, q_dtype, ((int64_t)seq * n_q_heads + kvh * G) * kD + i);
  __syncthreads();
  for (int i = tid; i < G * kD; i += kThreads) {
    const int h = i / kD, c = i % kD;
    float acc = 0.f;
#pragma unroll 16
    for (int j = 0; j < kD; ++j) acc += hk->T[j * kD + c] * qs[h][j];
    const int b = hk->bits[c];
    qp[h][c] = b ? acc * hk->s[c] * ldexpf(1.f, 1 - b) * scale * kLog2e : 0.f;
  }
  __syncthreads();
  // Weight of record bit v: q'_c 2^k, negated for the sign bit k = b_c - 1.
  for (int i = tid; i < G * bk; i += kThreads) {
    const int h = i / bk, v = i % bk;
    const int c = hk->virt_chan[v], k = hk->virt_bit[v];
    const float w = ldexpf(qp[h][c], k);
    vq[h * VS + v] = (k == hk->bits[c] - 1) ? -w : w;
  }
  // Midrise levels (code + 1/2) add (1/2) sum_c q'_c to every score (before alpha^K).
  if (tid < G) {
    float a = 0.f;
    if (hk->quantizer == AATC_QUANT_MIDRISE)
      for (int c = 0; c < kD; ++c) a += qp[tid][c];
    chq[tid] = 0.5f * a;
  }
  __syncthreads();

  // Scores z = alpha^K sum_v Q_v bit_v in the log2 domain.
  const int64_t kv_row = (int64_t)seq * n_kv_heads + kvh;
  for (int tl = tid; tl < kSplit; tl += kThreads) {
    float acc[kMaxGroup];
#pragma unroll
    for (int h = 0; h < kMaxGroup; ++h) acc[h] = 0.f;
    if (tl < nt) {
      const int64_t t = t0 + tl;
      const uint32_t* rec = reinterpret_cast<const uint32_t*>(k_codes + (kv_row * cap + t) * rk);
      for (int w = 0; w < rk / 4; ++w) {
        uint32_t bits = rec[w];
        while (bits) {
          const int v = 32 * w + __builtin_ctz(bits);
          bits &= bits - 1;
#pragma unroll
          for (int h = 0; h < kMaxGroup; ++h)
            if (h < G) acc[h] += vq[h * VS + v];
        }
      }
      const float ak = half_bits_to_float(k_alpha[kv_row * cap + t]);
#pragma unroll
      for (int h = 0; h < kMaxGroup; ++h)
        if (h < G) sc[h * kSplit + tl] = ak * (acc[h] + chq[h]);
    } else {
      for (int h = 0; h < G; ++h) sc[h * kSplit + tl] = -INFINITY;
    }
  }
  __syncthreads();

  // Split-local softmax statistics per head; weights become 2^(z - m) * alpha^V.
  for (int h = 0; h < G; ++h) {
    float m = -INFINITY;
    for (int tl = tid; tl < kSplit; tl += kThreads) m = fmaxf(m, sc[h * kSplit + tl]);
    m = block_reduce(m, true, red);
    float l = 0.f;
    for (int tl = tid; tl < kSplit; tl += kThreads) {
      float p = (tl < nt) ? exp2f(sc[h * kSplit + tl] - m) : 0.f;
      float w = (tl < nt) ? p * half_bits_to_float(v_alpha[kv_row * cap + t0 + tl]) : 0.f;
      sc[h * kSplit + tl] = w;
      l += p;
    }
    l = block_reduce(l, false, red);
    float ws = 0.f;
    for (int tl = tid; tl < nt; tl += kThreads) ws += sc[h * kSplit + tl];
    ws = block_reduce(ws, false, red);
    if (tid == 0) {
      mh[h] = m;
      lh[h] = l;
      wh[h] = ws;
    }
  }
  __syncthreads();

  // Value bits: sum over tokens of w_t * bit_v(t), one thread per record bit.
  const uint32_t* vt = reinterpret_cast<const uint32_t*>(v_codes) +
                       (kv_row * (cap / kTile) + t0 / kTile) * (16 * rv);
  for (int v = tid; v < bv; v += kThreads) {
    float acc[kMaxGroup];
#pragma unroll
    for (int h = 0; h < kMaxGroup; ++h) acc[h] = 0.f;
    for (int tile = 0; tile * kTile < nt; ++tile) {
      for (int W = 0; W < 2; ++W) {
        uint32_t word = vt[tile * 16 * rv + 2 * v + W];
        while (word) {
          const int p = __builtin_ctz(word);
          word &= word - 1;
          // bit p of word W: token 16 d + 4 g + i, d = 2 W + p % 2, g = p / 2 % 4, i = p / 8
          const int t = tile * kTile + 16 * (2 * W + (p & 1)) + 4 * ((p >> 1) & 3) + (p >> 3);
          if (t >= nt) continue;
#pragma unroll
          for (int h = 0; h < kMaxGroup; ++h)
            if (h < G) acc[h] += sc[h * kSplit + t];
        }
      }
    }
#pragma unroll
    for (int h = 0; h < kMaxGroup; ++h)
      if (h < G) vq[h * VS + v] = acc[h];
  }
  __syncthreads();

  // Partial o~_c = s_c 2^(1-b_c) (sum_{k < b-1} 2^k S_(c,k) - 2^(b-1) S_(c,b-1)).
  Partial* part = partials + (kv_row * n_splits + split) * G;
  for (int i = tid; i < G * kD; i += kThreads) {
    const int h = i / kD, c = i % kD;
    const int b = hv->bits[c];
    float o = 0.f;
    if (b && nt > 0) {
      float acc = 0.f;
      for (int k = 0; k < b; ++k) {
        const float t = ldexpf(vq[h * VS + hv->bit_off[c] + k], k);
        acc += (k == b - 1) ? -t : t;
      }
      // (midrise: the half step of every level, s_c 2^(-b_c) sum_t P_t alpha^V_t)
      o = fmaf(hv->s[c] * hv->half_step[c], wh[h], hv->s[c] * ldexpf(acc, 1 - b));
    }
    st_dev(&part[h].o[c], o);
  }
  if (tid < G) {
    st_dev(&part[tid].m, !layout_ok ? NAN : (nt > 0) ? mh[tid] : -INFINITY);
    st_dev(&part[tid].l, !layout_ok ? NAN : (nt > 0) ? lh[tid] : 0.f);
  }
  float* out_rows = out + ((int64_t)seq * n_q_heads + kvh * G) * kD;
  if (seg) {
    __shared__ float seg_w[kMaxGroup];
    SegHook sh{seg + kv_row * G, seg_w};
    merge_if_last<kThreads>(params_v, kvh, kv_row, G, n_splits, partials, counters,
                                  out_rows, dyn, sh);
  } else {
    NoHook none;
    merge_if_last<kThreads>(params_v, kvh, kv_row, G, n_splits, partials, counters,
                                  out_rows, dyn, none);
  }
}

// Deals the chunks of S tokens of a ragged batch to the workgroups: every workgroup chooses the
// same run length (choose_runs) and finds its row and run from the prefix sums over the
// sequences (64 per pass, one per lane).  A row has max(1, ceil(chunks / q)) runs; workgroups
// without a run return false.  The host gives the grid at least as many workgroups as rows.
// The lengths of the first 64 kSeqBlocks sequences are read at once and stay in registers, and
// sums run over the lanes before the wave (a load, a division and a reduction per 64 sequences and
// pass made 300 sequences of 4000 tokens 95 us, 83 now).
constexpr int kSeqBlocks = 8;
__device__ inline int clamped_chunks(int len, int64_t cap, int S, int app) {
  return max(1, ((int)min<int64_t>(max(len, 0), cap) - app + S - 1) / S);
}
template <int S, bool APPEND>
__device__ inline bool assign_runs(const int32_t* seq_len, int64_t cap, int batch, int rps,
                                   int& vrow, int& split, int& ns, int& per, int& len_raw) {
  const int lane = threadIdx.x & 63;                 // (rps: rows per sequence)
  const int nb = (batch + 63) / 64;
  int len[kSeqBlocks], nch[kSeqBlocks];
#pragma unroll
  for (int i = 0; i < kSeqBlocks; ++i) nch[i] = 0;
#pragma unroll
  for (int i = 0; i < kSeqBlocks; ++i) {
    if (i >= nb) break;                              // (uniform)
    len[i] = seq_len[min(64 * i + lane, batch - 1)];
  }
  auto chunks_of = [&](int l, int b) {               // of sequence b, 0 past the batch
    return b < batch ? clamped_chunks(l, cap, S, APPEND ? 1 : 0) : 0;
  };
#pragma unroll
  for (int i = 0; i < kSeqBlocks; ++i) {
    if (i >= nb) break;
    nch[i] = chunks_of(len[i], 64 * i + lane);
  }
  // Calls f(chunks of the lane's sequence) for every block of 64 sequences.
  auto each = [&](auto f) {
#pragma unroll
    for (int i = 0; i < kSeqBlocks; ++i) {
      if (i >= nb) break;
      f(nch[i]);
    }
    for (int b0 = 64 * kSeqBlocks; b0 < batch; b0 += 64)
      f(chunks_of(seq_len[min(b0 + lane, batch - 1)], b0 + lane));
  };
  int sum = 0, most = 0;
  each([&](int n) {
    sum += n;
    most = max(most, n);
  });
  const int tot = __builtin_amdgcn_readfirstlane(wave_sum_i32(sum));
  // (chunks of a row stay below 2^20)
  const int longest = __builtin_amdgcn_readfirstlane((int)wave_max_dpp((float)most));
  const RunPlan p = choose_runs(tot * rps, batch * rps, longest, (int)gridDim.x, [&](int q) {
    const float rq = __builtin_amdgcn_rcpf((float)q);
    int cnt = 0;
    each([&](int n) { cnt += runs_of_row(n, q, rq); });
    return __builtin_amdgcn_readfirstlane(wave_sum_i32(cnt)) * rps;
  });
  const int q = p.q, lb = run_of_block((int)blockIdx.x, p.runs);
  if (lb < 0) return false;
  const float rq = __builtin_amdgcn_rcpf((float)q);
  int left = lb;
  // Whether the workgroup's run is one of sequences b0 .. b0 + 63 (the lane's has n chunks and
  // length l).
  auto find = [&](int b0, int n, int l) {
    const int cnt = runs_of_row(n, q, rq) * rps;
    // inclusive prefix sums: within rows of 16 lanes by row shifts, then the row totals
    int v = cnt;
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);
    const int r0 = __builtin_amdgcn_readlane(v, 15), r1 = __builtin_amdgcn_readlane(v, 31),
              r2 = __builtin_amdgcn_readlane(v, 47);
    v += (lane >= 16 ? r0 : 0) + (lane >= 32 ? r1 : 0) + (lane >= 48 ? r2 : 0);
    const unsigned long long past = __builtin_amdgcn_ballot_w64(v > left);
    if (past) {
      const int i = __builtin_ctzll(past);
      const int cb = __builtin_amdgcn_readlane(cnt, i);
      left -= __builtin_amdgcn_readlane(v, i) - cb;
      ns = cb / rps;
      vrow = (b0 + i) * rps + left / ns;
      split = left % ns;
      per = q;
      len_raw = __builtin_amdgcn_readlane(l, i);
      return true;
    }
    left -= __builtin_amdgcn_readlane(v, 63);
    return false;
  };
#pragma unroll
  for (int i = 0; i < kSeqBlocks; ++i) {
    if (i >= nb) break;
    if (find(64 * i, nch[i], len[i])) return true;
  }
  for (int b0 = 64 * kSeqBlocks; b0 < batch; b0 += 64) {
    const int l = seq_len[min(b0 + lane, batch - 1)];
    if (find(b0, chunks_of(l, b0 + lane), l)) return true;
  }
  return false;
}

// ---------------------------------------------------------------------------------------
// MFMA decode kernel (records of at most 128 bytes; up to 8 query heads of a KV head per
// workgroup, more heads as further workgroups over the same cache).
//
// Both contractions run on v_mfma_i32_16x16x64_i8 over the bits of the codes.
//  * Keys: D[token, (head, limb)] = sum_bits bit(token) * Qlimb[bit, (head, limb)].
//    One record dword w (32 bits of one token) expands to MFMA bytes by
//    r_d = w & (0x01010101 << d): byte j of r_d is 2^d * bit (8j + d).  The factor 2^d
//    (and the sign of int8 0x80 for d = 7) is folded into the query weights, which are
//    32-bit fixed point split into four int8 limbs: four heads times four limbs fill
//    the 16 MFMA columns.  Lane (column (h, L), row group g) of the result holds limb L
//    of the scores of tokens 4g .. 4g + 3; a reduce-scatter over the lane quad leaves
//    lane L with the full score of token 4g + L.  (FINE: the upper four bits of each byte are
//    shifted down first, factor 2^(d & 3).)
//  * Values: D[bit, (head, limb)] = sum_tokens bit(token) * Plimb[token, (head, limb)]
//    with P = 2^(z - m) alpha^V in 32-bit fixed point (one exponent per workgroup).
//    The value tiles store the bit of token 16 d + 4 g + i at bit 8 i + 2 g + d % 2 of
//    word d / 2, so a lane of row group g expands its two words with two masks into
//    exactly the tokens whose scores its quad computed; a byte transpose inside the quad
//    turns (one token, four limbs) per lane into (four tokens, one limb).
// Each wave scores and weights its own share of the split; the value bits are then
// split across the waves, over all tokens of the split.  Integer accumulation is exact;
// limbs are recombined in fp32.
//
// Every workgroup derives its query bit weights itself, while its cache loads are in
// flight: q~ = T_K^T q (fp32), then per bit the 32-bit fixed-point limbs.
//
// Streaming.  A workgroup takes a run of consecutive S-token chunks of its (sequence, KV
// head).  One chunk's compute (masks, products, softmax: about 4-6 us) is longer than its
// 94 KB take to arrive, so a workgroup per chunk leaves the memory idle for most of its life
// and repeats the query planes each time; a run builds them once, has the next chunk's
// records in flight while it computes (the key region is refilled once the scores are
// formed, the value region once the values are summed), and leaves one partial for the
// whole run.
// ---------------------------------------------------------------------------------------
// ONE: evenly dealt and at most one chunk per workgroup, known at the launch (a context that
// every compute unit takes one chunk of): the loop and its refills compiled out (32768 tokens:
// 16.1 -> 15.3 us).
template <int NT, int NTILE, int NP, bool APPEND, bool ONE>
// At most two waves per SIMD ever share a compute unit with this kernel (LDS holds one
// eight-wave workgroup), so it may use up to 256 VGPRs per lane.
__global__ __attribute__((amdgpu_flat_work_group_size(512, 512), amdgpu_waves_per_eu(2, 2)))
void decode_mfma_kernel(const int32_t* seq_len, const void* params_k, const void* params_v,
                        const void* q, int n_splits, int n_kv_heads, int batch, uint32_t shape,
                        const DecodeArgs a) {
  constexpr int NW = 8;               // waves per workgroup
  constexpr int NTHR = 64 * NW;       // threads per workgroup
  constexpr int NH = 4 * NT;          // head slots: 4 per column tile
  constexpr int TW = 16 * NTILE;      // tokens per wave
  constexpr int S = NW * TW;          // tokens per chunk
  constexpr int NCH = S / 64;         // 64-token blocks per chunk
  constexpr int CPW = NTILE / 4;      // blocks per wave
  // With factors up to 2^7 in the bytes the weights of d = 7 keep 23 bits below the head's largest,
  // and tokens far outside the calibration's distribution, whose scale times that largest weight is
  // many times their score, lose precision: up to 6.6e-5 of an output.  FINE (27 bits, 6e-6) for
  // the shapes that had fp32 scores before they came here, at most 9e-6: records over 64 bytes, and
  // more than eight heads, which without an append share the instances of the fewer (a segmented
  // step 29.3 -> 29.6 us).  The others never had more: one instruction per dword there took 4 x
  // 131072 tokens from 85.6 to 87.1 us.
  constexpr bool FINE = NP > 4 || !APPEND;
  constexpr int DM = FINE ? 3 : 7;    // the factor of bit d: 2^(d & DM)
  // The cache streams straight into LDS.  For the first chunk the upper half of the waves
  // issues the transfers; the lower half builds the query planes meanwhile (a wave whose
  // loads wait for queue space can do nothing else).
  constexpr int NWC = NW / 2;               // waves that build the query planes
  constexpr int NTC = 64 * NWC;             // their threads
  constexpr int NJQ = NTC / 32;       // row blocks of the query transform
  constexpr int RJ = kD / NJQ;        // rows per block
  constexpr int NR = NH * kD / NTHR;  // (head, channel) items per thread
  constexpr int NRC = NH * kD / NTC;  // the same per plane-building thread
  constexpr int NPI = (NH * 4 * NP * 8 + NTC - 1) / NTC;    // plane items per thread
  static_assert(NTILE % 4 == 0, "a wave owns whole 64-token blocks (and tile pairs)");
  static_assert(kMaxNH * (kD / 4) <= NTHR, "the merge takes one (head, 4 columns) slot per thread");
  static_assert(NR >= 1 && NCH % 2 == 0, "thread mapping");
  extern __shared__ __align__(16) uint8_t smem[];
  __shared__ unsigned qmx[NH];
  __shared__ int fexp_s[NH];
  __shared__ float wmax[NW][NH], wsum[NW][NH], wpa[NW][NH];
  __shared__ float mfin[NH];
  __shared__ float chs[NH];           // midrise: the half-step term of each head's scores
  __shared__ float wpav[NW][NH];      // sum of P alpha^V per wave and head
  __shared__ unsigned csync;          // arrivals of the plane-building waves
  __shared__ int hdr_s[6];            // V budget, widest V code, V and K quantizer, record bytes

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 15, g = lane >> 4, hc = n >> 2, L = n & 3;
  // The scalar arguments arrive in registers with the wave (kernel argument preloading); the
  // first loads need nothing else.  `shape`: query heads
  // per KV head (bits 0-7), their groups (8-15), evenly dealt (16), bf16 queries (17).
  const int all_heads = (int)(shape & 0xff), hg = (int)((shape >> 8) & 0xff);
  const bool even = ONE || (shape & 0x10000u) != 0, q_bf = (shape & 0x20000u) != 0;
  // The workgroup's row (sequence, KV head, group of NH query heads), its run of `per`
  // chunks and the row's number of runs.  Evenly dealt: every row has the same number of
  // workgroups (known without a load).  Otherwise by the lengths (assign_runs).
  int vrow, split, ns, per, len_raw;
  if (even) {
    // XCD-aware order (grid a multiple of 8): workgroups are dealt to the 8 XCDs round robin,
    // so consecutive runs of a (sequence, KV head) are given block ids that land on one XCD.
    const int nb8 = (int)(gridDim.x >> 3);
    const int lb = (gridDim.x & 7) ? (int)blockIdx.x
                                   : (int)(blockIdx.x & 7) * nb8 + (int)(blockIdx.x >> 3);
    vrow = lb / n_splits;                            // (32-bit: rows x splits < 2^30)
    split = lb - vrow * n_splits;
    // (one sequence: known without a division)
    len_raw = seq_len[batch == 1 ? 0 : vrow / (n_kv_heads * hg)];   // gates the cache loads
  } else {
    if (!assign_runs<S, APPEND>(seq_len, a.cap, batch, n_kv_heads * hg, vrow, split, ns, per, len_raw))
      return;
  }
  __builtin_amdgcn_sched_barrier(0);
  const int row32 = hg == 1 ? vrow : vrow / hg, hgi = vrow - row32 * hg;
  const int seq = batch == 1 ? 0 : row32 / n_kv_heads, kvh = row32 - seq * n_kv_heads;
  const int64_t row = row32;
  const int RK = a.rk, RV = a.rv;
  const int G = min(NH, all_heads - NH * hgi);        // query heads of this workgroup
  const int RWK = RK >> 2;
  const HeadParams* hk = head_params(params_k, kvh);
  const HeadParams* hv = head_params(params_v, kvh);

  // (0) Loads that need nothing, by the plane-building threads (tc < NTC): T_K rows
  //     RJ jq .. RJ jq + RJ - 1 at columns 4 c4 .. + 3, the bit descriptors, the queries, and
  //     (fused append) their share of the new token's transform.  Loads are unconditional
  //     (clamped indices or empty descriptors), so the wait counters stay exact.
  const bool cw = wave < NWC;                         // builds the query planes (per wave)
  // The query transform: lane l of plane-building wave w holds T_K rows RJ jq .. + RJ - 1
  // (row block jq = l / 8) at columns 4 c4 .. + 3 (c4 = 8 w + l % 8), so the sums over the
  // row blocks stay inside the wave.
  static_assert(NJQ == 8 && RJ == 16 && NWC == 4, "query transform mapping");
  const int jq = lane >> 3, c4 = 8 * (wave % NWC) + (lane & 7), cq = tid & (kD - 1);
  constexpr int NVL = NH / 2;                   // q~ values a lane ends with
  // Scale and width of the lane's channels 4 c4 + (NVL jq + i) % 4 (head (NVL jq + i) / 4).
  float ksq[NVL];
  int kbq[NVL];
  float khs[2];                       // key half steps of channels lane and lane + 64
  // The channel tables, used only after the last value phase and loaded at its start.  In the
  // front they would queue behind the cache stream, and the wait before the join would then
  // cover them.  Values that steer uniform code come from a plane-building wave through LDS
  // (a scalar load would hold up every LDS wait until it returns).
  int vbc = 0, voc = 0;
  float vsc = 0.f, vhs = 0.f;
  // Fused append: waves 0 and 1 encode the key and the value token, lane l channels l and
  // l + 64 (their widths, first bits and scales).
  int e_b[2] = {0, 0}, e_off[2] = {0, 0};
  float e_s[2] = {0.f, 0.f};
  auto load_tables = [&]() {
    if (APPEND && wave < 2) {
      const HeadParams* eh = wave == 0 ? hk : hv;
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        e_b[i] = eh->bits[lane + 64 * i];
        e_off[i] = eh->bit_off[lane + 64 * i];
        e_s[i] = eh->s[lane + 64 * i];
      }
    }
    vbc = hv->bits[cq];
    voc = hv->bit_off[cq];
    vsc = hv->s[cq];
    vhs = hv->half_step[cq];
  };
  int hdr = 0;                        // wave 0, lanes 0..5: the fields of hdr_s
  v4f tr[RJ];
  uint2 desc[NPI];
  uint32_t qraw[NRC];
  bool qhi[NRC];
  // Fused append: dot products d = split + ns k, k = wave + NWC i, of the 2 x 128 (key
  // channels, then value channels); the first two of each plane-building wave are fetched
  // up front (the token's two elements of this lane and the matching two of column d % kD of
  // Tq), further ones (fewer than 32 runs) are formed by the transfer waves, one per lane.
  const int x_eb = a.x_dtype == AATC_BF16 ? 2 : 4;
  constexpr int KF = 2;                               // coefficients fetched up front
  int adk[KF];
  uint32_t ax[KF][2];
  int atq[KF][2];
  float a_inv_s[KF];
  auto front_loads = [&]() {
#pragma unroll
    for (int i = 0; i < NVL; ++i) {
      const int c = 4 * c4 + ((NVL * jq + i) & 3);
      ksq[i] = hk->s[c];
      kbq[i] = hk->bits[c];
    }
#pragma unroll
    for (int jj = 0; jj < RJ; ++jj)
      tr[jj] = reinterpret_cast<const v4f*>(hk->T)[(RJ * jq + jj) * (kD / 4) + c4];
    khs[0] = hk->half_step[lane];
    khs[1] = hk->half_step[lane + 64];
    if (wave == 0 && lane < 6) {
      const int32_t* f = lane == 0 ? &hv->budget : lane == 1 ? &hv->max_bits
                       : lane == 2 ? &hv->quantizer : lane == 3 ? &hk->quantizer
                       : lane == 4 ? &hk->record_bytes : &hv->record_bytes;
      hdr = *f;
    }
    // Plane items (head, record dword D, bit d of each byte): the 4 record bits 32 D +
    // 8 j + d, j = 0..3, of one head.
#pragma unroll
    for (int r = 0; r < NPI; ++r) {
      const int dd = (r * NTC + tid) % (8 * RWK);                // < 8 RWK: in the table
      desc[r] = reinterpret_cast<const uint2*>(hk->bit_desc)[dd];
    }
    // Queries, element r NTC + tid, read as the aligned dword that holds the element
    // (either type, no branch; the dword never leaves the element's page).
    const int64_t qb = ((int64_t)row * all_heads + NH * hgi) * kD;
#pragma unroll
    for (int r = 0; r < NRC; ++r) {
      const int64_t i = qb + min(r * NTC + tid, G * kD - 1);
      const uintptr_t ad = reinterpret_cast<uintptr_t>(q) + (q_bf ? 2 * i : 4 * i);
      qraw[r] = *reinterpret_cast<gdword>(ad & ~(uintptr_t)3);
      qhi[r] = (ad & 2) != 0;
    }
  };
  auto front_coefficients = [&]() {
    if constexpr (APPEND) {
#pragma unroll
      for (int f = 0; f < KF; ++f) {
        const int d = split + ns * (wave + NWC * f);
        adk[f] = d;
        const bool on = d < 2 * kD;
        const HeadParams* eh = d >= kD ? hv : hk;
        const int ac = d & (kD - 1);
        const __amdgpu_buffer_rsrc_t xrs =
            make_rsrc(static_cast<const uint8_t*>(d >= kD ? a.x_v : a.x_k) + row * kD * x_eb,
                      on ? (uint32_t)(kD * x_eb) : 0u);
        const __amdgpu_buffer_rsrc_t trs = make_rsrc(eh->Tqt + ac * kD, on ? 4u * kD : 0u);
        ax[f][0] = __builtin_amdgcn_raw_buffer_load_b32(xrs, (lane * x_eb) & ~3, 0, 0);
        ax[f][1] = __builtin_amdgcn_raw_buffer_load_b32(xrs, ((lane + 64) * x_eb) & ~3, 0, 0);
        atq[f][0] = (int)__builtin_amdgcn_raw_buffer_load_b32(trs, 4 * lane, 0, 0);
        atq[f][1] = (int)__builtin_amdgcn_raw_buffer_load_b32(trs, 4 * (lane + 64), 0, 0);
        a_inv_s[f] = eh->inv_s[ac];
      }
    }
  };

  // The loads that do not need the length go out before its round trip.
  if (cw) front_loads();
  __builtin_amdgcn_sched_barrier(0);
  const int len = (int)min<int64_t>(max(len_raw, 0), a.cap);
  // With a fused append the chunks stop short of the new token at len - 1; the merging
  // workgroup encodes it and adds it to the merge.
  const int len_c = max(0, APPEND ? len - 1 : len);
  const int nchunk = (len_c + S - 1) / S;
  if (even) {
    // runs of the row (the other workgroups exit)
    per = 1;
    ns = max(1, nchunk);
    if (!ONE && nchunk > n_splits) {
      per = (nchunk + n_splits - 1) / n_splits;
      ns = (nchunk + per - 1) / per;
    }
  }
  // (1) The run's packed cache (loads past the capacity read 0).
  const __amdgpu_buffer_rsrc_t krs = make_rsrc(a.k_codes + row * a.cap * RK, (uint32_t)(a.cap * RK));
  const __amdgpu_buffer_rsrc_t vrs = make_rsrc(a.v_codes + row * a.cap * RV, (uint32_t)(a.cap * RV));
  const __amdgpu_buffer_rsrc_t akrs = make_rsrc(a.k_alpha + row * a.cap, (uint32_t)(a.cap * 2));
  const __amdgpu_buffer_rsrc_t avrs = make_rsrc(a.v_alpha + row * a.cap, (uint32_t)(a.cap * 2));
  uint8_t* kbuf = smem;
  uint8_t* vbuf = smem + a.off_v;
  uint16_t* akb = reinterpret_cast<uint16_t*>(smem + a.off_ak);
  uint16_t* avb = reinterpret_cast<uint16_t*>(smem + a.off_av);
  // 1 KiB transfers straight into LDS (lane l's 16 bytes at 16 l): the key records and the
  // token scales of chunk c, or its value tiles, dealt to waves w0, w0 + 1, .. (nw of them)
  // round robin; each returns this wave's count.  Only whole 1 KiB blocks of the regions are
  // written (their sizes are 1 KiB multiples).  No branch on the chunk's contents: an empty
  // chunk computes on masked tokens.
  auto chunk_load = [&](int c) {                      // tokens of chunk c, whole tiles
    return min(S, (max(0, len_c - c * S) + kTile - 1) / kTile * kTile);
  };
  auto issue_keys = [&](int c, int wd, int nw) {
    const int t0 = c * S, nl = chunk_load(c);
    const int nki = (nl * RK + 1023) >> 10, nai = (2 * nl + 1023) >> 10;
    int cnt = 0;
    for (int j = wd; j < nki; j += nw) {
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          krs, (__attribute__((address_space(3))) void*)(kbuf + 1024 * j), 16,
          t0 * RK + 1024 * j + 16 * lane, 0, 0, 0);
      ++cnt;
    }
    for (int j = wd; j < nai; j += nw) {
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          akrs, (__attribute__((address_space(3))) void*)((uint8_t*)akb + 1024 * j), 16,
          2 * t0 + 1024 * j + 16 * lane, 0, 0, 0);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          avrs, (__attribute__((address_space(3))) void*)((uint8_t*)avb + 1024 * j), 16,
          2 * t0 + 1024 * j + 16 * lane, 0, 0, 0);
      cnt += 2;
    }
    return cnt;
  };
  auto issue_values = [&](int c, int wd, int nw) {
    const int t0 = c * S, nvi = (chunk_load(c) * RV + 1023) >> 10;
    int cnt = 0;
    for (int j = wd; j < nvi; j += nw) {
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          vrs, (__attribute__((address_space(3))) void*)(vbuf + 1024 * j), 16,
          t0 * RV + 1024 * j + 16 * lane, 0, 0, 0);
      ++cnt;
    }
    return cnt;
  };
  // Records that do not match the parameters store a NaN maximum (the value budget is
  // clamped to the record so LDS accesses stay in range).
  Partial* parts = a.partials + (row * all_heads + NH * hgi) * a.max_splits;
  float* out_rows = a.out + (row * all_heads + NH * hgi) * kD;
  const __amdgpu_buffer_rsrc_t prs = make_rsrc(parts, (uint32_t)(ns * G * sizeof(Partial)));

  // (2) Query planes, by the plane-building waves; they synchronize among themselves
  //     (the other waves are busy issuing the cache) through an LDS arrival count.
  unsigned csync_target = 0u;
  auto plane_sync = [&]() {
    csync_target += NWC;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    if (lane == 0) __hip_atomic_fetch_add(&csync, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    while (__hip_atomic_load(&csync, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) < csync_target)
      __builtin_amdgcn_s_sleep(1);
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
  };
  // The channel weights (kept for the fused append's score); the queries as scratch over
  // the value operands (written only after the planes).
  float* qcl = reinterpret_cast<float*>(smem + a.off_qc);              // [NH][kD]
  float* qs = reinterpret_cast<float*>(smem + a.off_pb);               // [NH][kD]
  uint8_t* ql = smem + a.off_ql;                     // [4][NH][2 NP][64]
  float rcf[KF] = {0.f, 0.f};                        // fused append: this wave's coefficients
  float reh[KF] = {0.f, 0.f};                        // and the token's error bounds
  auto build_planes = [&]() {
#pragma unroll
    for (int r = 0; r < NRC; ++r) {
      const uint32_t w = qraw[r];
      const float qv = q_bf ? __uint_as_float((qhi[r] ? (w >> 16) : (w & 0xffffu)) << 16)
                            : __uint_as_float(w);
      qs[r * NTC + tid] = ((r * NTC + tid) / kD < G) ? qv : 0.f;
    }
    plane_sync();                                    // qs, qmx
    // q~ = T_K^T q: RJ-row partial sums per lane, then over the wave's 8 row blocks
    // (reduce-scatter across lane bits 3..5): lane l ends with value NVL jq + i of the 4 NH
    // (head, column) sums of its column quad.
    {
      v4f acc[NH];
#pragma unroll
      for (int h = 0; h < NH; ++h) acc[h] = (v4f){0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int jj = 0; jj < RJ; jj += 4)
#pragma unroll
        for (int h = 0; h < NH; ++h) {
          const v4f qv = *reinterpret_cast<const v4f*>(qs + h * kD + RJ * jq + jj);
          acc[h] += tr[jj] * qv.x + tr[jj + 1] * qv.y + tr[jj + 2] * qv.z + tr[jj + 3] * qv.w;
        }
      float v0[4 * NH], v1[2 * NH], v2[NH], v3[NVL];
#pragma unroll
      for (int h = 0; h < NH; ++h) {
        v0[4 * h] = acc[h].x;
        v0[4 * h + 1] = acc[h].y;
        v0[4 * h + 2] = acc[h].z;
        v0[4 * h + 3] = acc[h].w;
      }
      reduce_scatter_step<4 * NH, 32>(v0, v1);
      reduce_scatter_step<2 * NH, 16>(v1, v2);
      reduce_scatter_step<NH, 8>(v2, v3);
      // Channel weight Q_c = q~_c s_c scale log2(e) (the weight of the code's sign bit up
      // to sign), kept in LDS; the largest |Q_c| of a head sets its fixed-point exponent.
      const int hl = (NVL * jq) >> 2;                // the lane's head
      float mloc = 0.f;
#pragma unroll
      for (int i = 0; i < NVL; ++i) {
        const int c = 4 * c4 + ((NVL * jq + i) & 3);
        const float qc = (hl < G && kbq[i] > 0) ? v3[i] * ksq[i] * a.scale_log2e : 0.f;
        qcl[hl * kD + c] = qc;
        mloc = fmaxf(mloc, fabsf(qc));
      }
      // Over the lanes that hold head hl: lane bits 0..2, and bit 3 when NH = 4.
      mloc = fmaxf(mloc, dpp_f<0xB1>(mloc));         // quad_perm [1,0,3,2]
      mloc = fmaxf(mloc, dpp_f<0x4E>(mloc));         // quad_perm [2,3,0,1]
      mloc = fmaxf(mloc, dpp_f<0x141>(mloc));        // row_half_mirror
      if constexpr (NH == 4) mloc = fmaxf(mloc, dpp_f<0x128>(mloc));   // row_ror:8
      if ((lane & (NH == 4 ? 15 : 7)) == 0) atomicMax(&qmx[hl], __float_as_uint(mloc));
    }
    plane_sync();                                    // qcl, qmx
    // Midrise: every score has the term alpha^K C_h with C_h = sum_c Q_c 2^(-b_c) over the
    // stored channels (the half step of each level); 0 for the midtread reading.
    for (int h = wave % NWC; h < NH; h += NWC) {
      const float cp = wave_sum_dpp(qcl[h * kD + lane] * khs[0] + qcl[h * kD + lane + 64] * khs[1]);
      if (lane == 0) chs[h] = cp;
    }
    if (tid < NH) {
      int e = 0;
      frexpf(__uint_as_float(qmx[tid]), &e);
      fexp_s[tid] = qmx[tid] ? 30 - e : 0;
    }
    // Record bit v = 32 D + 8 j + d  ->  K-step 2 (D % NP) + d / 4, lane group D / NP,
    // byte 4 (d % 4) + j of the 16-byte operand; dwords RWK .. 4 NP - 1 get weight 0.
    // Weight 2^(k + 1 - b) Q_c / 2^(d & DM), negated for the sign bit and for a factor of 2^7 (int8
    // 0x80 = -128); the four limbs of the four bits j = 0..3 are transposed into one dword per
    // limb plane.
    for (int i = tid; i < 4 * NH * 2 * 4 * (4 * NP - RWK); i += NTC) {
      const int D = RWK + i / (4 * NH * 2 * 4), rest = i % (4 * NH * 2 * 4);
      const int plane = rest / 8, st = 2 * (D % NP) + ((rest >> 2) & 1);
      *reinterpret_cast<uint32_t*>(ql + (plane * 2 * NP + st) * 64 + ((D / NP) << 4) +
                                   4 * (rest & 3)) = 0u;
    }
    // Items without branches or divisions, all channel-weight reads issued together:
    // the fixed-point exponent of every head first, then every item's four weights.
    const int nbh = 8 * RWK;                         // items per head
    int fe_h[NH];
#pragma unroll
    for (int h = 0; h < NH; ++h) {
      int e = 0;
      const unsigned qm = qmx[h];
      frexpf(__uint_as_float(qm), &e);
      fe_h[h] = qm ? 30 - e : 0;
    }
    int hi_[NPI], dd_[NPI];
    float qv_[NPI][4];
#pragma unroll
    for (int r = 0; r < NPI; ++r) {
      const int i = r * NTC + tid;
      int h = 0;
#pragma unroll
      for (int hh = 1; hh < NH; ++hh) h += (i >= hh * nbh) ? 1 : 0;
      hi_[r] = h;
      dd_[r] = i - h * nbh;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const uint32_t ent = ((j < 2 ? desc[r].x : desc[r].y) >> (16 * (j & 1))) & 0xffffu;
        qv_[r][j] = qcl[h * kD + (ent & 127)];
      }
    }
#pragma unroll
    for (int r = 0; r < NPI; ++r) {
      const int i = r * NTC + tid, h = hi_[r], D = dd_[r] >> 3, d = dd_[r] & 7;
      int fe = fe_h[0];
#pragma unroll
      for (int hh = 1; hh < NH; ++hh) fe = (h == hh) ? fe_h[hh] : fe;
      uint32_t x[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const uint32_t ent = ((j < 2 ? desc[r].x : desc[r].y) >> (16 * (j & 1))) & 0xffffu;
        int fx = (int)rintf(ldexpf(qv_[r][j], (int)((ent >> 8) & 15) - kDescBias + fe - (d & DM)));
        if ((((ent >> 14) & 1) != 0) != ((d & DM) == 7)) fx = -fx;
        x[j] = (ent & 0x8000u) ? pack_limbs(fx) : 0u;
      }
      // x[j] = (limb 0..3 of bit j)  ->  y[L] = (limb L of bits 0..3)
      const uint32_t t0 = __builtin_amdgcn_perm(x[1], x[0], 0x05010400u);
      const uint32_t t1 = __builtin_amdgcn_perm(x[3], x[2], 0x05010400u);
      const uint32_t t2 = __builtin_amdgcn_perm(x[1], x[0], 0x07030602u);
      const uint32_t t3 = __builtin_amdgcn_perm(x[3], x[2], 0x07030602u);
      const uint32_t y[4] = {__builtin_amdgcn_perm(t1, t0, 0x05040100u),
                             __builtin_amdgcn_perm(t1, t0, 0x07060302u),
                             __builtin_amdgcn_perm(t3, t2, 0x05040100u),
                             __builtin_amdgcn_perm(t3, t2, 0x07060302u)};
      const int st = 2 * (D % NP) + (d >> 2);
      const int pos = ((D / NP) << 4) + ((d & 3) << 2);
      // Items past the last head's go to the consumed queries instead.
      const bool ok = i < G * nbh;
#pragma unroll
      for (int l4 = 0; l4 < 4; ++l4) {
        uint8_t* dst = ok ? ql + ((l4 * NH + h) * 2 * NP + st) * 64 + pos
                          : reinterpret_cast<uint8_t*>(qs) + 16 * (tid & 63) + 4 * l4;
        *reinterpret_cast<uint32_t*>(dst) = y[l4];
      }
    }
    // Fused append: this wave's coefficients (stored after the value phase, when no
    // cache transfer is queued ahead of the stores).
    if constexpr (APPEND)
      append_coefficients<KF>(ax, atq, a.x_dtype, a_inv_s, rcf, reh);  // (past 2 kD: unused)
  };

  // Fused append with fewer than 32 runs: the coefficients that the plane-building waves do
  // not cover (k = NWC KF, ..), one per lane of the last transfer wave, or of the last two for
  // fewer than four runs (and two per lane for one run): exact integer sums over the lane's column
  // of Tq, with the tokens' integers in LDS.  These waves issue no cache transfers, behind which
  // their loads would wait: dealt over all four they held up the join until the value tiles were in
  // (20000 tokens, 8 KV heads, capacity 32768: 18.5 us, 15.7 now; 8192 of 8192: 16.3, 13.7).  (One coefficient
  // per wave at a time took 40 us for a row of one run: a round trip and a wave reduction each.)
  const int n_tail = !APPEND || ns * NWC * KF >= 2 * kD ? 0 : ns >= 4 ? 1 : 2;   // tail waves
  const bool tail_wave = wave >= NW - n_tail;
  const int tail_rounds = ns == 1 ? 2 : 1;
  float r_tail[2] = {0.f, 0.f}, eh_tail[2] = {0.f, 0.f};
  auto tail_dot = [&](int r) {                       // (2 kD and more: none)
    return split + ns * (NWC * KF + 64 * (NW - 1 - wave + n_tail * r) + lane);
  };
  auto tail_coefficients = [&]() {
    int* xi = reinterpret_cast<int*>(smem + a.off_es);   // [2][kD] (the merge's scratch later)
    int shift[2];
    float eh[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const uint8_t* xr = static_cast<const uint8_t*>(t ? a.x_v : a.x_k) + row * kD * x_eb;
      const float xa = load_elem(xr, a.x_dtype, lane), xb = load_elem(xr, a.x_dtype, lane + 64);
      shift[t] = token_shift(wave_max_dpp(fmaxf(fabsf(xa), fabsf(xb))));
      const float va = ldexpf(xa, shift[t]), vb = ldexpf(xb, shift[t]);
      const float ra = rintf(va), rb = rintf(vb);
      const float E = wave_sum_dpp(fabsf(va - ra) + fabsf(vb - rb));
      eh[t] = shift[t] < 0 ? INFINITY : ldexpf(E * (1.f + 0x1p-16f), -shift[t]);
      xi[t * kD + lane] = (int)ra;                   // (every tail wave writes the same values)
      xi[t * kD + lane + 64] = (int)rb;
    }
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      if (r >= tail_rounds) break;                   // (uniform)
      const int d = tail_dot(r);
      const bool tv = (d & kD) != 0;                 // value channel (past 2 kD: unused)
      const HeadParams* eh_p = tv ? hv : hk;
      const int c = d & (kD - 1);
      const int4* tc = reinterpret_cast<const int4*>(eh_p->Tqt + c * kD);
      const int4* xq = reinterpret_cast<const int4*>(xi + (tv ? kD : 0));
      const float isv = eh_p->inv_s[c];
      long long H = 0;
#pragma unroll
      for (int jb = 0; jb < kD / 4; jb += 16) {
        int4 t4[16];
#pragma unroll
        for (int q = 0; q < 16; ++q) t4[q] = tc[jb + q];
#pragma unroll
        for (int q = 0; q < 16; ++q) {
          const int4 x4 = xq[jb + q];
          H += (long long)x4.x * t4[q].x;
          H += (long long)x4.y * t4[q].y;
          H += (long long)x4.z * t4[q].z;
          H += (long long)x4.w * t4[q].w;
        }
      }
      r_tail[r] = integer_result((double)H, tv ? shift[1] : shift[0]) * isv;
      eh_tail[r] = tv ? eh[1] : eh[0];
    }
  };

  // (3) Front.  The plane-building and the issuing waves take separate arms up to the
  //     barrier where the key records and scales have landed; the value tiles keep landing
  //     through the key phase.  The barriers are plain s_barrier after explicit waits:
  //     __syncthreads() would make the issuing waves wait for all of their transfers.  The
  //     explicit vmcnt(0) waits cost nothing (no load of the wave is in flight there) but
  //     tell the compiler so: with the two arms merged, it would otherwise take the other
  //     arm's loads as pending and wait on them later with counts that also cover the cache
  //     transfers.
  const int c0 = split * per, c1 = min(c0 + per, nchunk);   // (an empty row runs one empty chunk)
  if (split >= ns) return;                           // (whole workgroup, before any barrier)
  if (cw) {
    front_coefficients();
    if (tid < NH) qmx[tid] = 0u;
    if (tid == 0) csync = 0u;
    __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
    plain_barrier();                                 // the small loads are queued first
    build_planes();
    if (wave == 0 && lane < 6) hdr_s[lane] = hdr;
    __builtin_amdgcn_s_waitcnt(kWaitVm0);
  } else {
    plain_barrier();
    __builtin_amdgcn_s_waitcnt(kWaitVm0);
    if (APPEND && tail_wave) {
      tail_coefficients();
    } else {
      issue_keys(c0, wave - NWC, NW - NWC - n_tail);
      wait_vmcnt(issue_values(c0, wave - NWC, NW - NWC - n_tail));   // key records and scales landed
    }
  }
  __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
  plain_barrier();
  const int v_budget = __builtin_amdgcn_readfirstlane(hdr_s[0]);
  float sfx[NT], chk[NT];
#pragma unroll
  for (int rt = 0; rt < NT; ++rt) {
    sfx[rt] = ldexpf(1.f, -fexp_s[4 * rt + g]);   // (the head of this lane's scores)
    chk[rt] = chs[4 * rt + g];
  }
  // The value phase's constants.  Value-bit tiles of 16 bits are dealt to the waves round
  // robin; the chunk's 64-token blocks go in two halves: waves 0-3 take the first half of
  // every tile, waves 4-7 the second (each reads only its half's P operands), and the two
  // groups walk the tiles in opposite orders, so that the two waves of a SIMD (s and s + 4)
  // have the same number of tiles between them on every SIMD.
  const int BV = min(v_budget, 8 * RV);
  const int NVT = (BV + 15) >> 4;
  const uint32_t m0 = 0x01010101u << (2 * g), m1 = m0 << 1;
  constexpr int NCW = NCH / 2;                        // blocks of a wave's tile pass
  constexpr int NWT = NW / 2;                         // waves over the tiles of one half
  const int hf = wave >> 2;                           // this wave's half of the blocks
  const int wj = hf ? 3 - (wave & 3) : (wave & 3);    // its first tile
  v4i* pb = reinterpret_cast<v4i*>(smem + a.off_pb);  // [NCH][NT][64] value operands
  const v4i* pbh = pb + hf * NCW * NT * 64;
  // LDS address of this lane's value-bit dword pair in each block of the half for tile
  // vt = wj; tile wj + NWT it is 128 NWT it bytes further (an immediate offset: no address
  // arithmetic in the loop).
  uint32_t vaddr[NCW];
  {
    const uint32_t vb = (uint32_t)reinterpret_cast<uintptr_t>(
        (__attribute__((address_space(3))) uint8_t*)vbuf) + 8 * n + 128 * wj;
#pragma unroll
    for (int ch = 0; ch < NCW; ++ch) {
      vaddr[ch] = vb + (hf * NCW + ch) * kTile * RV;
      asm volatile("" : "+v"(vaddr[ch]));          // computed once, not per tile
    }
  }
  // Records of at most 64 bytes (NP <= 4) have up to 32 tiles, wider ones up to 64.
  constexpr int kMaxIt = (NP <= 4 ? 32 : 64) / NWT;
  // Running state of the run: the maximum per head, and per lane the sums of P and P alpha^V
  // (of its tokens) and the value sums of its bits (value bit 16 vt + n of head 4 rt + g), all
  // relative to that maximum.
  float mrun[NT], lrun[NT], parun[NT], oacc[kMaxIt][NT];
#pragma unroll
  for (int rt = 0; rt < NT; ++rt) {
    mrun[rt] = -INFINITY;
    lrun[rt] = parun[rt] = 0.f;
#pragma unroll
    for (int it = 0; it < kMaxIt; ++it) oacc[it][rt] = 0.f;
  }
  const uint32_t sel_a = (L & 2) ? 0x03020706u : 0x05040100u;
  const uint32_t sel_b = (L & 1) ? 0x03070105u : 0x06020400u;
  const int wb = wave * TW;

  for (int c = c0;; ++c) {
  const int nt = max(0, min(S, len_c - c * S));
  const bool more = !ONE && c + 1 < c1;
  // (4) Key scores of this wave's tokens.  The query planes are the A operand (row 4 h + L:
  //     head h, limb L) and the record bits the B operand (column: token), so lane 16 h + n
  //     ends with the four limb sums of head h for token n of the tile and recombines them
  //     itself.
  float zr[NTILE][NT];
  float avt[NTILE];
  float lav[NTILE];                      // log2 alpha^V (-inf for 0 and past the tokens)
  auto scores = [&]() {
  // The query planes, every tile's record dwords and the token scales first (one LDS round
  // trip), then the products; lane group g holds record dwords g NP .. g NP + NP - 1, and
  // dwords past the record (they belong to the next token) meet zero query weights.
  v4i bq[NT][2 * NP];
#pragma unroll
  for (int rt = 0; rt < NT; ++rt)
#pragma unroll
    for (int s = 0; s < 2 * NP; ++s)
      bq[rt][s] = *reinterpret_cast<const v4i*>(ql + ((L * NH + 4 * rt + hc) * 2 * NP + s) * 64 + 16 * g);
  uint32_t wda[NTILE][NP];
  uint16_t aka[NTILE], ava[NTILE];
#pragma unroll
  for (int tt = 0; tt < NTILE; ++tt) {
    const uint8_t* rec = kbuf + (wb + 16 * tt + n) * RK;
#pragma unroll
    for (int P = 0; P < NP; ++P) wda[tt][P] = *reinterpret_cast<const uint32_t*>(rec + 4 * (g * NP + P));
    aka[tt] = akb[wb + 16 * tt + n];
    ava[tt] = avb[wb + 16 * tt + n];
  }
  __builtin_amdgcn_sched_barrier(0);
  // Tiles go in pairs: two independent MFMA chains interleave.
#pragma unroll
  for (int tp = 0; tp < NTILE; tp += 2) {
    v4i acc[2][NT];
    uint32_t wd[2][NP];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
#pragma unroll
      for (int P = 0; P < NP; ++P) wd[u][P] = wda[tp + u][P];
#pragma unroll
      for (int rt = 0; rt < NT; ++rt) acc[u][rt] = (v4i){0, 0, 0, 0};
    }
#pragma unroll
    for (int P = 0; P < NP; ++P) {
      v4i a0[2], a1[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const uint32_t w = wd[u][P];
        a0[u] = (v4i){(int)(w & 0x01010101u), (int)(w & 0x02020202u), (int)(w & 0x04040404u),
                      (int)(w & 0x08080808u)};
        const uint32_t v = FINE ? w >> 4 : w, m = FINE ? 0x01010101u : 0x10101010u;
        a1[u] = (v4i){(int)(v & m), (int)(v & (m << 1)), (int)(v & (m << 2)), (int)(v & (m << 3))};
      }
#pragma unroll
      for (int rt = 0; rt < NT; ++rt)
#pragma unroll
        for (int u = 0; u < 2; ++u) acc[u][rt] = mfma_i8(bq[rt][2 * P], a0[u], acc[u][rt]);
#pragma unroll
      for (int rt = 0; rt < NT; ++rt)
#pragma unroll
        for (int u = 0; u < 2; ++u) acc[u][rt] = mfma_i8(bq[rt][2 * P + 1], a1[u], acc[u][rt]);
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int tt = tp + u;
      const int tok = wb + 16 * tt + n;
      const bool tok_ok = tok < nt;
      const float ak = half_bits_to_float(aka[tt]);
      const float av = half_bits_to_float(ava[tt]);
      avt[tt] = tok_ok ? av : 0.f;
      lav[tt] = avt[tt] > 0.f ? __builtin_amdgcn_logf(avt[tt]) : -INFINITY;
#pragma unroll
      for (int rt = 0; rt < NT; ++rt) {
        const v4i d = acc[u][rt];                 // limbs 0..3 (weights 256^i)
        float f = fmaf((float)d[3], 256.f, (float)d[2]);
        f = fmaf(f, 256.f, (float)d[1]);
        f = fmaf(f, 256.f, (float)d[0]);
        zr[tt][rt] = (tok_ok && 4 * rt + g < G) ? fmaf(f, sfx[rt], chk[rt]) * ak : -INFINITY;
      }
    }
  }
  };
  // (a short context in a chunk of its own: the waves past its end have no scores to form, and the
  // second half's waves below no values; 200 tokens, 8 KV heads, capacity 32768: 18.0 -> 16.6 us)
  if (!ONE || wb < nt) {
    scores();
  } else {
#pragma unroll
    for (int tt = 0; tt < NTILE; ++tt) {
      avt[tt] = 0.f;
      lav[tt] = -INFINITY;
#pragma unroll
      for (int rt = 0; rt < NT; ++rt) zr[tt][rt] = -INFINITY;
    }
  }

  // (5) Softmax: one maximum per head over the run so far, and one fixed-point exponent per
  //     head for the chunk's P alpha^V from its largest value, max_i 2^(z_i - m) alpha^V_i =
  //     2^(max_i (z_i + log2 alpha^V_i) - m) (both maxima in one reduction).
#pragma unroll
  for (int rt = 0; rt < NT; ++rt) {
    float m = -INFINITY, m2 = -INFINITY;
#pragma unroll
    for (int tt = 0; tt < NTILE; ++tt) {
      m = fmaxf(m, zr[tt][rt]);
      m2 = fmaxf(m2, zr[tt][rt] + lav[tt]);
    }
    m = row16_max(m);
    m2 = row16_max(m2);
    if (n == 0) {
      wmax[wave][4 * rt + g] = m;
      wpa[wave][4 * rt + g] = m2;
    }
  }
  __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
  plain_barrier();                       // maxima in; every key record and scale of the chunk read
  int nk_mine = 0;
  if (more) nk_mine = issue_keys(c + 1, wave, NW);
  float mh[NT], sa[NT];
  int fvh[NT];
#pragma unroll
  for (int rt = 0; rt < NT; ++rt) {
    float m = wmax[0][4 * rt + g], m2 = wpa[0][4 * rt + g];
#pragma unroll
    for (int w = 1; w < NW; ++w) {
      m = fmaxf(m, wmax[w][4 * rt + g]);
      m2 = fmaxf(m2, wpa[w][4 * rt + g]);
    }
    mh[rt] = fmaxf(mrun[rt], m);
    // The rescale of the run's sums (nothing summed yet: they are 0).
    sa[rt] = mrun[rt] == -INFINITY ? 1.f : __builtin_amdgcn_exp2f(mrun[rt] - mh[rt]);
    mrun[rt] = mh[rt];
    // P alpha^V <= 2^(m2 - m) < 2^e; one bit of margin for the hardware exp2 and log2,
    // so P alpha^V 2^fv < 2^30.  (A chunk far below the run's maximum: e is held at -90, so
    // that 2^fv stays in range; what that rounds away is below 2^-119 of the sum.)
    int e = 0;
    frexpf(__builtin_amdgcn_exp2f(m2 - mh[rt]), &e);
    fvh[rt] = m2 > -INFINITY ? 29 - max(e, -90) : 0;
  }
  // Token 16 q + 4 e + L of a block sits at bit d = 2 e + q % 2 of its value byte; this
  // lane's tokens have e = hc.
  float sc_even[NT], sc_odd[NT];
#pragma unroll
  for (int rt = 0; rt < NT; ++rt) {
    sc_even[rt] = ldexpf(1.f, fvh[rt] - 2 * hc);
    sc_odd[rt] = (hc == 3 ? -1.f : 1.f) * ldexpf(1.f, fvh[rt] - 2 * hc - 1);
  }
#pragma unroll
  for (int rt = 0; rt < NT; ++rt) {
    float lsum = 0.f, pasum = 0.f;
#pragma unroll
    for (int ch = 0; ch < CPW; ++ch) {
      uint32_t y[4];
#pragma unroll
      for (int qd = 0; qd < 4; ++qd) {
        const int tt = 4 * ch + qd;
        const float z = zr[tt][rt];
        // (the hardware exp2: results below 2^-126 flush to 0, below any weight that counts)
        const float p = (z == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(z - mh[rt]);
        lsum += p;
        pasum = fmaf(p, avt[tt], pasum);
        const int fx = (int)rintf(p * avt[tt] * ((qd & 1) ? sc_odd[rt] : sc_even[rt]));
        uint32_t x = pack_limbs(fx);
        // quad byte transpose: (token L, limbs 0..3) -> (limb L, tokens 0..3)
        x = __builtin_amdgcn_perm(quad_xor2(x), x, sel_a);
        y[qd] = __builtin_amdgcn_perm(quad_xor1(x), x, sel_b);
      }
      // Limb L of head g for tokens 16 q + 4 hc + (0..3): lane 16 hc + 4 g + L of the
      // value phase's B operand.
      pb[((wave * CPW + ch) * NT + rt) * 64 + 16 * hc + 4 * g + L] =
          (v4i){(int)y[0], (int)y[1], (int)y[2], (int)y[3]};
    }
    lrun[rt] = fmaf(lrun[rt], sa[rt], lsum);
    parun[rt] = fmaf(parun[rt], sa[rt], pasum);
  }
  // The value tiles have landed (the next chunk's key transfers, issued after them, may
  // still be in flight).
  wait_vmcnt_small(nk_mine);
  __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
  plain_barrier();

  // (6) Value bits x P limbs, into the run's sums.
  if (!more) {
    load_tables();
  }
  // A operands (this half's blocks) stay in registers when they fit (16 x 4 VGPRs).
  constexpr bool kPbRegs = NCW * NT <= 16;
  v4i pbr[kPbRegs ? NCW * NT : 1];
  if constexpr (kPbRegs) {
    // All reads first (one LDS round trip), then the pins that keep them in registers
    // rather than re-read per tile.
#pragma unroll
    for (int i = 0; i < NCW * NT; ++i) pbr[i] = pbh[i * 64 + lane];
#pragma unroll
    for (int i = 0; i < NCW * NT; ++i) asm volatile("" : "+v"(pbr[i]));
  }
  float osc[NT];
#pragma unroll
  for (int rt = 0; rt < NT; ++rt) osc[rt] = ldexpf(1.f, -fvh[rt]);
#pragma unroll
  for (int it = 0; it < kMaxIt; ++it) {
    const int vt = wj + NWT * it;
    if (vt >= NVT || (ONE && hf * NCW * kTile >= nt)) break;   // (uniform; the half has no token)
    // One accumulator per column tile: a dependent product takes its predecessor's result
    // straight from the matrix unit.
    v4i acc[NT];
#pragma unroll
    for (int rt = 0; rt < NT; ++rt) acc[rt] = (v4i){0, 0, 0, 0};
    // All of the tile's value-bit words first (one LDS round trip), then the products.
    typedef uint32_t v2u __attribute__((ext_vector_type(2)));
    v2u wws[NCW];
#pragma unroll
    for (int ch = 0; ch < NCW; ++ch)
      wws[ch] = *(const __attribute__((address_space(3))) v2u*)(uintptr_t)(
          vaddr[ch] + 128 * NWT * it);
    // (The scheduler would otherwise pair each read with its products: one LDS round
    // trip per block.)
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int ch = 0; ch < NCW; ++ch) {
      const v2u ww = wws[ch];
      const v4i av4 = {(int)(ww.x & m0), (int)(ww.x & m1), (int)(ww.y & m0), (int)(ww.y & m1)};
#pragma unroll
      for (int rt = 0; rt < NT; ++rt) {
        const v4i bop = kPbRegs ? pbr[kPbRegs ? ch * NT + rt : 0] : pbh[(ch * NT + rt) * 64 + lane];
        acc[rt] = mfma_i8(bop, av4, acc[rt]);
      }
    }
    // (P limbs are the A operand: lane 16 h + n ends with the four limb sums of head h for
    // value bit 16 vt + n.)
#pragma unroll
    for (int rt = 0; rt < NT; ++rt) {
      const v4i d = acc[rt];
      float f = fmaf((float)d[3], 256.f, (float)d[2]);
      f = fmaf(f, 256.f, (float)d[1]);
      f = fmaf(f, 256.f, (float)d[0]);
      oacc[it][rt] = fmaf(oacc[it][rt], sa[rt], f * osc[rt]);
    }
  }
  if (!more) break;
  // The next chunk's key records have landed and every wave is done with the value tiles
  // and operands: the value region takes the next chunk's tiles.
  __builtin_amdgcn_s_waitcnt(kWaitVm0);
  __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
  plain_barrier();
  issue_values(c + 1, wave, NW);
  }

  // T_V's matrix-core operands (32 VGPRs): every run loads them, and the one that merges has
  // them at hand.
  TvMfma tv;
  const bool triple = NP > 4 || (!APPEND && hg > 1);
  tv.load(hv, triple);
  // O'(v) of both halves to LDS (over the consumed key records), the sums per wave.
  float* ob = reinterpret_cast<float*>(smem + a.off_ob);   // [halves][NH][ob_stride]
  float* obh = ob + hf * NH * a.ob_stride;
#pragma unroll
  for (int it = 0; it < kMaxIt; ++it) {
    const int vt = wj + NWT * it;
    if (vt >= NVT) break;                           // (uniform)
#pragma unroll
    for (int rt = 0; rt < NT; ++rt) obh[(4 * rt + g) * a.ob_stride + 16 * vt + n] = oacc[it][rt];
  }
#pragma unroll
  for (int rt = 0; rt < NT; ++rt) {
    const float lsum = row16_sum(lrun[rt]), pasum = row16_sum(parun[rt]);
    if (n == 0) {
      wsum[wave][4 * rt + g] = lsum;
      wpav[wave][4 * rt + g] = pasum;
      if (wave == 0) mfin[4 * rt + g] = mrun[rt];
    }
  }
  __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
  plain_barrier();

  if constexpr (APPEND) {
    // Fused append: the coefficients into the workspace (device-coherent, before this
    // workgroup's arrival).  Coefficient d at d; the wave or lane with the token's first
    // channel (d = 0 keys, 128 values) also stores the token's error bound at 2 kD + d / kD.
    const __amdgpu_buffer_rsrc_t rrs = make_rsrc(a.append_r + row * kAppStride, kAppStride * 4);
    if (cw) {
#pragma unroll
      for (int f = 0; f < KF; ++f) {
        if (adk[f] < 2 * kD && lane == 0) buf_store4_coherent(rcf[f], rrs, (uint32_t)(4 * adk[f]));
        if (adk[f] < 2 * kD && (adk[f] & (kD - 1)) == 0 && lane == 0)
          buf_store4_coherent(reh[f], rrs, (uint32_t)(4 * (2 * kD + adk[f] / kD)));
      }
    } else if (tail_wave) {
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        const int d = tail_dot(r);
        if (r >= tail_rounds || d >= 2 * kD) continue;
        buf_store4_coherent(r_tail[r], rrs, (uint32_t)(4 * d));
        if ((d & (kD - 1)) == 0)
          buf_store4_coherent(eh_tail[r], rrs, (uint32_t)(4 * (2 * kD + d / kD)));
      }
    }
  }
  const int v_maxb = hdr_s[1];
  const bool layout_ok = (hdr_s[4] == RK) & (hdr_s[5] == RV);
  // (7) Partial: o~_c = s_c 2^(1-b_c) (sum_{k < b-1} 2^k O'(c,k) - 2^(b-1) O'(c,b-1)),
  //     one (head, channel) per thread; midrise adds s_c 2^(-b_c) sum_i P_i alpha^V_i
  //     (the half step of every level).
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    const int h = (r * NTHR + tid) / kD;
    if (h < G) {
      const float* oh = ob + h * a.ob_stride;
      float acc = 0.f;
      auto bit_term = [&](int k) {
        const int v = min(voc + k, 8 * RV - 1);
        const float t = ldexpf(oh[v] + oh[NH * a.ob_stride + v], k);
        acc += (k < vbc) ? ((k == vbc - 1) ? -t : t) : 0.f;
      };
      // (the first eight bits unrolled with their reads issued together; wider codes take
      // the loop after)
#pragma unroll
      for (int k = 0; k < 8; ++k) bit_term(k);
      for (int k = 8; k < v_maxb; ++k) bit_term(k);
      float pa = 0.f;
#pragma unroll
      for (int w = 0; w < NW; ++w) pa += wpav[w][h];
      const float o = vbc ? fmaf(vsc * vhs, pa, ldexpf(vsc * acc, 1 - vbc)) : 0.f;
      buf_store4_coherent(o, prs, (uint32_t)((split * G + h) * sizeof(Partial) + 16 + 4 * cq));
    }
  }
  if (tid < G) {
    float l = wsum[0][tid];
#pragma unroll
    for (int w = 1; w < NW; ++w) l += wsum[w][tid];
    buf_store16_coherent((v4f){layout_ok ? mfin[tid] : NAN, l, 0.f, 0.f}, prs,
                         (uint32_t)((split * G + tid) * sizeof(Partial)));
  }
  // The merge's scratch: from the start of the front region (its cache and O' are consumed).
  float* merge_scratch = reinterpret_cast<float*>(smem);
  unsigned* counter = a.counters + row * kCtrStride + 16 * hgi;
  if constexpr (APPEND) {
    AppendHook<NTHR, NH> hook;
    hook.coeff = a.append_r + row * kAppStride;
    hook.ehp[0] = hk;
    hook.ehp[1] = hv;
    hook.xrow[0] = static_cast<const uint8_t*>(a.x_k) + row * kD * x_eb;
    hook.xrow[1] = static_cast<const uint8_t*>(a.x_v) + row * kD * x_eb;
    hook.x_dtype = a.x_dtype;
    hook.k_codes = a.k_codes;
    hook.k_alpha = a.k_alpha;
    hook.v_codes = a.v_codes;
    hook.v_alpha = a.v_alpha;
    hook.row = row;
    hook.cap = a.cap;
    hook.len = len;
    hook.G = G;
    hook.rk = RK;
    hook.rv = RV;
    hook.on = len > 0;
    hook.e_mr = hdr_s[wave == 0 ? 3 : 2] == AATC_QUANT_MIDRISE;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      hook.e_b[i] = e_b[i];
      hook.e_off[i] = e_off[i];
      hook.e_s[i] = e_s[i];
    }
    hook.qc = qcl;
    hook.sc = reinterpret_cast<AppendScratch*>(smem + a.off_es);
    merge_if_last_wide<NTHR, NH>(G, ns, parts, counter, out_rows, merge_scratch, tv, triple, hook);
  } else if (a.seg) {
    SegHook sh{a.seg + row * all_heads + NH * hgi, mfin};
    merge_if_last_wide<NTHR, NH>(G, ns, parts, counter, out_rows, merge_scratch, tv, triple, sh);
  } else {
    NoHook none;
    merge_if_last_wide<NTHR, NH>(G, ns, parts, counter, out_rows, merge_scratch, tv, triple, none);
  }
}

}  // namespace

size_t decode_workspace_bytes(int batch, int n_q_heads, int n_kv_heads, int64_t cap,
                              int counter_rows) {
  return ws_layout(batch, n_q_heads, n_kv_heads, cap, counter_rows).total;
}

// The dynamic LDS limit of one kernel, raised on each device the first time a launch there
// needs more.  Safe for concurrent callers: a race can only repeat the (idempotent)
// attribute call, and the recorded limit only grows.
class LdsLimit {
 public:
  bool ensure(const void* kernel, size_t lds) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return false;
    if (dev < 0 || dev >= kDevices)      // beyond the table: set it every time
      return hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                                 (int)lds) == hipSuccess;
    size_t cur = set_[dev].load(std::memory_order_acquire);
    if (lds <= cur) return true;
    if (hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) !=
        hipSuccess)
      return false;
    while (cur < lds && !set_[dev].compare_exchange_weak(cur, lds, std::memory_order_acq_rel)) {
    }
    return true;
  }

 private:
  static constexpr int kDevices = 64;
  std::atomic<size_t> set_[kDevices] = {};
};

template <int NT, int NTILE, int NP, bool APPEND>
static aatc_status launch_mfma(DecodeArgs a, hipStream_t st) {
  constexpr int NTHR = kMfmaThreads, S = 128 * NTILE;
  const int64_t chunks = (a.cap + S - 1) / S;
  const int64_t rows = (int64_t)a.batch * a.n_kv_heads * a.hg;
  // About one workgroup per compute unit: a row's chunks in runs of equal length, or runs dealt by
  // the sequences' lengths.
  int64_t grid;
  const bool even = evenly_dealt(a.batch, rows, chunks);
  int n_splits = 0;                                   // workgroups per row (even)
  if (even) {
    n_splits = (int)std::min(chunks, std::max<int64_t>(1, kComputeUnits / rows));
    a.max_splits = n_splits;
    grid = rows * n_splits;
  } else {
    a.max_splits = (int)chunks;
    grid = ragged_grid(rows, chunks);
  }
  const MfmaLds l = mfma_lds(NT, NTILE, NP, a.rk, a.rv, APPEND);
  a.off_v = l.off_v;
  a.off_ak = l.off_ak;
  a.off_av = l.off_av;
  a.off_ql = l.off_ql;
  a.off_qc = l.off_qc;
  a.off_pb = l.off_pb;
  a.off_ob = l.off_ob;
  a.ob_stride = l.ob_stride;
  a.off_es = l.off_es;
  const size_t lds = l.total;
  const uint32_t shape = (uint32_t)a.G | (uint32_t)a.hg << 8 | (even ? 0x10000u : 0u) |
                         (a.q_dtype == AATC_BF16 ? 0x20000u : 0u);
  auto launch = [&](auto kernel, LdsLimit& limit) {
    if (!limit.ensure((const void*)kernel, lds)) return AATC_E_DEVICE;
    hipLaunchKernelGGL(kernel, dim3((unsigned)grid), dim3(NTHR), lds, st, a.seq_len, a.params_k,
                       a.params_v, a.q, n_splits, a.n_kv_heads, a.batch, shape, a);
    return hipGetLastError() == hipSuccess ? AATC_OK : AATC_E_DEVICE;
  };
  static LdsLimit limit_one, limit_run;
  return even && chunks <= n_splits
             ? launch(decode_mfma_kernel<NT, NTILE, NP, APPEND, true>, limit_one)
             : launch(decode_mfma_kernel<NT, NTILE, NP, APPEND, false>, limit_run);
}

template <int NT, int NTILE, bool APPEND>
static aatc_status launch_mfma_np(const DecodeArgs& a, int np, hipStream_t st) {
  switch (np) {
    case 1: return launch_mfma<NT, NTILE, 1, APPEND>(a, st);
    case 2: return launch_mfma<NT, NTILE, 2, APPEND>(a, st);
    case 3: return launch_mfma<NT, NTILE, 3, APPEND>(a, st);
    default: return launch_mfma<NT, NTILE, 4, APPEND>(a, st);
  }
}

template <int NT, bool APPEND>
static aatc_status launch_mfma_nt(const DecodeArgs& a, const MfmaPlan& p, hipStream_t st) {
  if (p.np == 8) return launch_mfma<1, 4, 8, APPEND>(a, st);      // (four heads)
  if (p.np == 6) return launch_mfma<NT, 4, 6, APPEND>(a, st);
  return p.ntile == 8 ? launch_mfma_np<NT, 8, APPEND>(a, p.np, st)
                      : launch_mfma_np<NT, 4, APPEND>(a, p.np, st);
}

aatc_status launch_decode(const void* params_k, const void* params_v, int batch,
                          int n_q_heads, int n_kv_heads, const void* q, aatc_dtype q_dtype,
                          const void* k_codes, const uint16_t* k_alpha, const void* v_codes,
                          const uint16_t* v_alpha, const int32_t* seq_len, int64_t cap,
                          int rk, int rv, float softmax_scale, float* out, void* workspace,
                          void* stream, const void* x_k, const void* x_v, aatc_dtype x_dtype,
                          int counter_rows, const void* seg_k, const void* seg_v,
                          aatc_dtype seg_dtype, const int32_t* seg_len, int seg_cap) {
  const int G = n_q_heads / n_kv_heads;
  const WsLayout wl = ws_layout(batch, n_q_heads, n_kv_heads, cap, counter_rows);
  char* ws = static_cast<char*>(workspace);
  auto* ctr = reinterpret_cast<unsigned*>(ws + wl.counters);
  auto* parts = reinterpret_cast<Partial*>(ws + wl.partials);
  const hipStream_t st = (hipStream_t)stream;
  // Buffer descriptors address at most 2^31 bytes of one (sequence, KV head).
  if (cap * std::max(rk, rv) >= ((int64_t)1 << 31)) return AATC_E_UNSUPPORTED;
  if ((cap / kMinSplit + 1) * G * (int64_t)sizeof(Partial) >= ((int64_t)1 << 31))
    return AATC_E_UNSUPPORTED;
  // Everything that can refuse the call comes before the first launch.
  const bool mfma = rk <= kMfmaRecord && rv <= kMfmaRecord;
  const MfmaPlan plan = mfma_plan(rk, rv, G, (int64_t)batch * n_kv_heads, cap, x_k != nullptr);
  if (mfma && (int64_t)batch * n_kv_heads * plan.hg * ((cap + 511) / 512) > (1 << 30))
    return AATC_E_UNSUPPORTED;
  const size_t lds = std::max((size_t)G * (kSplit + 8 * std::max(rk, rv)) * sizeof(float),
                              merge_lds_bytes(G, kThreads));      // (wider records)
  if (!mfma && lds > 160 * 1024 - 24 * 1024) return AATC_E_UNSUPPORTED;
  if (seg_k && (seg_cap > kSegMax || x_k)) return AATC_E_UNSUPPORTED;
  // The full-precision segment's partials first (stream order makes them visible to the
  // merging workgroups of the launch below).
  const Partial* seg = nullptr;
  if (seg_k) {
    Partial* sp = reinterpret_cast<Partial*>(ws + wl.seg);
    hipLaunchKernelGGL(segment_partial_kernel, dim3((unsigned)(batch * n_kv_heads)),
                       dim3(kSegThreads), 0, st, n_q_heads, n_kv_heads, q, (int)q_dtype, seg_k, seg_v, (int)seg_dtype, seg_len, seg_cap,
                       softmax_scale * kLog2e, sp);
    if (hipGetLastError() != hipSuccess) return AATC_E_DEVICE;
    seg = sp;
  }
  // A new token's append is part of the matrix-core launch where that has one workgroup row per
  // KV head; other shapes run the per-token encode first.
  if (x_k && !(mfma && plan.fused)) {
    aatc_status e = launch_encode_last(params_k, n_kv_heads, batch, x_k, x_dtype,
                                       AATC_LAYOUT_RECORDS, const_cast<void*>(k_codes),
                                       const_cast<uint16_t*>(k_alpha), cap, rk, seq_len, stream);
    if (e == AATC_OK)
      e = launch_encode_last(params_v, n_kv_heads, batch, x_v, x_dtype, AATC_LAYOUT_TILES,
                             const_cast<void*>(v_codes), const_cast<uint16_t*>(v_alpha), cap, rv,
                             seq_len, stream);
    if (e != AATC_OK) return e;
  }
  if (mfma) {
    DecodeArgs a{};
    a.params_k = params_k;
    a.params_v = params_v;
    a.q = q;
    a.k_codes = static_cast<uint8_t*>(const_cast<void*>(k_codes));
    a.k_alpha = const_cast<uint16_t*>(k_alpha);
    a.v_codes = static_cast<uint8_t*>(const_cast<void*>(v_codes));
    a.v_alpha = const_cast<uint16_t*>(v_alpha);
    a.seq_len = seq_len;
    a.x_k = x_k;
    a.x_v = x_v;
    a.x_dtype = (int)x_dtype;
    a.out = out;
    a.counters = ctr;
    a.partials = parts;
    a.append_r = reinterpret_cast<float*>(ws + wl.append_r);
    a.seg = seg;
    a.cap = cap;
    a.batch = batch;
    a.n_q_heads = n_q_heads;
    a.n_kv_heads = n_kv_heads;
    a.G = G;
    a.hg = plan.hg;
    a.q_dtype = (int)q_dtype;
    a.rk = rk;
    a.rv = rv;
    a.scale_log2e = softmax_scale * kLog2e;
    if (plan.fused)
      return plan.nt == 1 ? launch_mfma_nt<1, true>(a, plan, st) : launch_mfma_nt<2, true>(a, plan, st);
    return plan.nt == 1 ? launch_mfma_nt<1, false>(a, plan, st) : launch_mfma_nt<2, false>(a, plan, st);
  }
  const int n_splits = (int)((cap + kSplit - 1) / kSplit);
  static LdsLimit limit;
  if (!limit.ensure((const void*)decode_split_kernel, lds)) return AATC_E_DEVICE;
  dim3 grid((unsigned)n_splits, (unsigned)n_kv_heads, (unsigned)batch);
  hipLaunchKernelGGL(decode_split_kernel, grid, dim3(kThreads), lds, st, params_k, params_v,
                     n_q_heads, n_kv_heads, q, (int)q_dtype,
                     static_cast<const uint8_t*>(k_codes), k_alpha,
                     static_cast<const uint8_t*>(v_codes), v_alpha, seq_len, cap,
                     softmax_scale, out, ctr, parts, n_splits, rk, rv, seg);
  return hipGetLastError() == hipSuccess ? AATC_OK : AATC_E_DEVICE;
}

}  // namespace aatc
