// Arguments and fused per-value loads and stores shared by the DFT pass
// kernels (lines, planes and tiles of the general path, and the 256^3 path).
#pragma once
#include <hip/hip_bf16.h>
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include "fft_radix.h"
#include "os3d_internal.h"

namespace os3d {

constexpr int kMaxBatch = 64;    // orientation pairs per launch

enum LoadMode { LM_REAL = 0, LM_C = 1, LM_MULBANK = 2, LM_UIN = 3, LM_DIVM = 4 };
enum StoreMode { SM_C = 0, SM_UOUT = 1, SM_ACCUM = 2, SM_REAL = 3 };

struct PassArgs {
  int Nz, Ny, Nx;
  long long V;
  const float2* tw;     // exp(-2 pi i j / N) of the x axis
  float sgn;            // -1: forward DFT, +1: inverse DFT
  int nb;               // pairs in this launch
  int split;            // factor B of the y axis that the z-line passes take (0: none)
  int newest_first;     // the pairs in descending order (their source was written in ascending order)
  // sources
  const float* src_r;
  const float2* src_c;
  long long src_stride;  // per pair (elements)
  const float* psi;      // bank rows (without kappa)
  float kappa;           // the bank's normaliser: LM_MULBANK multiplies by kappa psi, LM_DIVM by kappa
  int rows[kMaxBatch];
  int oa[kMaxBatch], ob[kMaxBatch];  // stored member, partner (-1 if none)
  const void* U;
  int dtype;
  const float* scales;   // [N_o] of this volume
  const float* M;
  float eps;
  int divide;
  // destinations
  float2* dst_c;
  long long dst_stride;
  float* dst_r;
  void* Uout;
  float out_scale;
  float* partial;        // [nb][tiles] sums of |value| (scale bound), or null
  const float* tsc;      // 256^3 fp16 intermediates: scales of the writing workgroups [nb][1024]
  float* tsc_out;        // where the writing pass puts them
  int accumulate;        // SM_ACCUM: 1 adds to X, 0 overwrites
  int phi_kind;          // phi_apply: 0 identity, 1 |U|^phi_p sgn(U)
  float phi_p;
};

// Non-temporal loads for values a pass streams through once (a plain read
// kernel reaches 6.3 TB/s on this GPU, 7.0 TB/s with the hint).  Measured per
// kernel: they speed up the bank-row and intermediate reads of the
// orientation-sum passes and the z-line and plane passes, and slow down the
// other 256^3 passes, which keep plain loads.
typedef float nt_float2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ float2 ldnt(const float2* p) {
  const nt_float2 v = __builtin_nontemporal_load((const nt_float2*)p);
  return make_float2(v.x, v.y);
}
__device__ __forceinline__ float ldnt(const float* p) { return __builtin_nontemporal_load(p); }
__device__ __forceinline__ unsigned int ldnt(const unsigned int* p) { return __builtin_nontemporal_load(p); }

__device__ __forceinline__ unsigned int bf16_rne(float x) {
  unsigned int u = __float_as_uint(x);
  unsigned int lsb = (u >> 16) & 1u;
  return (u + 0x7fffu + lsb) >> 16;
}

// Score element i as complex float (16-bit pairs times their scale s).  The
// storage type is a template parameter so that the loads of a pass are not
// separated by branches and can all be in flight together.
// A stored 16-bit pair times its scale s.
template <int DT>
__device__ __forceinline__ float2 score_value(unsigned int q, float s) {
  float re, im;
  if constexpr (DT == OS3D_F16X2) {
    re = __half2float(__ushort_as_half((unsigned short)(q & 0xffffu)));
    im = __half2float(__ushort_as_half((unsigned short)(q >> 16)));
  } else {
    re = __uint_as_float((q & 0xffffu) << 16);
    im = __uint_as_float(q & 0xffff0000u);
  }
  return make_float2(re * s, im * s);
}

template <int DT>
__device__ __forceinline__ float2 load_score(const void* U, long long i, float s) {
  if constexpr (DT == OS3D_C64)
    return ((const float2*)U)[i];
  else
    return score_value<DT>(((const unsigned int*)U)[i], s);
}


template <int DT>
__device__ __forceinline__ void store_score(void* U, long long i, float2 v, float inv_s) {
  if constexpr (DT == OS3D_C64) {
    ((float2*)U)[i] = v;
  } else {
    const float re = v.x * inv_s, im = v.y * inv_s;
    unsigned int q;
    if constexpr (DT == OS3D_F16X2)
      q = (unsigned int)__half_as_ushort(__float2half_rn(re)) |
          ((unsigned int)__half_as_ushort(__float2half_rn(im)) << 16);
    else
      q = bf16_rne(re) | (bf16_rne(im) << 16);
    ((unsigned int*)U)[i] = q;
  }
}

// Phi of processing via scores applied to one transformed value v (times
// out_scale = 1/V), times 2 for a stored antipodal pair: for real f the pair
// contributes Phi(U_n) + conj(Phi(U_-n)) = 2 Phi(U_n) to the reconstruction.
// |U|^(p-1) = 2^((p-1)/2 log2 |U|^2) with the hardware base-2 logarithm
// and exponential (about 1 ulp each; powf costs ~170 instructions).  The
// hardware logarithm flushes denormal inputs to zero, so a score whose
// components are both below 2^-60 is scaled by 2^96 before it is squared
// (every such |U|^2, down to the smallest denormal component, is then a
// normal number) and log2 |U|^2 is corrected by -192.
__device__ __forceinline__ float2 phi_apply(const PassArgs& a, int j, float2 v) {
  const float2 u = cscale(v, a.out_scale);
  const float mult = (a.ob[j] >= 0) ? 2.f : 1.f;
  if (a.phi_kind == 1) {
    const bool tiny = fmaxf(fabsf(u.x), fabsf(u.y)) < 0x1p-60f;
    const float2 w = tiny ? cscale(u, 0x1p96f) : u;
    const float l2 = __builtin_amdgcn_logf(w.x * w.x + w.y * w.y) - (tiny ? 192.f : 0.f);
    const float f = __builtin_amdgcn_exp2f(0.5f * (a.phi_p - 1.f) * l2);
    return cscale(u, (u.x != 0.f || u.y != 0.f) ? mult * f : 0.f);
  }
  return cscale(u, mult);
}

// K values of one thread at the affine positions g0 + r d (r < K), for pair
// slot j (LM_REAL, LM_UIN, LM_DIVM; the others are loaded by their kernels).
// Uniform conditions (partner present, division, scales) are
// decided once, outside the unrolled loops, so that each group of loads sits
// in one basic block and is issued back to back.
template <int LM, int DT, int K>
__device__ __forceinline__ void load_k(const PassArgs& a, int j, long long g0, long long d, float2 (&v)[K]) {
  if constexpr (LM == LM_REAL) {
#pragma unroll
    for (int r = 0; r < K; ++r) v[r] = make_float2(a.src_r[g0 + r * d], 0.f);
  } else if constexpr (LM == LM_UIN) {
    const int ia = a.oa[j], ib = a.ob[j];
    float sa = 1.f, sb = 1.f;
    if constexpr (DT != OS3D_C64) {
      sa = a.scales[ia];
      if (ib >= 0) sb = a.scales[ib];
    }
    const long long ba = (long long)ia * a.V + g0;
#pragma unroll
    for (int r = 0; r < K; ++r) v[r] = load_score<DT>(a.U, ba + r * d, sa);
    if (ib >= 0) {
      const long long bb = (long long)ib * a.V + g0;
      float2 w[K];
#pragma unroll
      for (int r = 0; r < K; ++r) w[r] = load_score<DT>(a.U, bb + r * d, sb);
#pragma unroll
      for (int r = 0; r < K; ++r) v[r] = cadd(v[r], cconj(w[r]));
    }
  } else {  // LM_DIVM
#pragma unroll
    for (int r = 0; r < K; ++r) v[r] = a.src_c[g0 + r * d];
    if (a.divide) {
      float m[K];
#pragma unroll
      for (int r = 0; r < K; ++r) m[r] = a.M[g0 + r * d];
#pragma unroll
      for (int r = 0; r < K; ++r) v[r] = cscale(v[r], a.kappa / fmaxf(m[r], a.eps));
    } else {
#pragma unroll
      for (int r = 0; r < K; ++r) v[r] = cscale(v[r], a.kappa);
    }
  }
}

// K values of one thread stored at g0 + r d for pair slot j; SM_ACCUM adds
// psi_hat_j * value into acc[r] instead.
template <int SM, int DT, int K>
__device__ __forceinline__ void store_k(const PassArgs& a, int j, long long g0, long long d, const float2 (&v)[K],
                                        float2 (&acc)[K]) {
  if constexpr (SM == SM_C) {
    float2* p = a.dst_c + j * a.dst_stride;
#pragma unroll
    for (int r = 0; r < K; ++r) p[g0 + r * d] = v[r];
  } else if constexpr (SM == SM_UOUT) {
    const int ia = a.oa[j], ib = a.ob[j];
    const float inv_s = (DT != OS3D_C64) ? 1.f / a.scales[ia] : 1.f;
    const long long ba = (long long)ia * a.V + g0;
#pragma unroll
    for (int r = 0; r < K; ++r) store_score<DT>(a.Uout, ba + r * d, cscale(v[r], a.out_scale), inv_s);
    if (ib >= 0) {
      const long long bb = (long long)ib * a.V + g0;
#pragma unroll
      for (int r = 0; r < K; ++r) store_score<DT>(a.Uout, bb + r * d, cconj(cscale(v[r], a.out_scale)), inv_s);
    }
  } else if constexpr (SM == SM_ACCUM) {
    const float* pr = a.psi + (long long)a.rows[j] * a.V;
    float ps[K];
#pragma unroll
    for (int r = 0; r < K; ++r) ps[r] = ldnt(pr + g0 + r * d);
#pragma unroll
    for (int r = 0; r < K; ++r) acc[r] = make_float2(acc[r].x + ps[r] * v[r].x, acc[r].y + ps[r] * v[r].y);
  } else {  // SM_REAL
#pragma unroll
    for (int r = 0; r < K; ++r) a.dst_r[g0 + r * d] = v[r].x * a.out_scale;
  }
}

// X (+)= acc at g0 + r d, the read of X (when adding) issued as one group.
template <int K>
__device__ __forceinline__ void flush_k(const PassArgs& a, long long g0, long long d, const float2 (&acc)[K]) {
  if (a.accumulate) {
    float2 x[K];
#pragma unroll
    for (int r = 0; r < K; ++r) x[r] = a.dst_c[g0 + r * d];
#pragma unroll
    for (int r = 0; r < K; ++r) a.dst_c[g0 + r * d] = cadd(x[r], acc[r]);
  } else {
#pragma unroll
    for (int r = 0; r < K; ++r) a.dst_c[g0 + r * d] = acc[r];
  }
}

// Per-kernel timer slots (os3d_profile_*): first / middle / last pass of the
// DFT of f, of the forward transform, of the reconstruction's orientation
// sum and of its final inverse DFT.
enum ProfKernel {
  kProfDftFirst = 0, kProfDftMid, kProfDftLast, kProfFwdFirst, kProfScales, kProfFwdMid, kProfFwdLast,
  kProfRecFirst, kProfRecMid, kProfRecLast, kProfInvFirst, kProfInvMid, kProfInvLast, kProfBank, kProfCount
};

void launch_scales(const float* partial, int ntiles, const PassArgs& a, int dtype, float* scales, int nb,
                   hipStream_t st);
int forward4(const os3d_bank* b, const float* f, int batch, void* U, int dtype, float* scales, void* ws, int nbmax,
             void* stream);
int reduce4(const os3d_bank* b, const void* U, int dtype, const float* scales, int batch, float* f_out, void* ws,
            bool divide_M, int nbmax, void* stream);
template <int LM, int SM>
void launch_plane(const PassArgs& a, int grid_y, hipStream_t st);
void launch_plane_phi(const PassArgs& a, int grid_y, hipStream_t st);
int process4(const os3d_bank* b, const float* f, int batch, int phi_kind, float phi_p, float* f_out, void* ws,
             int nbmax, void* stream);

}  // namespace os3d
