// Mixed-radix DFTs on tiles staged in LDS, for every axis length n = 2^a 3^b
// 5^c up to 4096 (host plan and device stages).
//
// An axis of length N = R_0 R_1 ... R_k is transformed in place by one
// butterfly pass per factor.  Position p = ((d_0 R_1 + d_1) R_2 + d_2) ... has
// digits d_i with strides S_i = R_{i+1} ... R_k.  The decimation in frequency
// (DIF) takes natural order and runs the stages 0 .. k: stage i replaces digit
// d_i by the frequency digit k_i, the twiddles W_N^(t n_i S_i) applied to its
// inputs, t = k_0 + R_0 k_1 + ... of the digits before it; position p then
// holds frequency freq(p) = k_0 + R_0 (k_1 + R_1 (k_2 + ...)).  The decimation
// in time (DIT) is its mirror image: it takes that digit-reversed order, runs
// the stages k .. 0 with the twiddles W_N^(l d_i N / (R_i S_i)), l the position's
// part below digit i, and leaves natural order.  A butterfly owns the
// positions it reads and writes, so a stage needs one buffer and one barrier,
// and a DIF followed by a pointwise product and a DIT (spectral multiply,
// orientation sum and division, Phi) never reorders: the product runs in
// registers between the last DIF and the first DIT butterfly, which are the
// same digit.
//
// Two factorisations.  The balanced one (radix_schedule) has the fewest
// stages and twiddle-free composite butterflies.  The sequential one is for
// the forward transform into 16-bit scores: there a last-bit difference of a
// value near a rounding boundary changes the stored word, and stored words are
// kept from one version of the library to the next (a score written earlier
// equals the one computed again).  So its sums keep one fixed order (the factors
// 16 .., 8 | 4 | 2, 5 .., 3 .. by decimation in frequency in both directions, y
// before x on the way to space) however the work is divided, and its products
// the roundings that the words were first written with.  Two neighbouring
// factors share a stage when their product is at most 16: the butterflies of
// both run in registers, with the second one's twiddles in between.
#pragma once
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>
#include <vector>

#include "fft_pass.h"
#include "fft_radix.h"

namespace os3d {

constexpr int kMaxFactors = 8;  // of a sequential schedule: 2187 = 3^7

struct AxisT {
  int N, nst;
  int R[kMaxStages], S[kMaxStages];
  int RB[kMaxStages];           // second factor of a two-factor stage (sequential), else 1 (or 0: seq_butterfly)
  int nb[kMaxStages];           // N / R: butterflies of a stage
  int tstep[kMaxStages];        // N / (R S): the product of the factors before the stage
  unsigned mS[kMaxStages];      // fast division by S
  int nf, F[kMaxFactors];       // single factors
  unsigned mF[kMaxFactors];
  const float2* tw;             // exp(-2 pi i j / N) at tw[j tws]
  int tws;
};

struct TileArgs {
  PassArgs p;
  AxisT x, y;     // x: the contiguous axis of a tile; y: its row axis (the line axis of a line kernel)
  // line kernels (y or z lines): W = 2^lw lines side by side per workgroup
  int lw;
  int lb;              // split passes: 2^lb of the 2^lw lines are one residue class of y
  long long lines;     // lines per volume (split: per class member)
  long long dn;        // elements between consecutive points of a line
  int chunks;          // y lines: workgroups along x (per z plane); z lines: all workgroups
  int xcd;             // chunks of an XCD (0: in the order of the workgroups)
  int groups;          // workgroups that share the pairs of a launch
  int two;             // the LDS holds two tiles: successive pairs alternate, one barrier a pair less
  float2* part;        // the pairs' intermediates: group g > 0 sums into the first of its own
  int finish;          // the orientation sum goes on through the division and the inverse DFT
  // plane and row kernels
  int rows, P, A;      // rows = P A rows of x.N values per tile
  int RS, pad;         // LDS row stride; values skipped after every x.R[last]
  int B;                 // split passes: tile of class yb = rows yb, yb + B, ... of its plane in space
  unsigned mB;
  unsigned mrows, mNx, mRL, mP, mA, mnf;
  long long tiles;     // tiles per volume
  long long nlines;    // x lines per volume
};

// ---------------------------------------------------------------- device helpers
// n / d for the multiplier m = ceil(2^32 / d) (0 for d = 1), exact for n d < 2^32
__device__ __forceinline__ int fdiv(int n, unsigned m) { return m ? (int)__umulhi((unsigned)n, m) : n; }

__device__ __forceinline__ float2 cmulc(float2 a, float2 b) {  // a conj(b)
  return make_float2(a.x * b.x + a.y * b.y, a.y * b.x - a.x * b.y);
}

// f(integral_constant<R>) for the run-time radix R
template <class F>
__host__ __device__ __forceinline__ void with_radix(int R, F f) {
  switch (R) {
    case 2: f(std::integral_constant<int, 2>{}); break;
    case 3: f(std::integral_constant<int, 3>{}); break;
    case 4: f(std::integral_constant<int, 4>{}); break;
    case 5: f(std::integral_constant<int, 5>{}); break;
    case 6: f(std::integral_constant<int, 6>{}); break;
    case 8: f(std::integral_constant<int, 8>{}); break;
    case 9: f(std::integral_constant<int, 9>{}); break;
    case 10: f(std::integral_constant<int, 10>{}); break;
    case 12: f(std::integral_constant<int, 12>{}); break;
    case 15: f(std::integral_constant<int, 15>{}); break;
    default: f(std::integral_constant<int, 16>{}); break;
  }
}
#define OS3D_RADIX_FN(rc) [&](auto rc) __attribute__((always_inline))

// v[r] *= W^(r idx) (conjugated for the inverse direction)
template <int R, bool INV>
__device__ __forceinline__ void twiddle(float2* v, const float2* tw, int idx) {
#pragma unroll
  for (int r = 1; r < R; ++r) v[r] = INV ? cmulc(v[r], tw[r * idx]) : cmul(v[r], tw[r * idx]);
}

// frequency held at position p after a DIF
__device__ __forceinline__ int freq_of(const AxisT& ax, int p) {
  int f = 0;
  for (int i = ax.nf - 1; i >= 0; --i) {
    const int q = fdiv(p, ax.mF[i]);
    f = (p - q * ax.F[i]) + ax.F[i] * f;
    p = q;
  }
  return f;
}

// f(integral_constant<R>, integral_constant<RB>) for a stage of the sequential schedule
template <class Fn>
__host__ __device__ __forceinline__ void with_seq(int R, int RB, Fn f) {
  using std::integral_constant;
  switch (R * 16 + RB) {
    case 2 * 16 + 1: f(integral_constant<int, 2>{}, integral_constant<int, 1>{}); break;
    case 3 * 16 + 1: f(integral_constant<int, 3>{}, integral_constant<int, 1>{}); break;
    case 4 * 16 + 1: f(integral_constant<int, 4>{}, integral_constant<int, 1>{}); break;
    case 5 * 16 + 1: f(integral_constant<int, 5>{}, integral_constant<int, 1>{}); break;
    case 8 * 16 + 1: f(integral_constant<int, 8>{}, integral_constant<int, 1>{}); break;
    case 6 * 16 + 3: f(integral_constant<int, 6>{}, integral_constant<int, 3>{}); break;
    case 9 * 16 + 3: f(integral_constant<int, 9>{}, integral_constant<int, 3>{}); break;
    case 10 * 16 + 5: f(integral_constant<int, 10>{}, integral_constant<int, 5>{}); break;
    case 12 * 16 + 3: f(integral_constant<int, 12>{}, integral_constant<int, 3>{}); break;
    case 15 * 16 + 3: f(integral_constant<int, 15>{}, integral_constant<int, 3>{}); break;
    case 4 * 16 + 0: f(integral_constant<int, 4>{}, integral_constant<int, 0>{}); break;
    case 8 * 16 + 0: f(integral_constant<int, 8>{}, integral_constant<int, 0>{}); break;
    case 16 * 16 + 0: f(integral_constant<int, 16>{}, integral_constant<int, 0>{}); break;
    default: f(integral_constant<int, 16>{}, integral_constant<int, 1>{}); break;
  }
}
#define OS3D_SEQ_FN(rc, rb) [&](auto rc, auto rb) __attribute__((always_inline))

// Butterflies of the sequential schedule.  Left to itself the compiler picks
// which product of a sum it fuses by the code around it, so here every sum
// with two products names the fused one; hold() keeps a value rounded.  Which
// product that is follows from no rule of the method: it is what the stored
// words were first computed with (the lines of 64, 128 and 256 points by kernels
// of their own, hence their second and third forms), each as accurate as the other.
__device__ __forceinline__ void hold(float2& v) { asm("" : "+v"(v.x), "+v"(v.y)); }

__device__ __forceinline__ float2 seq_mul(float2 a, float2 b) {
  float2 p = make_float2(a.y * b.y, a.x * b.y);
  hold(p);
  float2 r = make_float2(__builtin_fmaf(a.x, b.x, -p.x), __builtin_fmaf(a.y, b.x, p.y));
  hold(r);
  return r;
}
// the imaginary part's other product fused
__device__ __forceinline__ float2 seq_mul_alt(float2 a, float2 b) {
  float2 p = make_float2(a.y * b.y, a.y * b.x);
  hold(p);
  float2 r = make_float2(__builtin_fmaf(a.x, b.x, -p.x), __builtin_fmaf(a.x, b.y, p.y));
  hold(r);
  return r;
}

__device__ __forceinline__ void seq_dft3(float2* v, float sgn) {
  const float s3 = 0.866025403784438646764f * sgn;
  const float2 t1 = cadd(v[1], v[2]), t2 = csub(v[1], v[2]);
  const float2 m = make_float2(__builtin_fmaf(-0.5f, t1.x, v[0].x), __builtin_fmaf(-0.5f, t1.y, v[0].y));
  v[0] = cadd(v[0], t1);
  v[1] = make_float2(__builtin_fmaf(-s3, t2.y, m.x), __builtin_fmaf(s3, t2.x, m.y));
  v[2] = make_float2(__builtin_fmaf(s3, t2.y, m.x), __builtin_fmaf(-s3, t2.x, m.y));
}

__device__ __forceinline__ void seq_dft5(float2* v, float sgn) {
  const float c1 = 0.309016994374947424102f, c2 = -0.809016994374947424102f;
  const float s1 = 0.951056516295153572116f * sgn, s2 = 0.587785252292473129169f * sgn;
  const float2 t1 = cadd(v[1], v[4]), t2 = cadd(v[2], v[3]), t3 = csub(v[1], v[4]), t4 = csub(v[2], v[3]);
  const float2 a1 = make_float2(__builtin_fmaf(c2, t2.x, __builtin_fmaf(c1, t1.x, v[0].x)),
                                __builtin_fmaf(c2, t2.y, __builtin_fmaf(c1, t1.y, v[0].y)));
  const float2 a2 = make_float2(__builtin_fmaf(c1, t2.x, __builtin_fmaf(c2, t1.x, v[0].x)),
                                __builtin_fmaf(c1, t2.y, __builtin_fmaf(c2, t1.y, v[0].y)));
  float2 p = cscale(t3, s1), q = cscale(t4, s1);
  hold(p);
  hold(q);
  float2 b1 = make_float2(__builtin_fmaf(s2, t4.x, p.x), __builtin_fmaf(s2, t4.y, p.y));
  float2 b2 = make_float2(__builtin_fmaf(s2, t3.x, -q.x), __builtin_fmaf(s2, t3.y, -q.y));
  hold(b1);
  hold(b2);
  v[0] = cadd(v[0], cadd(t1, t2));
  v[1] = make_float2(a1.x - b1.y, a1.y + b1.x);
  v[4] = make_float2(a1.x + b1.y, a1.y - b1.x);
  v[2] = make_float2(a2.x - b2.y, a2.y + b2.x);
  v[3] = make_float2(a2.x + b2.y, a2.y - b2.x);
}

__device__ __forceinline__ void seq_dft8(float2* v, float sgn) {
  const float r = 0.707106781186547524401f;
  float2 e0 = v[0], e1 = v[2], e2 = v[4], e3 = v[6];
  float2 o0 = v[1], o1 = v[3], o2 = v[5], o3 = v[7];
  dft4(e0, e1, e2, e3, sgn);
  dft4(o0, o1, o2, o3, sgn);
  const float2 p = make_float2(__builtin_fmaf(-sgn, o1.y, o1.x), __builtin_fmaf(sgn, o1.x, o1.y));
  const float2 q = make_float2(__builtin_fmaf(-sgn, o3.y, -o3.x), __builtin_fmaf(sgn, o3.x, -o3.y));
  const float2 w2o = cmul_si(o2, sgn);
  v[0] = cadd(e0, o0);
  v[4] = csub(e0, o0);
  v[1] = make_float2(__builtin_fmaf(r, p.x, e1.x), __builtin_fmaf(r, p.y, e1.y));
  v[5] = make_float2(__builtin_fmaf(-r, p.x, e1.x), __builtin_fmaf(-r, p.y, e1.y));
  v[2] = cadd(e2, w2o);
  v[6] = csub(e2, w2o);
  v[3] = make_float2(__builtin_fmaf(r, q.x, e3.x), __builtin_fmaf(r, q.y, e3.y));
  v[7] = make_float2(__builtin_fmaf(-r, q.x, e3.x), __builtin_fmaf(-r, q.y, e3.y));
}

// KIND 0; 1: lines of 64, 128 and 256 points; 2: those of a real volume
// (its two middle products of row 2 are fused into the sums).
template <int KIND>
__device__ __forceinline__ void seq_dft16(float2* v, float sgn) {
  const float c1 = 0.923879532511286756128f, s1 = 0.382683432365089771728f, r = 0.707106781186547524401f;
#pragma unroll
  for (int n2 = 0; n2 < 4; ++n2) dft4(v[n2], v[4 + n2], v[8 + n2], v[12 + n2], sgn);
  const float2 w1 = make_float2(c1, sgn * s1), w2 = make_float2(r, sgn * r), w3 = make_float2(s1, sgn * c1);
  const float2 w4 = make_float2(0.f, sgn), w6 = make_float2(-r, sgn * r), w9 = make_float2(-c1, -sgn * s1);
  float2 a[4][4];
#pragma unroll
  for (int k1 = 0; k1 < 4; ++k1)
#pragma unroll
    for (int n2 = 0; n2 < 4; ++n2) a[k1][n2] = v[4 * k1 + n2];
  a[1][1] = seq_mul(a[1][1], w1);
  a[1][2] = seq_mul(a[1][2], w2);
  a[1][3] = seq_mul(a[1][3], w3);
  a[2][1] = KIND ? seq_mul_alt(a[2][1], w2) : seq_mul(a[2][1], w2);
  a[2][2] = seq_mul(a[2][2], w4);
  const float2 a23 = a[2][3];
  a[2][3] = seq_mul_alt(a[2][3], w6);
  a[3][1] = seq_mul(a[3][1], w3);
  a[3][2] = seq_mul_alt(a[3][2], w6);
  a[3][3] = seq_mul_alt(a[3][3], w9);
  if constexpr (KIND == 2) {
    const float2 t0 = cadd(a[2][0], a[2][2]), t1 = csub(a[2][0], a[2][2]);
    const float2 t2 = make_float2(a[2][1].x + a[2][3].x, __builtin_fmaf(w6.y, a23.x, a[2][1].y));
    const float2 d = make_float2(a[2][1].x - a[2][3].x, __builtin_fmaf(-w6.y, a23.x, a[2][1].y));
    const float2 t3 = cmul_si(d, sgn);
    a[2][0] = cadd(t0, t2);
    a[2][2] = csub(t0, t2);
    a[2][1] = cadd(t1, t3);
    a[2][3] = csub(t1, t3);
  }
#pragma unroll
  for (int k1 = 0; k1 < 4; ++k1) {
    if (KIND != 2 || k1 != 2) dft4(a[k1][0], a[k1][1], a[k1][2], a[k1][3], sgn);
#pragma unroll
    for (int k2 = 0; k2 < 4; ++k2) v[k1 + 4 * k2] = a[k1][k2];
  }
}

template <int R, int KIND>
__device__ __forceinline__ void seq_dft(float2* v, float sgn) {
  if constexpr (R == 3) seq_dft3(v, sgn);
  else if constexpr (R == 5) seq_dft5(v, sgn);
  else if constexpr (R == 8) seq_dft8(v, sgn);
  else if constexpr (R == 16) seq_dft16<KIND>(v, sgn);
  else dft_r<R>(v, sgn);
}

// A sequential stage on one butterfly: slot na RB + nb holds digits (na, nb),
// then (ka, kb).  tw is the table of the direction (conjugated for the
// inverse), t the frequency of the digits before the stage, S its stride, P
// the product of the factors before it.  RB = 0: one factor, in a line of 64,
// 128 or 256 points (REAL: its input is a real volume).
template <int R, int RB, bool REAL = false>
__device__ __forceinline__ void seq_butterfly(float2* v, const float2* tw, int t, int S, int P, bool first,
                                              float sgn) {
  constexpr int B = RB < 1 ? 1 : RB, RA = R / B;
  if (!first) {
#pragma unroll
    for (int na = 1; na < RA; ++na) {
      const float2 w = tw[t * S * B * na];
#pragma unroll
      for (int nb = 0; nb < B; ++nb) v[na * B + nb] = seq_mul(v[na * B + nb], w);
    }
  }
  if constexpr (B == 1) {
    if (RB == 0 && REAL && first)
      seq_dft<R, 2>(v, sgn);
    else
      seq_dft<R, RB == 0 ? 1 : 0>(v, sgn);
  } else {
#pragma unroll
    for (int nb = 0; nb < B; ++nb) {
      float2 u[RA];
#pragma unroll
      for (int na = 0; na < RA; ++na) u[na] = v[na * B + nb];
      seq_dft<RA, 0>(u, sgn);
#pragma unroll
      for (int na = 0; na < RA; ++na) {
        hold(u[na]);
        v[na * B + nb] = u[na];
      }
    }
#pragma unroll
    for (int ka = 0; ka < RA; ++ka) {
#pragma unroll
      for (int nb = 1; nb < B; ++nb) v[ka * B + nb] = seq_mul(v[ka * B + nb], tw[(t + P * ka) * S * nb]);
      seq_dft<B, 0>(v + ka * B, sgn);
    }
  }
}

// frequency of slot r of a stage relative to t, in units of P
template <int R, int RB>
__device__ __forceinline__ constexpr int seq_slot(int r) {
  return RB < 2 ? r : r / RB + (R / (RB < 2 ? 1 : RB)) * (r % (RB < 2 ? 1 : RB));
}

// ---------------------------------------------------------------- host plan
inline unsigned fdiv_mul(unsigned d) { return d <= 1 ? 0u : (unsigned)(((1ull << 32) + d - 1) / d); }

inline void set_stages(AxisT& a, int N, const float* tw) {
  a.N = N;
  int S = N;
  for (int i = 0; i < a.nst; ++i) {
    S /= a.R[i];
    a.S[i] = S;
    a.nb[i] = N / a.R[i];
    a.tstep[i] = N / (a.R[i] * S);
    a.mS[i] = fdiv_mul((unsigned)S);
  }
  for (int i = 0; i < a.nf; ++i) a.mF[i] = fdiv_mul((unsigned)a.F[i]);
  a.tw = (const float2*)tw;
  a.tws = 1;
}

// The balanced schedule.  odd_last moves an odd factor to the end: the
// digit-reversed rows of a plane are read in natural order, and an odd stride
// spreads those reads over the LDS banks.
inline AxisT make_axis(int N, const float* tw, bool odd_last = false) {
  AxisT a = {};
  std::vector<int> r = radix_schedule(N);
  if (odd_last && r.back() % 2 == 0)
    for (size_t i = r.size(); i-- > 0;)
      if (r[i] % 2) {
        std::swap(r[i], r.back());
        break;
      }
  a.nst = a.nf = (int)r.size();
  std::copy(r.begin(), r.end(), a.R);
  std::copy(r.begin(), r.end(), a.F);
  std::fill(a.RB, a.RB + kMaxStages, 1);
  set_stages(a, N, tw);
  return a;
}

// The sequential schedule, neighbouring factors joined into the fewest stages.
inline AxisT make_axis_seq(int N, const float* tw) {
  AxisT a = {};
  int m = N, p2 = 0;
  while (m % 2 == 0) m /= 2, ++p2;
  for (; p2 >= 4; p2 -= 4) a.F[a.nf++] = 16;
  if (p2) a.F[a.nf++] = 1 << p2;
  for (; m % 5 == 0; m /= 5) a.F[a.nf++] = 5;
  for (; m % 3 == 0; m /= 3) a.F[a.nf++] = 3;
  // best[i]: stages of the factors i ..; a stage takes two when that saves one
  int best[kMaxFactors + 2] = {};
  for (int i = a.nf - 1; i >= 0; --i) {
    best[i] = 1 + best[i + 1];
    if (i + 1 < a.nf && a.F[i] * a.F[i + 1] <= 16) best[i] = std::min(best[i], 1 + best[i + 2]);
  }
  for (int i = 0; i < a.nf;) {
    const bool two = i + 1 < a.nf && a.F[i] * a.F[i + 1] <= 16 && best[i] == 1 + best[i + 2];
    a.R[a.nst] = two ? a.F[i] * a.F[i + 1] : a.F[i];
    a.RB[a.nst++] = two ? a.F[i + 1] : 1;
    i += two ? 2 : 1;
  }
  if (N == 64 || N == 128 || N == 256) a.RB[0] = a.RB[1] = 0;
  set_stages(a, N, tw);
  return a;
}

// kernels_line.hip
int launch_zline_mul(const os3d_bank* b, const PassArgs& p, hipStream_t st);
int launch_zline_acc(const os3d_bank* b, const PassArgs& p, float2* T, int groups, bool finish, hipStream_t st);
int launch_zline_div(const os3d_bank* b, const PassArgs& p, float2* T, int groups, bool finish, hipStream_t st);
int launch_yline(const os3d_bank* b, const PassArgs& p, bool seq, hipStream_t st);
int zline_tiles(const os3d_bank* b);               // workgroups of one volume's z lines (16-bit scores)
int zline_acc_groups(const os3d_bank* b, int nb);  // partial sums of a launch over nb pairs
// kernels_tile.hip: whole (y, x) planes, or x lines
template <int LM, int SM>
int launch_tile(const os3d_bank* b, const PassArgs& p, bool plane, bool seq, hipStream_t st);
int launch_tile_phi(const os3d_bank* b, const PassArgs& p, bool plane, hipStream_t st);

}  // namespace os3d
