// Line passes of the general transform: the z lines with the spectral
// multiply, the orientation sum and the division fused in, and the y lines
// of volumes whose (y, x) planes do not fit in LDS (stages: fft_tile.h).
//
// A workgroup owns W neighbouring lines (consecutive x, so every access is a
// run of W values).  Each thread holds one butterfly: the first stage loads
// its inputs straight from memory and the last stage hands its outputs over
// in registers, so a two-factor line makes one LDS round trip.  The passes
// are bound by memory (a value costs one 8-byte read or write, its bank row
// entry and about 70 flops): the spectrum of a tile (k_line_mul) or its
// orientation sum (k_line_acc) stays in registers over the pairs of a launch.
//
// Split passes.  A (y, x) plane larger than LDS would take a pass over y and
// one over x.  Instead Ny = B A: the z-line passes take the factor B as well
// (a tile is W lines of each of the B rows ka + kb A) and the plane pass
// transforms the A rows of one class along y and x in LDS (kernels_tile.hip), so
// the intermediate goes through memory once, not twice, for one more stage
// in LDS.  Forward + reconstruction with 42 orientations, in three passes and
// split: 180 x 240 x 216 (B = 4) 4.58 and 3.52 ms, 64 x 320 x 320 (B = 8) 3.19 and
// 2.42 ms.  The forward into 16-bit scores keeps three passes: its order of sums
// is fixed.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <mutex>
#include <set>

#include "fft_tile.h"
#include "launch.h"

namespace os3d {

typedef unsigned short u16;

// One workgroup's LDS: the tile [position][W], twiddles, frequency of each position.
struct LineTile {
  float2* buf;
  float2* tw;
  float2* ts;  // split: twiddle between the classes and the z lines, per line
  u16* fq;
  float* red;
  int b, c, lw;  // butterfly, line of this thread
};

// The chunk of lines of a workgroup.  Workgroups go to the eight XCDs in turn,
// and each XCD has an L2 of its own: a run of a.xcd neighbouring chunks is given
// to each, so that the cache lines that two chunks share (runs start anywhere in
// a line of 128 bytes when Nx is no multiple of 16, and 16 bank entries are half a
// line) are fetched by one XCD and their stores merge there.  Forward +
// reconstruction with 42 orientations, chunks in turn and in runs: 256 x 192 x 192
// 3.63 and 3.46 ms, 64 x 320 x 320 2.52 and 2.42 ms, 128^3 601 and 600 us;
// processing of 120 x 100 x 90 309 and 296 us.
__device__ __forceinline__ int chunk_of(const TileArgs& a) {
  return a.xcd ? (int)(blockIdx.x & 7) * a.xcd + (int)(blockIdx.x >> 3) : (int)blockIdx.x;
}

// conj: the twiddles of the inverse direction (conjugated here, before the
// barrier: the first stage reads them where it joins two factors)
__device__ __forceinline__ LineTile line_tile(const TileArgs& a, float2* lds, bool conj = false) {
  const AxisT& z = a.y;
  LineTile t;
  t.lw = a.lw;
  t.c = threadIdx.x & ((1 << a.lw) - 1);
  t.b = threadIdx.x >> a.lw;
  t.buf = lds;
  t.tw = lds + ((z.N << a.lw) << a.two);
  t.ts = t.tw + z.N;
  t.fq = (u16*)(t.ts + (a.lb ? 1 << a.lw : 0));
  t.red = (float*)(t.fq + ((z.N + 1) & ~1));
  for (int i = threadIdx.x; i < z.N; i += blockDim.x) {
    t.tw[i] = conj ? cconj(z.tw[i]) : z.tw[i];
    t.fq[i] = (u16)freq_of(z, i);
  }
  if (a.lb) {
    const int w = a.lw - a.lb;
    for (int i = threadIdx.x; i < 1 << a.lw; i += blockDim.x) {
      const long long line = min(((long long)chunk_of(a) << w) + (i & ((1 << w) - 1)), a.lines - 1);
      t.ts[i] = a.x.tw[(int)line / a.p.Nx * (i >> w)];
    }
  }
  __syncthreads();
  return t;
}

// The thread's line and its offset in a z plane.  Split: line ka Nx + x of
// every class yb, at the row yb Ny / B + ka of the intermediate (and the row
// ka + kb Ny / B of the spectrum).
__device__ __forceinline__ bool line_of(const TileArgs& a, const LineTile& t, long long& col) {
  const int w = a.lw - a.lb;
  const long long line = ((long long)chunk_of(a) << w) + (t.c & ((1 << w) - 1));
  col = min(line, a.lines - 1) + (t.c >> w) * a.lines;
  return line < a.lines;
}

// Before the tile of the i-th pair is written: the other tile, whose reads
// ended before the barrier of the pair in between, or this one after a barrier.
// Two tiles let a wave go on to the next pair while others still transform
// this one (a stage of N / R butterflies leaves waves idle where the factors
// differ): 96 x 80 x 64 x 162, forward + reconstruction, with one tile 688 us, with
// two 679; processing of 120 x 100 x 90 x 42 301 and 296; 128^3 x 42 605 and 600.
__device__ __forceinline__ void next_tile(const TileArgs& a, const LineTile& t0, LineTile& t, int i) {
  if (a.two) {
    t.buf = t0.buf + (i & 1) * (a.y.N << a.lw);
    t.red = t0.red + (i & 1) * 16;
  } else {
    __syncthreads();
  }
}

// The stages between the first and the last factor are chosen at run time;
// the last factor RL is a template parameter of the kernels, because its
// butterflies' values live in registers across the stages.

// The thread's butterfly, opaque to the compiler: it otherwise moves the
// addresses of every radix out of the loop over the pairs and spills them.
__device__ __forceinline__ int butterfly(const LineTile& t) {
  int b = t.b;
  asm volatile("" : "+v"(b));
  return b;
}

// The thread's butterfly of the last factor.  Threads past the last one
// repeat the first (and store nothing): a branch around values that live
// across the stages would cost a second copy of them.
template <int RL>
__device__ __forceinline__ int last_butterfly(const AxisT& z, const LineTile& t) {
  const int b = butterfly(t);
  return b * RL < z.N ? b : 0;
}
template <int RL>
__device__ __forceinline__ bool has_last(const AxisT& z, const LineTile& t) {
  return butterfly(t) * RL < z.N;
}

// DIF of the tile: src(o) gives the thread's line at offset o = n dn (point n);
// out[r] receives frequency fq[b RL] + r N / RL of its last butterfly b.
// Offsets are a thread's base plus a scalar per value.  mid() runs after the
// first stage (its loads then don't hold registers next to that stage's).
// IN_LDS: the tile holds the values already.
template <bool INV, int RL, bool IN_LDS = false, class Src, class Mid>
__device__ __forceinline__ void line_dif(const AxisT& z, const LineTile& t, long long dn, Src src, Mid mid,
                                         float2 (&out)[RL]) {
  constexpr float sg = INV ? 1.f : -1.f;
  const int last = z.nst - 1, b = butterfly(t);
  if (last == 0) {
#pragma unroll
    for (int r = 0; r < RL; ++r) out[r] = IN_LDS ? t.buf[(r << t.lw) + t.c] : src(r * dn);
    dft_r<RL>(out, sg);
    mid();
    return;
  }
  if (b < z.S[0]) {
    with_radix(z.R[0], OS3D_RADIX_FN(rc) {
      constexpr int R = decltype(rc)::value;
      float2 v[R];
      const long long o = b * dn, step = z.S[0] * dn;
      float2* q = t.buf + (b << t.lw) + t.c;
      const int d = z.S[0] << t.lw;
#pragma unroll
      for (int r = 0; r < R; ++r) v[r] = IN_LDS ? q[r * d] : src(o + r * step);
      dft_r<R>(v, sg);
#pragma unroll
      for (int r = 0; r < R; ++r) q[r * d] = v[r];
    });
  }
  mid();
  __syncthreads();
  for (int i = 1; i < last; ++i) {
    const int S = z.S[i], u = fdiv(b, z.mS[i]), l = b - u * S;
    with_radix(z.R[i], OS3D_RADIX_FN(rc) {
      constexpr int R = decltype(rc)::value;
      if (u * R * S < z.N) {
        float2* q = t.buf + ((u * R * S + l) << t.lw) + t.c;
        const int d = S << t.lw;
        float2 v[R];
#pragma unroll
        for (int r = 0; r < R; ++r) v[r] = q[r * d];
        twiddle<R, INV>(v, t.tw, t.fq[u * R * S] * S);
        dft_r<R>(v, sg);
#pragma unroll
        for (int r = 0; r < R; ++r) q[r * d] = v[r];
      }
    });
    __syncthreads();
  }
  {
    const int p = last_butterfly<RL>(z, t) * RL;
    const float2* q = t.buf + (p << t.lw) + t.c;
    const int d = 1 << t.lw;
#pragma unroll
    for (int r = 0; r < RL; ++r) out[r] = q[r * d];
    twiddle<RL, INV>(out, t.tw, t.fq[p]);
    dft_r<RL>(out, sg);
  }
}

// DIT of the tile from the registers of the last factor's butterflies;
// sink(o, v) takes the value at offset o = n dn of the thread's line.  The
// caller synchronises before the tile's LDS is written again.  TO_LDS: the
// values stay in the tile, in natural order.
template <bool INV, int RL, bool TO_LDS = false, class Sink>
__device__ __forceinline__ void line_dit(const AxisT& z, const LineTile& t, long long dn, float2 (&in)[RL],
                                         Sink sink) {
  constexpr float sg = INV ? 1.f : -1.f;
  const int last = z.nst - 1, b = butterfly(t);
  dft_r<RL>(in, sg);
  if (b * RL < z.N) {
    if (!TO_LDS && last == 0) {
#pragma unroll
      for (int r = 0; r < RL; ++r) sink(r * dn, in[r]);
    } else {
      float2* q = t.buf + ((b * RL) << t.lw) + t.c;
      const int d = 1 << t.lw;
#pragma unroll
      for (int r = 0; r < RL; ++r) q[r * d] = in[r];
    }
  }
  for (int i = last - 1; i >= 0; --i) {
    __syncthreads();
    const int S = z.S[i], u = fdiv(b, z.mS[i]), l = b - u * S;
    with_radix(z.R[i], OS3D_RADIX_FN(rc) {
      constexpr int R = decltype(rc)::value;
      if (u * R * S < z.N) {
        float2* q = t.buf + ((u * R * S + l) << t.lw) + t.c;
        const int d = S << t.lw;
        float2 v[R];
#pragma unroll
        for (int r = 0; r < R; ++r) v[r] = q[r * d];
        twiddle<R, INV>(v, t.tw, l * z.tstep[i]);
        dft_r<R>(v, sg);
        if (!TO_LDS && i == 0) {
          const long long o = l * dn, step = S * dn;
#pragma unroll
          for (int r = 0; r < R; ++r) sink(o + r * step, v[r]);
        } else {
#pragma unroll
          for (int r = 0; r < R; ++r) q[r * d] = v[r];
        }
      }
    });
  }
}

// get(r, o) for the frequencies k of the thread's last-factor butterfly, at offsets o = k dn
template <int RL, class Get>
__device__ __forceinline__ void each_freq(const AxisT& z, const LineTile& t, long long dn, Get get) {
  const long long o = t.fq[last_butterfly<RL>(z, t) * RL] * dn, step = (z.N / RL) * dn;
#pragma unroll
  for (int r = 0; r < RL; ++r) get(r, o + r * step);
}

// f(integral_constant<B>) for the factor 2^lb of y
template <class F>
__device__ __forceinline__ void with_split(int lb, F f) {
  switch (lb) {
    case 1: f(std::integral_constant<int, 2>{}); break;
    case 2: f(std::integral_constant<int, 4>{}); break;
    default: f(std::integral_constant<int, 8>{}); break;
  }
}

// The factor B of the y axis on the tile of a split pass: y = yb + B ya, ky =
// ka + kb Ny / B.  split_out: the inverse DFT over kb -> yb and the twiddle, to
// memory; split_in: from memory, the twiddle and the DFT over yb -> kb.
__device__ __forceinline__ void split_out(const TileArgs& a, const LineTile& t, float2* T) {
  const int w = a.lw - a.lb, c = threadIdx.x & ((1 << w) - 1), nb = blockDim.x >> w;
  const long long line = ((long long)chunk_of(a) << w) + c;
  with_split(a.lb, OS3D_RADIX_FN(bc) {
    constexpr int B = decltype(bc)::value;
    for (int e = threadIdx.x >> w; e < a.y.N; e += nb) {
      const float2* q = t.buf + (e << t.lw) + c;
      float2 v[B];
#pragma unroll
      for (int r = 0; r < B; ++r) v[r] = q[r << w];
      dft_r<B>(v, 1.f);
#pragma unroll
      for (int r = 1; r < B; ++r) v[r] = cmulc(v[r], t.ts[(r << w) + c]);
      if (line < a.lines) {
#pragma unroll
        for (int r = 0; r < B; ++r) T[e * a.dn + r * a.lines + line] = v[r];
      }
    }
  });
}
__device__ __forceinline__ void split_in(const TileArgs& a, const LineTile& t, const float2* T) {
  const int w = a.lw - a.lb, c = threadIdx.x & ((1 << w) - 1), nb = blockDim.x >> w;
  const long long line = min(((long long)chunk_of(a) << w) + c, a.lines - 1);
  with_split(a.lb, OS3D_RADIX_FN(bc) {
    constexpr int B = decltype(bc)::value;
    for (int e = threadIdx.x >> w; e < a.y.N; e += nb) {
      float2 v[B];
#pragma unroll
      for (int r = 0; r < B; ++r) v[r] = ldnt(T + e * a.dn + r * a.lines + line);
#pragma unroll
      for (int r = 1; r < B; ++r) v[r] = cmul(v[r], t.ts[(r << w) + c]);
      dft_r<B>(v, -1.f);
      float2* q = t.buf + (e << t.lw) + c;
#pragma unroll
      for (int r = 0; r < B; ++r) q[r << w] = v[r];
    }
  });
}

// The DFT of f along z (f transformed along y and x), then for every pair:
// times the bank row, inverse DFT along z -> intermediate (complex64
// scores and processing; 16-bit scores: k_line_mul_seq).
template <int RL, bool SPLIT>
__global__ __launch_bounds__(1024) void k_line_mul(TileArgs a) {
  extern __shared__ float2 lds[];
  const PassArgs& p = a.p;
  const AxisT& z = a.y;
  if (chunk_of(a) >= a.chunks) return;
  const LineTile t0 = line_tile(a, lds);
  LineTile t = t0;
  long long col;
  const bool valid = line_of(a, t, col);
  float2 spec[RL];
#pragma unroll
  for (int r = 0; r < RL; ++r) spec[r] = make_float2(0.f, 0.f);
  line_dif<false>(z, t, a.dn, [&](long long o) { return p.src_c[o + col]; }, []() {}, spec);
  float ps[RL];
  const int j0 = (int)((long long)p.nb * blockIdx.y / a.groups);
  const int j1 = (int)((long long)p.nb * (blockIdx.y + 1) / a.groups);
  {
    const float* row = p.psi + (long long)p.rows[j0] * p.V + col;
    each_freq<RL>(z, t, a.dn, [&](int r, long long o) {
      ps[r] = row[o];
      spec[r] = cscale(spec[r], p.kappa);
    });
  }
  for (int j = j0; j < j1; ++j) {
    float2 v[RL];
#pragma unroll
    for (int r = 0; r < RL; ++r) v[r] = cscale(spec[r], ps[r]);
    if (j + 1 < j1) {
      const float* row = p.psi + (long long)p.rows[j + 1] * p.V + col;
      each_freq<RL>(z, t, a.dn, [&](int r, long long o) { ps[r] = row[o]; });
    }
    next_tile(a, t0, t, j - j0 + 1);  // (the DFT of f used the first one)
    if constexpr (SPLIT) {
      line_dit<true, RL, true>(z, t, a.dn, v, [](long long, float2) {});
      __syncthreads();
      split_out(a, t, p.dst_c + (long long)j * p.dst_stride);
    } else {
      float2* T = p.dst_c + (long long)j * p.dst_stride + col;
      line_dit<true>(z, t, a.dn, v, [&](long long o, float2 w) {
        if (valid) T[o] = w;
      });
    }
  }
}

// in *= kappa / max(M, eps) (kappa alone for the adjoint), then the inverse DFT along z -> dst.
template <int RL>
__device__ __forceinline__ void divide_inverse(const TileArgs& a, const LineTile& t, float2 (&x)[RL], long long col,
                                               bool valid) {
  const PassArgs& p = a.p;
  if (p.divide) {
    const float* M = p.M + col;
    each_freq<RL>(a.y, t, a.dn, [&](int r, long long o) { x[r] = cscale(x[r], p.kappa / fmaxf(M[o], p.eps)); });
  } else {
#pragma unroll
    for (int r = 0; r < RL; ++r) x[r] = cscale(x[r], p.kappa);
  }
  __syncthreads();
  float2* X = p.dst_c + col;
  line_dit<true>(a.y, t, a.dn, x, [&](long long o, float2 w) {
    if (valid) X[o] = w;
  });
}

// The first pair of group g.
__device__ __forceinline__ int group_begin(const TileArgs& a, int g) {
  return (int)((long long)a.p.nb * g / a.groups);
}

// DFT along z of every pair's intermediate, times its bank row, summed over
// the workgroup's share of the pairs.  With few lines the pairs of a launch
// are shared out to `groups` workgroups per tile: 64^3 x 21 pairs has 128 tiles
// for 256 CUs.  Group 0 sums into X, the others into the intermediate of their
// first pair, at the lines that the workgroup itself has read (k_line_div adds
// them up), so a shared sum takes no workspace of its own.
template <int RL, bool SPLIT>
__global__ __launch_bounds__(1024) void k_line_acc(TileArgs a) {
  extern __shared__ float2 lds[];
  const PassArgs& p = a.p;
  const AxisT& z = a.y;
  if (chunk_of(a) >= a.chunks) return;
  const LineTile t0 = line_tile(a, lds);
  LineTile t = t0;
  long long col;
  const bool valid = line_of(a, t, col);
  float2 acc[RL];
#pragma unroll
  for (int r = 0; r < RL; ++r) acc[r] = make_float2(0.f, 0.f);
  const int g = blockIdx.y;
  const int j0 = group_begin(a, g), j1 = group_begin(a, g + 1);
  for (int j = j0; j < j1; ++j) {
    const float* row = p.psi + (long long)p.rows[j] * p.V + col;
    const float2* T = p.src_c + (long long)j * p.src_stride + col;
    float ps[RL];
    float2 v[RL];
    if (j > j0) next_tile(a, t0, t, j - j0);
    if constexpr (SPLIT) {
      split_in(a, t, p.src_c + (long long)j * p.src_stride);
      __syncthreads();
    }
    line_dif<false, RL, SPLIT>(
        z, t, a.dn, [&](long long o) { return ldnt(T + o); },
        [&]() { each_freq<RL>(z, t, a.dn, [&](int r, long long o) { ps[r] = ldnt(row + o); }); }, v);
    each_freq<RL>(z, t, a.dn, [&](int r, long long) {
      acc[r] = make_float2(acc[r].x + ps[r] * v[r].x, acc[r].y + ps[r] * v[r].y);
    });
  }
  float2* X = (g == 0 ? p.dst_c : a.part + (long long)j0 * p.V) + col;
  if (p.accumulate && g == 0) each_freq<RL>(z, t, a.dn, [&](int r, long long o) { acc[r] = cadd(X[o], acc[r]); });
  if (a.finish) {
    divide_inverse(a, t, acc, col, valid);
  } else if (valid && has_last<RL>(z, t)) {
    each_freq<RL>(z, t, a.dn, [&](int r, long long o) { X[o] = acc[r]; });
  }
}

// The groups' orientation sums added up into X; finish: divided by M, inverse DFT along z.
template <int RL>
__global__ __launch_bounds__(1024) void k_line_div(TileArgs a) {
  extern __shared__ float2 lds[];
  const PassArgs& p = a.p;
  const LineTile t = line_tile(a, lds);
  long long col;
  const bool valid = line_of(a, t, col);
  float2 x[RL];
#pragma unroll
  for (int r = 0; r < RL; ++r) x[r] = make_float2(0.f, 0.f);
  each_freq<RL>(a.y, t, a.dn, [&](int r, long long o) { x[r] = p.src_c[o + col]; });
  for (int g = 1; g < a.groups; ++g) {
    const float2* X = a.part + (long long)group_begin(a, g) * p.V + col;
    each_freq<RL>(a.y, t, a.dn, [&](int r, long long o) { x[r] = cadd(x[r], X[o]); });
  }
  if (a.finish) {
    divide_inverse(a, t, x, col, valid);
  } else if (valid && has_last<RL>(a.y, t)) {
    each_freq<RL>(a.y, t, a.dn, [&](int r, long long o) { p.dst_c[o + col] = x[r]; });
  }
}

// DFT of the y lines of every pair's volume, in place or from src to dst (one
// tile per workgroup: taking the lines of several pairs through one workgroup
// measured slower, 780 -> 910 us at 180 x 240 x 216 x 21 pairs).
template <bool INV, int RL>
__global__ __launch_bounds__(1024) void k_line_y(TileArgs a) {
  extern __shared__ float2 lds[];
  const PassArgs& p = a.p;
  const AxisT& y = a.y;
  const LineTile t = line_tile(a, lds);
  const int zp = blockIdx.x / a.chunks, x = ((blockIdx.x - zp * a.chunks) << a.lw) + t.c;
  const bool valid = x < p.Nx;
  const long long col = (long long)zp * p.Ny * p.Nx + (valid ? x : p.Nx - 1);
  const float2* src = p.src_c + (long long)blockIdx.y * p.src_stride + col;
  float2* dst = p.dst_c + (long long)blockIdx.y * p.dst_stride + col;
  float2 v[RL];
  line_dif<INV>(y, t, a.dn, [&](long long o) { return ldnt(src + o); }, []() {}, v);
  if (y.nst > 1) __syncthreads();
  if (valid && has_last<RL>(y, t)) each_freq<RL>(y, t, a.dn, [&](int r, long long o) { dst[o] = v[r]; });
}

// ---------------------------------------------------------------- 16-bit scores
// The same passes in the sequential order (fft_tile.h), DIF in both
// directions.

// Stages after the first; sink(o, v) takes frequency k at offset o = k dn, or,
// TO_LDS, the tile keeps the values at their digit-reversed positions.
template <bool TO_LDS, class Sink>
__device__ __forceinline__ void line_seq_rest(const AxisT& z, const LineTile& t, long long dn, float sgn, Sink sink) {
  const int nbt = blockDim.x >> t.lw;
  for (int i = 1; i < z.nst; ++i) {
    __syncthreads();
    const int S = z.S[i];
    const bool last = i == z.nst - 1;
    with_seq(z.R[i], z.RB[i], OS3D_SEQ_FN(rc, rb) {
      constexpr int R = decltype(rc)::value, RB = decltype(rb)::value;
      for (int b = butterfly(t); b < z.nb[i]; b += nbt) {
        const int u = fdiv(b, z.mS[i]), l = b - u * S;
        float2* q = t.buf + ((u * R * S + l) << t.lw) + t.c;
        const int d = S << t.lw, f = t.fq[u * R * S];
        float2 v[R];
#pragma unroll
        for (int r = 0; r < R; ++r) v[r] = q[r * d];
        seq_butterfly<R, RB>(v, t.tw, f, S, z.tstep[i], false, sgn);
        if (TO_LDS || !last) {
#pragma unroll
          for (int r = 0; r < R; ++r) q[r * d] = v[r];
        } else {
          const long long o = f * dn, step = z.tstep[i] * dn;
#pragma unroll
          for (int r = 0; r < R; ++r) sink(o + seq_slot<R, RB>(r) * step, v[r]);
        }
      }
    });
  }
}

// Conjugates the tile's twiddles: the caller has a barrier before it (earlier
// stages read them) and one after it (so does the next stage, the first too
// where it joins two factors).
__device__ __forceinline__ void conj_twiddles(const AxisT& z, const LineTile& t) {
  for (int i = threadIdx.x; i < z.N; i += blockDim.x) t.tw[i].y = -t.tw[i].y;
}

// k_line_mul for 16-bit scores, with the sums of |value| of their scale
// bound.  (R0, RB0): the first stage, whose inputs (the tile's spectrum) stay
// in registers over the pairs.
template <int R0, int RB0>
__global__ __launch_bounds__(1024) void k_line_mul_seq(TileArgs a) {
  extern __shared__ float2 lds[];
  const PassArgs& p = a.p;
  const AxisT& z = a.y;
  const LineTile t0 = line_tile(a, lds);
  LineTile t = t0;
  u16* pos = (u16*)(t.red + 32);  // position of a frequency
  for (int i = threadIdx.x; i < z.N; i += blockDim.x) pos[t.fq[i]] = (u16)i;
  const long long line = ((long long)blockIdx.x << a.lw) + t.c;
  const bool valid = line < a.lines;
  const long long col = valid ? line : a.lines - 1;
  const bool first = t.b < z.S[0];
  const int b0 = first ? t.b : 0;
  float2 spec[R0];
  const long long o0 = b0 * a.dn, step0 = z.S[0] * a.dn;
#pragma unroll
  for (int r = 0; r < R0; ++r) spec[r] = p.src_c[o0 + r * step0 + col];
  seq_butterfly<R0, RB0>(spec, t.tw, 0, z.S[0], 1, true, -p.sgn);
  const int d0 = z.S[0] << t.lw, q0 = (b0 << t.lw) + t.c;
  if (first) {
#pragma unroll
    for (int r = 0; r < R0; ++r) t.buf[q0 + r * d0] = spec[r];
  }
  line_seq_rest<true>(z, t, a.dn, -p.sgn, [](long long, float2) {});
  __syncthreads();
#pragma unroll
  for (int r = 0; r < R0; ++r) spec[r] = t.buf[(pos[b0 + r * z.S[0]] << t.lw) + t.c];
  conj_twiddles(z, t);
  if (a.two) __syncthreads();
  const int j0 = (int)((long long)p.nb * blockIdx.y / a.groups);
  const int j1 = (int)((long long)p.nb * (blockIdx.y + 1) / a.groups);
  float ps[R0];
  {
    const float* row = p.psi + (long long)p.rows[j0] * p.V + col;
#pragma unroll
    for (int r = 0; r < R0; ++r) ps[r] = row[o0 + r * step0];
  }
  for (int j = j0; j < j1; ++j) {
    float2 v[R0];
#pragma unroll
    for (int r = 0; r < R0; ++r) {
      v[r] = cscale(spec[r], ps[r] * p.kappa);
      hold(v[r]);
    }
    if (j + 1 < j1) {
      const float* row = p.psi + (long long)p.rows[j + 1] * p.V + col;
#pragma unroll
      for (int r = 0; r < R0; ++r) ps[r] = row[o0 + r * step0];
    }
    // the hardware square root (1 ulp) is ample for a bound that is rounded
    // up to a power of two
    float s = 0.f;
#pragma unroll
    for (int r = 0; r < R0; ++r) s += __builtin_amdgcn_sqrtf(v[r].x * v[r].x + v[r].y * v[r].y);
    if (!valid || !first) s = 0.f;
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
    next_tile(a, t0, t, j - j0 + 1);  // and red
    if ((threadIdx.x & 63) == 0) t.red[threadIdx.x >> 6] = s;
    seq_butterfly<R0, RB0>(v, t.tw, 0, z.S[0], 1, true, p.sgn);
    float2* T = p.dst_c + (long long)j * p.dst_stride + col;
    if (z.nst > 1) {
      if (first) {
#pragma unroll
        for (int r = 0; r < R0; ++r) t.buf[q0 + r * d0] = v[r];
      }
    } else if (first && valid) {
#pragma unroll
      for (int r = 0; r < R0; ++r) T[seq_slot<R0, RB0>(r) * a.dn] = v[r];
    }
    line_seq_rest<false>(z, t, a.dn, p.sgn, [&](long long o, float2 w) {
      if (valid) T[o] = w;
    });
    if (z.nst == 1) __syncthreads();
    if (threadIdx.x == 0) {
      float sum = 0.f;
      for (int w = 0; w < (int)(blockDim.x >> 6); ++w) sum += t.red[w];
      p.partial[(long long)j * gridDim.x + blockIdx.x] = sum;
    }
  }
}

// DFT of the y lines of every pair's volume, in place or from src to dst.
__global__ __launch_bounds__(1024) void k_line_y_seq(TileArgs a) {
  extern __shared__ float2 lds[];
  const PassArgs& p = a.p;
  const AxisT& y = a.y;
  const LineTile t = line_tile(a, lds, p.sgn > 0.f);
  const int zp = blockIdx.x / a.chunks, x = ((blockIdx.x - zp * a.chunks) << a.lw) + t.c;
  const bool valid = x < p.Nx;
  const long long col = (long long)zp * p.Ny * p.Nx + (valid ? x : p.Nx - 1);
  const float2* src = p.src_c + (long long)blockIdx.y * p.src_stride + col;
  float2* dst = p.dst_c + (long long)blockIdx.y * p.dst_stride + col;
  if (t.b < y.S[0]) {
    with_seq(y.R[0], y.RB[0], OS3D_SEQ_FN(rc, rb) {
      constexpr int R = decltype(rc)::value, RB = decltype(rb)::value;
      float2 v[R];
      const long long o = t.b * a.dn, step = y.S[0] * a.dn;
#pragma unroll
      for (int r = 0; r < R; ++r) v[r] = ldnt(src + o + r * step);
      seq_butterfly<R, RB>(v, t.tw, 0, y.S[0], 1, true, p.sgn);
      if (y.nst > 1) {
        float2* q = t.buf + (t.b << t.lw) + t.c;
        const int d = y.S[0] << t.lw;
#pragma unroll
        for (int r = 0; r < R; ++r) q[r * d] = v[r];
      } else if (valid) {
#pragma unroll
        for (int r = 0; r < R; ++r) dst[seq_slot<R, RB>(r) * a.dn] = v[r];
      }
    });
  }
  line_seq_rest<false>(y, t, a.dn, p.sgn, [&](long long o, float2 w) {
    if (valid) dst[o] = w;
  });
}

// ---------------------------------------------------------------- host side
// Raises the dynamic-LDS limit of a kernel once.
static void reserve_lds(const void* kernel) {
  static std::mutex mu;
  static std::set<const void*> done;
  std::lock_guard<std::mutex> lock(mu);
  if (done.insert(kernel).second)
    (void)hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
}

static int check_line(const char* what) {
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) {
    set_error(std::string(what) + ": " + hipGetErrorString(e));
    return OS3D_EDEVICE;
  }
  return OS3D_OK;
}

struct LinePlan {
  int lw, threads, two;
  size_t lds;
  // workgroups that keep the chip busy: eight waves per CU (forward +
  // reconstruction with them and with thirty-two: 64^3 x 42 96 and 99.5 us, 128^3 x
  // 42 600 and 621, 96 x 80 x 64 x 162 679 and 693)
  long long fill() const { return 256LL * 512 / threads; }
};

template <class K>
static void launch_line(K kernel, dim3 grid, const LinePlan& q, const TileArgs& a, hipStream_t st) {
  reserve_lds((const void*)kernel);
  launch_k(kernel, grid, dim3(q.threads), (unsigned)q.lds, st, a);
}

// Lines per workgroup: as many as fill 512 threads with one butterfly each
// (up to 64 KB of tile, two workgroups per CU), at least runs of 16 values
// where 1024 threads allow; down to runs of 32 values while the grid is smaller
// than two workgroups per CU.  Shorter runs cost more than the idle CUs they
// fill: down to runs of 16 values forward + reconstruction of 64^3 x 42 takes 98.5
// us instead of 96, processing of 96 x 80 x 64 x 162 477 instead of 455.
static LinePlan line_plan(const AxisT& z, long long lines) {
  int rmin = 16;
  for (int i = 0; i < z.nst; ++i) rmin = std::min(rmin, z.R[i]);
  const int nbf = z.N / rmin;
  int lw = 0;
  while (lw < 8 && (2 << lw) * nbf <= 512 && (2 << lw) * z.N <= 8192) ++lw;
  while (lw < 4 && (2 << lw) * nbf <= 1024 && (2 << lw) * z.N <= 8192) ++lw;
  while (lw > 5 && ((lines + (1 << lw) - 1) >> lw) < 512) --lw;
  LinePlan q;
  q.lw = lw;
  q.threads = std::min(1024, ((nbf << lw) + 63) / 64 * 64);
  const size_t tile = ((size_t)z.N << lw) * 8, tables = (size_t)z.N * 8 + (size_t)((z.N + 1) & ~1) * 4 + 128;
  // a second tile where two workgroups still share a CU
  q.two = (z.nst > 1 && 2 * (2 * tile + tables) <= 160 * 1024) ? 1 : 0;
  q.lds = (tile << q.two) + tables;
  return q;
}

// Split passes (p.split = B): tiles of B classes x W lines, W = 32, or 16 where
// the LDS or 1024 threads don't hold that (100 x 180 x 180 x 42, B = 2, forward +
// reconstruction: 1.29 ms with 32, 1.43 with 16).  Runs of 8 lose what the pass
// over y costs: 256 x 192 x 192 x 42 takes 4.03 ms with them, 4.01 in three passes
// and 3.48 with runs of 16.
static bool split_plan(const AxisT& z, int B, LinePlan& q, int& lb) {
  int rmin = 16;
  for (int i = 0; i < z.nst; ++i) rmin = std::min(rmin, z.R[i]);
  const int nbf = z.N / rmin;
  for (lb = 0; (1 << lb) < B;) ++lb;
  for (int w = 5; w >= 4; --w) {
    q.lw = lb + w;
    q.threads = ((nbf << q.lw) + 63) / 64 * 64;
    const size_t tile = ((size_t)z.N << q.lw) * 8;
    const size_t tables = (size_t)z.N * 8 + ((size_t)8 << q.lw) + (size_t)((z.N + 1) & ~1) * 4 + 128;
    q.two = (z.nst > 1 && 2 * (2 * tile + tables) <= 160 * 1024) ? 1 : 0;
    q.lds = (tile << q.two) + tables;
    if (q.threads <= 1024 && q.lds <= 160 * 1024) return true;
  }
  return false;
}

// The smallest B = 2, 4, 8 that leaves planes of Ny / B rows in LDS.  The next
// larger one trades wider z-line tiles for smaller planes, within a few percent
// (forward + reconstruction with 42 orientations: 100 x 180 x 180 1.27 ms with B = 2
// and 1.25 with 4, 100 x 160 x 180 1.11 and 1.08, 64 x 192 x 192 900 us with B = 4 and
// 894 with 8).  None: the pairs take three passes (z lines, y lines, x lines).
int split_factor(int Nz, int Ny, int Nx) {
  for (int B = 2; B <= 8; B *= 2) {
    LinePlan q;
    int lb;
    if (Ny % B == 0 && plane_fits(Ny / B, Nx) && split_plan(make_axis(Nz, nullptr), B, q, lb)) return B;
  }
  return 0;
}

static TileArgs zline_args(const os3d_bank* b, const PassArgs& p, LinePlan& q, bool seq = false) {
  TileArgs a = {};
  a.p = p;
  a.y = seq ? make_axis_seq((int)b->dims[0], b->d.tw[0]) : make_axis((int)b->dims[0], b->d.tw[0]);
  a.lines = b->dims[1] * b->dims[2];
  a.dn = a.lines;
  if (p.split) {
    split_plan(a.y, p.split, q, a.lb);
    a.lines /= p.split;
    a.x.tw = (const float2*)b->d.tw[1];
  } else {
    q = line_plan(a.y, a.lines);
  }
  a.lw = q.lw;
  a.two = q.two;
  a.chunks = (int)((a.lines + (1LL << (q.lw - a.lb)) - 1) >> (q.lw - a.lb));
  a.groups = 1;
  return a;
}

int zline_tiles(const os3d_bank* b) {
  LinePlan q;
  return zline_args(b, PassArgs{}, q, true).chunks;
}

// With fewer tiles than fill the chip the pairs of a launch are shared out, at
// least three to a workgroup (each share costs a volume written and read).
int zline_acc_groups(const os3d_bank* b, int nb) {
  LinePlan q;
  PassArgs p = {};
  p.split = b->split;
  const TileArgs a = zline_args(b, p, q);
  return (int)std::max(1LL, std::min<long long>(std::min(8, nb / 3), q.fill() / a.chunks));
}

static int xcd_share(const TileArgs& a) { return (a.chunks + 7) / 8; }

int launch_zline_mul(const os3d_bank* b, const PassArgs& p, hipStream_t st) {
  LinePlan q;
  const bool seq = p.partial != nullptr;
  TileArgs a = zline_args(b, p, q, seq);
  // the forward DFT is repeated by every workgroup of a tile: share the
  // pairs only as far as it takes to fill the chip
  a.groups = (int)std::max(1LL, std::min<long long>(p.nb, (q.fill() + a.chunks - 1) / a.chunks));
  if (!seq) a.xcd = xcd_share(a);
  const dim3 grid((unsigned)(seq ? a.chunks : 8 * a.xcd), (unsigned)a.groups);
  if (seq)
    with_seq(a.y.R[0], a.y.RB[0], [&](auto rc, auto rb) {
      launch_line(k_line_mul_seq<decltype(rc)::value, decltype(rb)::value>, grid, q, a, st);
    });
  else
    with_radix(a.y.R[a.y.nst - 1], [&](auto rc) {
      constexpr int RL = decltype(rc)::value;
      launch_line(p.split ? k_line_mul<RL, true> : k_line_mul<RL, false>, grid, q, a, st);
    });
  return check_line("k_line_mul");
}

int launch_zline_acc(const os3d_bank* b, const PassArgs& p, float2* T, int groups, bool finish, hipStream_t st) {
  LinePlan q;
  TileArgs a = zline_args(b, p, q);
  a.groups = groups;
  a.part = T;
  a.finish = finish ? 1 : 0;
  a.xcd = xcd_share(a);
  const dim3 grid((unsigned)(8 * a.xcd), (unsigned)a.groups);
  with_radix(a.y.R[a.y.nst - 1], [&](auto rc) {
    constexpr int RL = decltype(rc)::value;
    launch_line(p.split ? k_line_acc<RL, true> : k_line_acc<RL, false>, grid, q, a, st);
  });
  return check_line("k_line_acc");
}

int launch_zline_div(const os3d_bank* b, const PassArgs& p, float2* T, int groups, bool finish, hipStream_t st) {
  LinePlan q;
  TileArgs a = zline_args(b, p, q);
  a.groups = groups;
  a.part = T;
  a.finish = finish ? 1 : 0;
  const dim3 grid((unsigned)a.chunks);
  with_radix(a.y.R[a.y.nst - 1], [&](auto rc) { launch_line(k_line_div<decltype(rc)::value>, grid, q, a, st); });
  return check_line("k_line_div");
}

int launch_yline(const os3d_bank* b, const PassArgs& p, bool seq, hipStream_t st) {
  TileArgs a = {};
  a.p = p;
  a.y = seq ? make_axis_seq((int)b->dims[1], b->d.tw[1]) : make_axis((int)b->dims[1], b->d.tw[1]);
  a.dn = b->dims[2];
  a.lines = b->dims[0] * b->dims[2];
  LinePlan q = line_plan(a.y, a.lines);
  if (q.two) q.lds -= ((size_t)a.y.N << q.lw) * 8;  // one pair per workgroup
  a.lw = q.lw;
  a.chunks = (int)((b->dims[2] + (1LL << q.lw) - 1) >> q.lw);
  const long long tiles = a.chunks * b->dims[0];
  const dim3 grid((unsigned)tiles, (unsigned)p.nb);
  if (seq) {
    launch_line(k_line_y_seq, grid, q, a, st);
    return check_line("k_line_y_seq");
  }
  with_radix(a.y.R[a.y.nst - 1], [&](auto rc) {
    constexpr int RL = decltype(rc)::value;
    launch_line(p.sgn > 0.f ? k_line_y<true, RL> : k_line_y<false, RL>, grid, q, a, st);
  });
  return check_line("k_line_y");
}

}  // namespace os3d
