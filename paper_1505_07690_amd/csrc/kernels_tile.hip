// Whole-plane and x-line passes of the general transform (stages:
// fft_tile.h).  A tile is a run of rows of Nx consecutive values: one or
// more whole (y, x) planes, transformed along both axes while they sit in
// LDS (one round trip of the intermediate instead of two), or, for planes
// larger than LDS, rows transformed along x alone.
//
// The tile is loaded linearly (fully coalesced) with the fused load of the
// pass; the x stages run with consecutive lanes on consecutive rows (the row
// stride is odd, so a wave's accesses fall on distinct banks and its
// twiddles are broadcasts), the y stages with consecutive lanes on
// consecutive x.  The rows end digit-reversed: the last y stage (or the
// store loop) reads them in natural order through a table and stores straight
// to memory with consecutive lanes on consecutive x; an odd last x factor, or
// one value of padding after every even one, keeps those reads off each
// other's banks.  Workgroups loop over (pair, tile) tasks and issue the next
// task's loads before transforming the current one, except complex64 score
// pairs, whose two members do not fit the registers beside the transform.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <mutex>
#include <set>

#include "fft_tile.h"
#include "launch.h"

namespace os3d {

typedef unsigned short u16;

// Stages of the balanced or (SEQ) the sequential schedule: f(R, RB).
template <bool SEQ, class Fn>
__device__ __forceinline__ void with_stage(const AxisT& x, int i, Fn f) {
  if constexpr (SEQ)
    with_seq(x.R[i], x.RB[i], f);
  else
    with_radix(x.R[i], [&](auto rc) __attribute__((always_inline)) { f(rc, std::integral_constant<int, 1>{}); });
}

// The tile and the tables of a workgroup.
struct TileLds {
  float2* buf;
  float2 *twx, *twy;
  u16* xl;  // natural x -> position in the row
  u16* xs;  // frequency kx -> position in the row after the DIF
  u16* fx;  // frequency at a DIF position (without padding)
  u16* fy;
  u16* ys;  // SEQ: frequency ky -> row after the DIF
};

// conj: the twiddles of the inverse direction
template <bool PLANE, bool SEQ>
__device__ __forceinline__ TileLds tile_lds(const TileArgs& a, float2* lds, bool conj) {
  TileLds t;
  t.buf = lds;
  t.twx = lds + a.rows * a.RS;
  t.twy = t.twx + a.x.N;
  t.xl = (u16*)(t.twy + (PLANE ? a.y.N : 0));
  t.xs = t.xl + a.x.N;
  t.fx = t.xs + a.x.N;
  t.fy = t.fx + a.x.N;
  t.ys = t.fy + (PLANE ? a.y.N : 0);
  for (int i = threadIdx.x; i < a.x.N; i += blockDim.x) {
    t.twx[i] = conj ? cconj(a.x.tw[i]) : a.x.tw[i];
    const int q = i + fdiv(i, a.mRL) * a.pad, f = freq_of(a.x, i);
    t.xl[i] = (u16)q;
    t.xs[f] = (u16)q;
    t.fx[i] = (u16)f;
  }
  if constexpr (PLANE) {
    for (int i = threadIdx.x; i < a.y.N; i += blockDim.x) {
      const int f = freq_of(a.y, i);
      t.twy[i] = conj ? cconj(a.y.tw[i]) : a.y.tw[i];
      t.fy[i] = (u16)f;
      if constexpr (SEQ) t.ys[f] = (u16)i;
    }
  }
  __syncthreads();
  return t;
}

// Stage i of the rows, in place.
template <bool SEQ, bool INV, bool DIT, bool REAL = false>
__device__ __forceinline__ void x_stage(const TileArgs& a, const TileLds& t, int i) {
  const AxisT& x = a.x;
  const int S = x.S[i];
  const bool last = i == x.nst - 1;
  // strides in LDS: RL + pad values per RL positions
  const int Sp = last ? 1 : S + fdiv(S, a.mRL) * a.pad;
  with_stage<SEQ>(x, i, OS3D_SEQ_FN(rc, rb) {
    constexpr int R = decltype(rc)::value, RB = decltype(rb)::value;
    const int block = last ? R + a.pad : R * Sp, total = a.rows * x.nb[i];
    for (int id = threadIdx.x; id < total; id += blockDim.x) {
      const int b = fdiv(id, a.mrows), row = id - b * a.rows;
      const int u = fdiv(b, x.mS[i]), l = b - u * S;
      float2* q = t.buf + row * a.RS + u * block + l + fdiv(l, a.mRL) * a.pad;
      float2 v[R];
#pragma unroll
      for (int r = 0; r < R; ++r) v[r] = q[r * Sp];
      if constexpr (SEQ) {
        seq_butterfly<R, RB, REAL>(v, t.twx, t.fx[u * R * S], S, x.tstep[i], i == 0, a.p.sgn);
      } else {
        if (DIT ? !last : i > 0) twiddle<R, INV>(v, t.twx, DIT ? l * x.tstep[i] : t.fx[u * R * S] * S);
        dft_r<R>(v, INV ? 1.f : -1.f);
      }
#pragma unroll
      for (int r = 0; r < R; ++r) q[r * Sp] = v[r];
    }
  });
}

// Stage i of the columns: fn(R, RB, v, q, d, pos, col, plane) takes the
// transformed butterfly at row position pos of column col (LDS address q,
// stride d).  Columns go by position in the row (xl), or in the order of
// their frequencies (NATURAL).
template <bool SEQ, bool INV, bool DIT, bool NATURAL, class Fn>
__device__ __forceinline__ void y_stage(const TileArgs& a, const TileLds& t, int i, Fn fn) {
  const AxisT& y = a.y;
  const int S = y.S[i];
  const bool last = i == y.nst - 1;
  with_stage<SEQ>(y, i, OS3D_SEQ_FN(rc, rb) {
    constexpr int R = decltype(rc)::value, RB = decltype(rb)::value;
    const int total = a.P * y.nb[i] * a.x.N;
    for (int id = threadIdx.x; id < total; id += blockDim.x) {
      const int e = fdiv(id, a.mNx), col = id - e * a.x.N;
      const int b = fdiv(e, a.mP), plane = e - b * a.P;
      const int u = fdiv(b, y.mS[i]), l = b - u * S;
      float2* q = t.buf + (plane * a.A + u * R * S + l) * a.RS + (NATURAL ? t.xs : t.xl)[col];
      const int d = S * a.RS;
      float2 v[R];
#pragma unroll
      for (int r = 0; r < R; ++r) v[r] = q[r * d];
      if constexpr (SEQ) {
        seq_butterfly<R, RB>(v, t.twy, t.fy[u * R * S], S, y.tstep[i], i == 0, a.p.sgn);
      } else {
        if (DIT ? !last : i > 0) twiddle<R, INV>(v, t.twy, DIT ? l * y.tstep[i] : t.fy[u * R * S] * S);
        dft_r<R>(v, INV ? 1.f : -1.f);
      }
      fn(rc, rb, v, q, d, u * R * S, col, plane);
    }
  });
}

struct KeepInLds {
  template <class RC, class RB>
  __device__ __forceinline__ void operator()(RC, RB, const float2* v, float2* q, int d, int, int, int) const {
#pragma unroll
    for (int r = 0; r < RC::value; ++r) q[r * d] = v[r];
  }
};

// The thread's values tid + i T of a tile: raw loads, converted when they are used.
template <int LM, int DT, int VPT>
struct TileIn {
  static constexpr bool kPair = LM == LM_UIN;
  static constexpr bool kPrefetch = !(LM == LM_UIN && DT == OS3D_C64);
  using Word = typename std::conditional<LM == LM_REAL, float,
                                         typename std::conditional<kPair && DT != OS3D_C64, unsigned int,
                                                                   float2>::type>::type;
  Word r[VPT], s[kPair ? VPT : 1];
  bool both;
  float sa, sb;

  // n values of the tile at g0 of pair j; only the first nval exist
  __device__ __forceinline__ void issue(const PassArgs& p, int j, long long g0, int n, int nval) {
    const Word *wr, *ws = nullptr;
    both = false;
    if constexpr (LM == LM_REAL) {
      wr = p.src_r + g0;
    } else if constexpr (LM == LM_C) {
      wr = p.src_c + j * p.src_stride + g0;
    } else {
      const int ia = p.oa[j], ib = p.ob[j];
      both = ib >= 0;
      wr = (const Word*)p.U + (long long)ia * p.V + g0;
      ws = (const Word*)p.U + (long long)(both ? ib : ia) * p.V + g0;
      if constexpr (DT != OS3D_C64) {
        sa = p.scales[ia];
        sb = both ? p.scales[ib] : 0.f;
      }
    }
    const int T = blockDim.x;
#pragma unroll
    for (int i = 0; i < VPT; ++i)
      if (i * T < n) r[i] = ldnt(wr + min((int)threadIdx.x + i * T, nval - 1));
    if constexpr (kPair) {
      if (both) {
#pragma unroll
        for (int i = 0; i < VPT; ++i)
          if (i * T < n) s[i] = ldnt(ws + min((int)threadIdx.x + i * T, nval - 1));
      }
    }
  }
  __device__ __forceinline__ static float2 val(Word w, float sc) {
    if constexpr (LM == LM_REAL) return make_float2(w, 0.f);
    else if constexpr (kPair && DT != OS3D_C64) return score_value<DT>(w, sc);
    else return w;
  }
  __device__ __forceinline__ void put(const TileArgs& a, const TileLds& t, int n) const {
    const int T = blockDim.x;
#pragma unroll
    for (int i = 0; i < VPT; ++i) {
      const int e = threadIdx.x + i * T;
      if (e < n) {
        float2 v = val(r[i], sa);
        if constexpr (kPair) {
          if (both) v = cadd(v, cconj(val(s[i], sb)));
        }
        const int row = fdiv(e, a.mNx), x = e - row * a.x.N;
        t.buf[row * a.RS + t.xl[x]] = v;
      }
    }
  }
};

// SEQ: the sequential order of the forward transform into 16-bit scores (x
// before y on the way to the spectrum, y before x on the way back).
template <int LM, int SM, int DT, bool PLANE, bool SEQ, int VPT>
__global__ __launch_bounds__(1024) void k_tile(TileArgs a) {
  constexpr bool INV = SM == SM_UOUT || SM == SM_REAL;  // the other stores end a forward DFT
  constexpr bool kYFirst = PLANE && SEQ && INV;
  extern __shared__ float2 lds[];
  const PassArgs& p = a.p;
  const TileLds t = tile_lds<PLANE, SEQ>(a, lds, SEQ && INV);
  const int n = a.rows * a.x.N;
  const long long ntask = a.tiles * p.nb;
  using In = TileIn<LM, DT, VPT>;
  In in;
  auto issue = [&](long long task) {
    const int j = (int)(task / a.tiles);
    const long long g0 = (task - j * a.tiles) * n;
    in.issue(p, j, g0, n, (int)min((long long)n, p.V - g0));
  };
  long long task = blockIdx.x;
  if (In::kPrefetch) issue(task);
  for (; task < ntask; task += gridDim.x) {
    const int j = (int)(task / a.tiles);
    const long long g0 = (task - j * a.tiles) * n;
    if (!In::kPrefetch) issue(task);
    in.put(a, t, n);
    if (In::kPrefetch && task + gridDim.x < ntask) issue(task + gridDim.x);
    __syncthreads();
    if constexpr (kYFirst) {
      for (int i = 0; i < a.y.nst; ++i) {
        y_stage<SEQ, INV, false, false>(a, t, i, KeepInLds{});
        __syncthreads();
      }
    }
    for (int i = 0; i < a.x.nst; ++i) {
      x_stage<SEQ, INV, false, LM == LM_REAL>(a, t, i);
      __syncthreads();
    }
    if constexpr (PLANE && !kYFirst) {
      const int last = a.y.nst - 1;
      for (int i = 0; i < last; ++i) {
        y_stage<SEQ, INV, false, false>(a, t, i, KeepInLds{});
        __syncthreads();
      }
      y_stage<SEQ, INV, false, true>(
          a, t, last, [&](auto rc, auto rb, const float2* v, float2*, int, int pos, int col, int plane) {
            constexpr int R = decltype(rc)::value, RB = decltype(rb)::value;
            const long long g = g0 + (plane * a.A + t.fy[pos]) * a.x.N + col, dn = (long long)(a.A / R) * a.x.N;
            float2 u[R], dummy[R];
#pragma unroll
            for (int r = 0; r < R; ++r) u[seq_slot<R, RB>(r)] = v[r];
            store_k<SM, DT, R>(p, j, g, dn, u, dummy);
          });
    } else {
      // row by row in natural order
      const int nval = (int)min((long long)n, p.V - g0);
      for (int e = threadIdx.x; e < nval; e += blockDim.x) {
        const int row = fdiv(e, a.mNx), x = e - row * a.x.N;
        int lrow = row;
        if constexpr (kYFirst) {
          const int plane = fdiv(row, a.mA);
          lrow = plane * a.A + t.ys[row - plane * a.A];
        }
        float2 u[1] = {t.buf[lrow * a.RS + t.xs[x]]}, dummy[1];
        store_k<SM, DT, 1>(p, j, g0 + e, 0, u, dummy);
      }
    }
    __syncthreads();  // the tile is rewritten by the next task
  }
}

// Processing via scores, both directions in one kernel and in place: inverse
// DFT of the tile, Phi on the scores, forward DFT.  The scores stay in
// digit-reversed order in between (DIF, Phi in the registers of its last
// stage, DIT).
template <bool PLANE, int VPT>
__global__ __launch_bounds__(1024) void k_tile_phi(TileArgs a) {
  extern __shared__ float2 lds[];
  const PassArgs& p = a.p;
  const TileLds t = tile_lds<PLANE, false>(a, lds, false);
  const int n = a.rows * a.x.N;
  const long long ntask = a.tiles * p.nb;
  using In = TileIn<LM_C, OS3D_C64, VPT>;
  In in;
  auto issue = [&](long long task) {
    const int j = (int)(task / a.tiles);
    const long long g0 = (task - j * a.tiles) * n;
    in.issue(p, j, g0, n, (int)min((long long)n, p.V - g0));
  };
  long long task = blockIdx.x;
  issue(task);
  const int lx = a.x.nst - 1;
  for (; task < ntask; task += gridDim.x) {
    const int j = (int)(task / a.tiles);
    const long long g0 = (task - j * a.tiles) * n;
    in.put(a, t, n);
    if (task + gridDim.x < ntask) issue(task + gridDim.x);
    __syncthreads();
    for (int i = 0; i <= lx; ++i) {
      x_stage<false, true, false>(a, t, i);
      __syncthreads();
    }
    if constexpr (PLANE) {
      const int ly = a.y.nst - 1;
      for (int i = 0; i < ly; ++i) {
        y_stage<false, true, false, false>(a, t, i, KeepInLds{});
        __syncthreads();
      }
      y_stage<false, true, false, false>(a, t, ly, [&](auto rc, auto, const float2* v, float2* q, int d, int, int, int) {
        constexpr int R = decltype(rc)::value;
        float2 u[R];
#pragma unroll
        for (int r = 0; r < R; ++r) u[r] = phi_apply(p, j, v[r]);
        dft_r<R>(u, -1.f);
#pragma unroll
        for (int r = 0; r < R; ++r) q[r * d] = u[r];
      });
      __syncthreads();
      for (int i = ly - 1; i >= 0; --i) {
        y_stage<false, false, true, false>(a, t, i, KeepInLds{});
        __syncthreads();
      }
    } else {
      for (int e = threadIdx.x; e < n; e += blockDim.x) {
        const int row = fdiv(e, a.mNx), x = e - row * a.x.N;
        float2* q = t.buf + row * a.RS + t.xl[x];
        *q = phi_apply(p, j, *q);
      }
      __syncthreads();
    }
    for (int i = lx; i >= 0; --i) {
      x_stage<false, false, true>(a, t, i);
      __syncthreads();
    }
    const int nval = (int)min((long long)n, p.V - g0);
    float2* dst = p.dst_c + j * p.dst_stride + g0;
    for (int e = threadIdx.x; e < nval; e += blockDim.x) {
      const int row = fdiv(e, a.mNx), x = e - row * a.x.N;
      dst[e] = t.buf[row * a.RS + t.xl[x]];
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------- host side
constexpr size_t kLdsBytes = 160 * 1024;
constexpr int kMaxVpt = 20;  // values per thread and task

struct TilePlan {
  int threads, wgs;  // per workgroup; workgroups per CU
  size_t lds;
};

static int row_stride(const AxisT& x, int& pad) {
  const int RL = x.R[x.nst - 1];
  pad = (x.nst > 1 && RL % 2 == 0) ? 1 : 0;
  const int row = x.N + (pad ? x.N / RL : 0);
  return row | 1;
}

static size_t tile_bytes(int rows, int RS, int Nx, int Ny) {
  return (size_t)rows * RS * 8 + (size_t)(Nx + Ny) * 8 + (size_t)(3 * Nx + 2 * Ny) * 2;
}

bool plane_fits(int Ny, int Nx) {
  if ((long long)Ny * Nx > kMaxVpt * 1024) return false;
  int pad;
  const int RS = std::max(row_stride(make_axis(Nx, nullptr, true), pad), row_stride(make_axis_seq(Nx, nullptr), pad));
  return tile_bytes(Ny, RS, Nx, Ny) <= kLdsBytes;
}

static TileArgs tile_args(const os3d_bank* b, const PassArgs& p, bool plane, bool seq, TilePlan& q) {
  const int Nz = (int)b->dims[0], Ny = (int)b->dims[1], Nx = (int)b->dims[2];
  TileArgs a = {};
  a.p = p;
  a.x = seq ? make_axis_seq(Nx, b->d.tw[2]) : make_axis(Nx, b->d.tw[2], true);
  a.y = seq ? make_axis_seq(Ny, b->d.tw[1]) : make_axis(Ny, b->d.tw[1]);
  a.RS = row_stride(a.x, a.pad);
  if (plane) {
    // several planes of a small grid share a workgroup, as long as that
    // leaves four workgroups per CU
    a.A = Ny;
    a.P = 1;
    for (int P = 2; P <= Nz; ++P)
      if (Nz % P == 0 && P * Ny * Nx <= 4096 && (long long)(Nz / P) * p.nb >= 1024) a.P = P;
    a.rows = a.P * Ny;
    a.tiles = Nz / a.P;
  } else {
    a.P = 1;
    a.A = a.rows = std::max(1, std::min(64, 6144 / Nx));
    a.tiles = ((long long)Nz * Ny + a.rows - 1) / a.rows;
  }
  a.mrows = fdiv_mul((unsigned)a.rows);
  a.mNx = fdiv_mul((unsigned)Nx);
  a.mRL = fdiv_mul((unsigned)a.x.R[a.x.nst - 1]);
  a.mP = fdiv_mul((unsigned)a.P);
  a.mA = fdiv_mul((unsigned)a.A);
  q.lds = tile_bytes(a.rows, a.RS, Nx, plane ? Ny : 0);
  // eight values per thread; a workgroup that shares its CU takes up to 512 threads
  const int n = a.rows * Nx;
  const int cap = 2 * q.lds <= kLdsBytes ? 512 : 1024;
  q.threads = std::min(cap, (n + 511) / 512 * 64);
  if ((n + q.threads - 1) / q.threads > kMaxVpt) q.threads = 1024;
  q.wgs = (int)std::max<size_t>(1, std::min<size_t>(kLdsBytes / q.lds, 1024 / q.threads));
  return a;
}

static int cu_count() {
  static const int n = [] {
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0)
      cus = 256;
    return cus;
  }();
  return n;
}

template <class K>
static int launch_tiles(K kernel, const TilePlan& q, const TileArgs& a, hipStream_t st) {
  static std::mutex mu;
  static std::set<const void*> done;
  {
    std::lock_guard<std::mutex> lock(mu);
    if (done.insert((const void*)kernel).second)
      (void)hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsBytes);
  }
  const long long ntask = a.tiles * a.p.nb;
  const unsigned grid = (unsigned)std::min<long long>(ntask, (long long)cu_count() * q.wgs);
  launch_k(kernel, dim3(grid), dim3(q.threads), (unsigned)q.lds, st, a);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) {
    set_error(std::string("k_tile: ") + hipGetErrorString(e));
    return OS3D_EDEVICE;
  }
  return OS3D_OK;
}

template <int LM, int SM, int DT, bool PLANE, bool SEQ>
static int launch_tile_dt(const TilePlan& q, const TileArgs& a, hipStream_t st) {
  const int n = a.rows * a.x.N;
  if (n <= 8 * q.threads) return launch_tiles(k_tile<LM, SM, DT, PLANE, SEQ, 8>, q, a, st);
  return launch_tiles(k_tile<LM, SM, DT, PLANE, SEQ, kMaxVpt>, q, a, st);
}

template <int LM, int SM, bool PLANE>
static int launch_tile_p(const TilePlan& q, const TileArgs& a, bool seq, hipStream_t st) {
  if constexpr (SM == SM_UOUT) {
    if (a.p.dtype == OS3D_BF16X2) return launch_tile_dt<LM, SM, OS3D_BF16X2, PLANE, true>(q, a, st);
    if (a.p.dtype == OS3D_F16X2) return launch_tile_dt<LM, SM, OS3D_F16X2, PLANE, true>(q, a, st);
  }
  if constexpr (LM == LM_UIN) {
    if (a.p.dtype == OS3D_BF16X2) return launch_tile_dt<LM, SM, OS3D_BF16X2, PLANE, false>(q, a, st);
    if (a.p.dtype == OS3D_F16X2) return launch_tile_dt<LM, SM, OS3D_F16X2, PLANE, false>(q, a, st);
  }
  if constexpr (LM == LM_REAL) {
    if (seq) return launch_tile_dt<LM, SM, OS3D_C64, PLANE, true>(q, a, st);
  }
  return launch_tile_dt<LM, SM, OS3D_C64, PLANE, false>(q, a, st);
}

template <int LM, int SM>
int launch_tile(const os3d_bank* b, const PassArgs& p, bool plane, bool seq, hipStream_t st) {
  TilePlan q;
  const TileArgs a = tile_args(b, p, plane, seq, q);
  return plane ? launch_tile_p<LM, SM, true>(q, a, seq, st) : launch_tile_p<LM, SM, false>(q, a, seq, st);
}

int launch_tile_phi(const os3d_bank* b, const PassArgs& p, bool plane, hipStream_t st) {
  TilePlan q;
  const TileArgs a = tile_args(b, p, plane, false, q);
  const bool few = a.rows * a.x.N <= 8 * q.threads;
  if (plane)
    return few ? launch_tiles(k_tile_phi<true, 8>, q, a, st) : launch_tiles(k_tile_phi<true, kMaxVpt>, q, a, st);
  return few ? launch_tiles(k_tile_phi<false, 8>, q, a, st) : launch_tiles(k_tile_phi<false, kMaxVpt>, q, a, st);
}

template int launch_tile<LM_REAL, SM_C>(const os3d_bank*, const PassArgs&, bool, bool, hipStream_t);
template int launch_tile<LM_C, SM_UOUT>(const os3d_bank*, const PassArgs&, bool, bool, hipStream_t);
template int launch_tile<LM_C, SM_REAL>(const os3d_bank*, const PassArgs&, bool, bool, hipStream_t);
template int launch_tile<LM_UIN, SM_C>(const os3d_bank*, const PassArgs&, bool, bool, hipStream_t);

}  // namespace os3d
