// Whole-plane and x-line passes of the general transform (stages:
// fft_tile.h).  A tile is a run of rows of Nx consecutive values: one or
// more whole (y, x) planes, transformed along both axes while they sit in
// LDS (one round trip of the intermediate instead of two), or, for planes
// larger than LDS, one class of their rows (yb, yb + B, ..: kernels_line.hip,
// "split passes") or rows transformed along x alone.  y goes before x: the loads
// are whole rows then, and the shorter runs are the stores' (the pair load of
// 96 x 80 x 64 x 41 pairs: 108 us, 117 with x first); only the spectrum of a
// volume whose scores are stored in 16 bits takes x first (its order is fixed).
//
// The first stage of the first axis loads its butterflies straight from
// memory (the fused load of the pass) and the last stage of the last axis
// stores straight to memory (the fused store); the stages in between run in
// place in LDS.  Memory accesses and the y stages take consecutive lanes on
// consecutive x (an x stage's accesses to memory are runs of N / R values, 64
// bytes and more); the x stages in LDS take consecutive lanes on consecutive
// rows: the row stride is odd, so a wave's accesses fall on distinct banks and
// its twiddles are broadcasts.  The passes are bound by the latency of that
// chain, not by arithmetic, so a butterfly keeps few registers (no tile in
// flight) and two or more workgroups share a CU where LDS allows; a workgroup
// loops over (pair, tile) tasks to keep its tables.
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
  u16* ys;  // frequency ky -> row after the DIF
};

// Where the rows of a tile lie in space: row r of the tile at g + r d.  Split
// planes: the tile of class yb holds the rows yb + B r (elsewhere, in the
// intermediate, its rows are consecutive).
struct RowMap {
  long long g;
  int d;
};
template <bool PLANE>
__device__ __forceinline__ RowMap space_rows(const TileArgs& a, long long tile) {
  if constexpr (PLANE) {
    if (a.B) {
      const int z = fdiv((int)tile, a.mB), yb = (int)tile - z * a.B;
      return {(long long)z * a.p.Ny * a.x.N + yb * a.x.N, a.B * a.x.N};
    }
  }
  return {tile * a.rows * a.x.N, a.x.N};
}

// conj: the twiddles of the inverse direction
template <bool PLANE>
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
      const float2 w = a.y.tw[i * a.y.tws];
      t.twy[i] = conj ? cconj(w) : w;
      const int f = freq_of(a.y, i);
      t.fy[i] = (u16)f;
      t.ys[f] = (u16)i;
    }
  }
  __syncthreads();
  return t;
}

// R values of one thread at g + r d of pair j
template <int LM, int DT, int R>
__device__ __forceinline__ void tile_load(const PassArgs& p, int j, long long g, long long d, float2* v) {
  if constexpr (LM == LM_REAL) {
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] = make_float2(ldnt(p.src_r + g + r * d), 0.f);
  } else if constexpr (LM == LM_C) {
    const float2* s = p.src_c + j * p.src_stride + g;
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] = ldnt(s + r * d);
  } else {
    using Word = typename std::conditional<DT == OS3D_C64, float2, unsigned int>::type;
    const int ia = p.oa[j], ib = p.ob[j];
    auto value = [](Word w, float sc) -> float2 {
      if constexpr (DT == OS3D_C64) return w;
      else return score_value<DT>(w, sc);
    };
    const float sa = DT == OS3D_C64 ? 1.f : p.scales[ia];
    const Word* ua = (const Word*)p.U + (long long)ia * p.V + g;
    Word wa[R];
#pragma unroll
    for (int r = 0; r < R; ++r) wa[r] = ldnt(ua + r * d);
    if (ib >= 0) {
      const float sb = DT == OS3D_C64 ? 1.f : p.scales[ib];
      const Word* ub = (const Word*)p.U + (long long)ib * p.V + g;
      Word wb[R];
#pragma unroll
      for (int r = 0; r < R; ++r) wb[r] = ldnt(ub + r * d);
#pragma unroll
      for (int r = 0; r < R; ++r) v[r] = cadd(value(wa[r], sa), cconj(value(wb[r], sb)));
    } else {
#pragma unroll
      for (int r = 0; r < R; ++r) v[r] = value(wa[r], sa);
    }
  }
}

// The transformed values of a butterfly, slot r at frequency seq_slot(r), stored at g + k d
template <int SM, int DT, int R, int RB>
__device__ __forceinline__ void tile_store(const PassArgs& p, int j, long long g, long long d, const float2* v) {
  float2 u[R], dummy[R];
#pragma unroll
  for (int r = 0; r < R; ++r) u[seq_slot<R, RB>(r)] = v[r];
  store_k<SM, DT, R>(p, j, g, d, u, dummy);
}

template <bool SEQ, bool INV, bool DIT, int R, int RB, bool REAL = false>
__device__ __forceinline__ void butterfly(const AxisT& x, int i, const float2* tw, int t, float2* v, float sgn) {
  if constexpr (SEQ) {
    seq_butterfly<R, RB, REAL>(v, tw, t, x.S[i], x.tstep[i], i == 0, sgn);
  } else {
    if (DIT ? i < x.nst - 1 : i > 0) twiddle<R, INV>(v, tw, DIT ? t * x.tstep[i] : t * x.S[i]);
    dft_r<R>(v, INV ? 1.f : -1.f);
  }
}

// Stage i of the rows in LDS, in place; phi: between the last stage of the
// inverse DFT and the first of the forward one.
template <bool SEQ, bool INV, bool DIT, bool PHI = false>
__device__ __forceinline__ void x_stage(const TileArgs& a, const TileLds& t, int i, int j = 0) {
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
      butterfly<SEQ, INV, DIT, R, RB>(x, i, t.twx, DIT ? l : t.fx[u * R * S], v, a.p.sgn);
      if constexpr (PHI) {
#pragma unroll
        for (int r = 0; r < R; ++r) v[r] = phi_apply(a.p, j, v[r]);
        dft_r<R>(v, -1.f);
      }
#pragma unroll
      for (int r = 0; r < R; ++r) q[r * Sp] = v[r];
    }
  });
}

// First stage of the rows, from memory.
template <int LM, int DT, bool SEQ, bool INV, class Done>
__device__ __forceinline__ void x_first(const TileArgs& a, const TileLds& t, int j, long long g0, int nrows,
                                        Done done) {
  const AxisT& x = a.x;
  const int S = x.S[0], Sp = x.nst == 1 ? 1 : S + fdiv(S, a.mRL) * a.pad;
  with_stage<SEQ>(x, 0, OS3D_SEQ_FN(rc, rb) {
    constexpr int R = decltype(rc)::value, RB = decltype(rb)::value;
    const int total = nrows * S;
    for (int id = threadIdx.x; id < total; id += blockDim.x) {
      const int row = fdiv(id, x.mS[0]), l = id - row * S;
      float2 v[R];
      tile_load<LM, DT, R>(a.p, j, g0 + row * x.N + l, S, v);
      butterfly<SEQ, INV, false, R, RB, LM == LM_REAL>(x, 0, t.twx, 0, v, a.p.sgn);
      done(rc, rb, v, t.buf + row * a.RS + t.xl[l], Sp, row);
    }
  });
}

// Last stage of the rows, to memory (PLANE: the rows are digit-reversed).
template <int SM, int DT, bool PLANE, bool SEQ, bool INV>
__device__ __forceinline__ void x_last(const TileArgs& a, const TileLds& t, int j, RowMap m, int nrows) {
  const AxisT& x = a.x;
  const int i = x.nst - 1;
  with_stage<SEQ>(x, i, OS3D_SEQ_FN(rc, rb) {
    constexpr int R = decltype(rc)::value, RB = decltype(rb)::value;
    const int nf = x.nb[i], total = nrows * nf;
    for (int id = threadIdx.x; id < total; id += blockDim.x) {
      const int row = fdiv(id, a.mnf), f = id - row * nf;  // lowest frequency of the butterfly
      int lrow = row;
      if constexpr (PLANE) {
        const int plane = fdiv(row, a.mA);
        lrow = plane * a.A + t.ys[row - plane * a.A];
      }
      const float2* q = t.buf + lrow * a.RS + t.xs[f];
      float2 v[R];
#pragma unroll
      for (int r = 0; r < R; ++r) v[r] = q[r];
      butterfly<SEQ, INV, false, R, RB>(x, i, t.twx, f, v, a.p.sgn);
      tile_store<SM, DT, R, RB>(a.p, j, m.g + row * m.d + f, nf, v);
    }
  });
}

// Stage i of the columns in LDS: fn(R, RB, v, q, d, pos, col, plane) takes the
// transformed butterfly at row position pos of column col (LDS address q,
// stride d).  Columns go by position in the row (xl), or in the order of
// their frequencies (NATURAL).
template <bool SEQ, bool INV, bool DIT, bool NATURAL, class Fn>
__device__ __forceinline__ void y_stage(const TileArgs& a, const TileLds& t, int i, Fn fn) {
  const AxisT& y = a.y;
  const int S = y.S[i];
  with_stage<SEQ>(y, i, OS3D_SEQ_FN(rc, rb) {
    constexpr int R = decltype(rc)::value, RB = decltype(rb)::value;
    const int total = a.P * y.nb[i] * a.x.N;
    for (int id = threadIdx.x; id < total; id += blockDim.x) {
      const int e = fdiv(id, a.mNx), col = id - e * a.x.N;
      const int b = fdiv(e, a.mP), plane = e - b * a.P;
      const int u = fdiv(b, y.mS[i]), l = b - u * S, pos = u * R * S + l;
      float2* q = t.buf + (plane * a.A + pos) * a.RS + (NATURAL ? t.xs : t.xl)[col];
      const int d = S * a.RS;
      float2 v[R];
#pragma unroll
      for (int r = 0; r < R; ++r) v[r] = q[r * d];
      butterfly<SEQ, INV, DIT, R, RB>(y, i, t.twy, DIT ? l : t.fy[u * R * S], v, a.p.sgn);
      fn(rc, rb, v, q, d, pos, col, plane);
    }
  });
}

// First stage of the columns, from memory.
template <int LM, int DT, bool SEQ, bool INV>
__device__ __forceinline__ void y_first(const TileArgs& a, const TileLds& t, int j, RowMap m) {
  const AxisT& y = a.y;
  const int S = y.S[0];
  with_stage<SEQ>(y, 0, OS3D_SEQ_FN(rc, rb) {
    constexpr int R = decltype(rc)::value, RB = decltype(rb)::value;
    const int total = a.P * S * a.x.N;
    for (int id = threadIdx.x; id < total; id += blockDim.x) {
      const int e = fdiv(id, a.mNx), col = id - e * a.x.N;
      const int b = fdiv(e, a.mP), row = (e - b * a.P) * a.A + b;
      float2 v[R];
      tile_load<LM, DT, R>(a.p, j, m.g + row * m.d + col, (long long)S * m.d, v);
      butterfly<SEQ, INV, false, R, RB>(y, 0, t.twy, 0, v, a.p.sgn);
      float2* q = t.buf + row * a.RS + t.xl[col];
      const int d = S * a.RS;
#pragma unroll
      for (int r = 0; r < R; ++r) q[r * d] = v[r];
    }
  });
}

struct KeepInLds {
  // columns
  template <class RC, class RB>
  __device__ __forceinline__ void operator()(RC, RB, const float2* v, float2* q, int d, int, int, int) const {
#pragma unroll
    for (int r = 0; r < RC::value; ++r) q[r * d] = v[r];
  }
  // rows
  template <class RC, class RB>
  __device__ __forceinline__ void operator()(RC, RB, const float2* v, float2* q, int d, int) const {
#pragma unroll
    for (int r = 0; r < RC::value; ++r) q[r * d] = v[r];
  }
};

// SEQ: the sequential order of the forward transform into 16-bit scores.
template <int LM, int SM, int DT, bool PLANE, bool SEQ>
__global__ __launch_bounds__(1024) void k_tile(TileArgs a) {
  constexpr bool INV = SM == SM_UOUT || SM == SM_REAL;  // the other stores end a forward DFT
  constexpr bool kXFirst = SEQ && !INV;
  extern __shared__ float2 lds[];
  const PassArgs& p = a.p;
  const TileLds t = tile_lds<PLANE>(a, lds, SEQ && INV);
  const int n = a.rows * a.x.N, lx = a.x.nst - 1, ly = a.y.nst - 1;
  const long long ntask = a.tiles * p.nb;
  for (long long step = blockIdx.x; step < ntask; step += gridDim.x) {
    const long long task = p.newest_first ? ntask - 1 - step : step;
    const int j = (int)(task / a.tiles);
    const long long tile = task - j * a.tiles, g0 = tile * n;
    if constexpr (!PLANE) {
      const int nrows = (int)min((long long)a.rows, a.nlines - tile * a.rows);
      if (lx == 0) {
        x_first<LM, DT, SEQ, INV>(a, t, j, g0, nrows,
                                  [&](auto rc, auto rb, const float2* v, float2*, int, int row) {
          tile_store<SM, DT, decltype(rc)::value, decltype(rb)::value>(p, j, g0 + row * a.x.N, 1, v);
        });
      } else {
        x_first<LM, DT, SEQ, INV>(a, t, j, g0, nrows, KeepInLds{});
        __syncthreads();
        for (int i = 1; i < lx; ++i) {
          x_stage<SEQ, INV, false>(a, t, i);
          __syncthreads();
        }
        x_last<SM, DT, PLANE, SEQ, INV>(a, t, j, {g0, a.x.N}, nrows);
      }
    } else if constexpr (!kXFirst) {
      y_first<LM, DT, SEQ, INV>(a, t, j, LM == LM_UIN ? space_rows<PLANE>(a, tile) : RowMap{g0, a.x.N});
      __syncthreads();
      for (int i = 1; i <= ly; ++i) {
        y_stage<SEQ, INV, false, false>(a, t, i, KeepInLds{});
        __syncthreads();
      }
      for (int i = 0; i < lx; ++i) {
        x_stage<SEQ, INV, false>(a, t, i);
        __syncthreads();
      }
      x_last<SM, DT, PLANE, SEQ, INV>(a, t, j, SM == SM_UOUT ? space_rows<PLANE>(a, tile) : RowMap{g0, a.x.N}, a.rows);
    } else {
      x_first<LM, DT, SEQ, INV>(a, t, j, g0, a.rows, KeepInLds{});
      __syncthreads();
      for (int i = 1; i <= lx; ++i) {
        x_stage<SEQ, INV, false>(a, t, i);
        __syncthreads();
      }
      for (int i = 0; i < ly; ++i) {
        y_stage<SEQ, INV, false, false>(a, t, i, KeepInLds{});
        __syncthreads();
      }
      y_stage<SEQ, INV, false, true>(
          a, t, ly, [&](auto rc, auto rb, const float2* v, float2*, int, int pos, int col, int plane) {
            constexpr int R = decltype(rc)::value, RB = decltype(rb)::value;
            tile_store<SM, DT, R, RB>(p, j, g0 + (plane * a.A + t.fy[pos]) * a.x.N + col,
                                      (long long)(a.A / R) * a.x.N, v);
          });
    }
    __syncthreads();  // the tile is rewritten by the next task
  }
}

// Processing via scores, both directions in one kernel and in place: inverse
// DFT of the tile, Phi on the scores, forward DFT.  The scores stay in
// digit-reversed order in between (DIF, Phi in the registers of its last
// stage, DIT).
template <bool PLANE>
__global__ __launch_bounds__(1024) void k_tile_phi(TileArgs a) {
  extern __shared__ float2 lds[];
  const PassArgs& p = a.p;
  const TileLds t = tile_lds<PLANE>(a, lds, false);
  const int n = a.rows * a.x.N, lx = a.x.nst - 1, ly = a.y.nst - 1;
  const long long ntask = a.tiles * p.nb;
  for (long long task = blockIdx.x; task < ntask; task += gridDim.x) {
    const int j = (int)(task / a.tiles);
    const long long tile = task - j * a.tiles, g0 = tile * n;
    const int nrows = PLANE ? a.rows : (int)min((long long)a.rows, a.nlines - tile * a.rows);
    if constexpr (PLANE) {
      y_first<LM_C, OS3D_C64, false, true>(a, t, j, {g0, a.x.N});
      __syncthreads();
      for (int i = 1; i <= ly; ++i) {
        y_stage<false, true, false, false>(a, t, i, KeepInLds{});
        __syncthreads();
      }
    } else {
      for (int e = threadIdx.x; e < nrows * a.x.N; e += blockDim.x) {
        const int row = fdiv(e, a.mNx), x = e - row * a.x.N;
        t.buf[row * a.RS + t.xl[x]] = p.src_c[j * p.src_stride + g0 + e];
      }
      __syncthreads();
    }
    for (int i = 0; i < lx; ++i) {
      x_stage<false, true, false>(a, t, i);
      __syncthreads();
    }
    x_stage<false, true, false, true>(a, t, lx, j);
    __syncthreads();
    for (int i = lx - 1; i >= 0; --i) {
      x_stage<false, false, true>(a, t, i);
      __syncthreads();
    }
    float2* dst = p.dst_c + j * p.dst_stride + g0;
    if constexpr (PLANE) {
      for (int i = ly; i > 0; --i) {
        y_stage<false, false, true, false>(a, t, i, KeepInLds{});
        __syncthreads();
      }
      y_stage<false, false, true, false>(
          a, t, 0, [&](auto rc, auto, const float2* v, float2*, int, int pos, int col, int plane) {
            constexpr int R = decltype(rc)::value;
            const int o = (plane * a.A + pos) * a.x.N + col, d = (a.A / R) * a.x.N;
#pragma unroll
            for (int r = 0; r < R; ++r) dst[o + r * d] = v[r];
          });
    } else {
      for (int e = threadIdx.x; e < nrows * a.x.N; e += blockDim.x) {
        const int row = fdiv(e, a.mNx), x = e - row * a.x.N;
        dst[e] = t.buf[row * a.RS + t.xl[x]];
      }
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------- host side
constexpr size_t kLdsBytes = 160 * 1024;

constexpr int kMaxPlane = 20 * 1024;  // values of a plane in LDS

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
  if ((long long)Ny * Nx > kMaxPlane) return false;
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
  if (p.split) {  // a class of the rows of a plane
    a.B = p.split;
    a.mB = fdiv_mul((unsigned)a.B);
    a.y = make_axis(Ny / a.B, b->d.tw[1]);
    a.y.tws = a.B;
    a.P = 1;
    a.A = a.rows = Ny / a.B;
    a.tiles = (long long)Nz * a.B;
  } else if (plane) {
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
    a.nlines = (long long)Nz * Ny;
    a.tiles = (a.nlines + a.rows - 1) / a.rows;
  }
  a.mrows = fdiv_mul((unsigned)a.rows);
  a.mNx = fdiv_mul((unsigned)Nx);
  a.mRL = fdiv_mul((unsigned)a.x.R[a.x.nst - 1]);
  a.mP = fdiv_mul((unsigned)a.P);
  a.mA = fdiv_mul((unsigned)a.A);
  q.lds = tile_bytes(a.rows, a.RS, Nx, plane ? a.A : 0);
  a.mnf = fdiv_mul((unsigned)a.x.nb[a.x.nst - 1]);
  // a butterfly of ten values or so per thread; a workgroup that shares its CU takes up to 512 threads
  const int n = a.rows * Nx;
  const int cap = 2 * q.lds <= kLdsBytes ? 512 : 1024;
  q.threads = std::min(cap, (n + 639) / 640 * 64);
  q.wgs = (int)std::max<size_t>(1, std::min<size_t>(kLdsBytes / q.lds, 1280 / q.threads));  // five waves per SIMD
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

template <int LM, int SM, bool PLANE>
static int launch_tile_p(const TilePlan& q, const TileArgs& a, bool seq, hipStream_t st) {
  if constexpr (SM == SM_UOUT) {
    if (a.p.dtype == OS3D_BF16X2) return launch_tiles(k_tile<LM, SM, OS3D_BF16X2, PLANE, true>, q, a, st);
    if (a.p.dtype == OS3D_F16X2) return launch_tiles(k_tile<LM, SM, OS3D_F16X2, PLANE, true>, q, a, st);
  }
  if constexpr (LM == LM_UIN) {
    if (a.p.dtype == OS3D_BF16X2) return launch_tiles(k_tile<LM, SM, OS3D_BF16X2, PLANE, false>, q, a, st);
    if (a.p.dtype == OS3D_F16X2) return launch_tiles(k_tile<LM, SM, OS3D_F16X2, PLANE, false>, q, a, st);
  }
  if constexpr (LM == LM_REAL) {
    if (seq) return launch_tiles(k_tile<LM, SM, OS3D_C64, PLANE, true>, q, a, st);
  }
  return launch_tiles(k_tile<LM, SM, OS3D_C64, PLANE, false>, q, a, st);
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
  return plane ? launch_tiles(k_tile_phi<true>, q, a, st) : launch_tiles(k_tile_phi<false>, q, a, st);
}

template int launch_tile<LM_REAL, SM_C>(const os3d_bank*, const PassArgs&, bool, bool, hipStream_t);
template int launch_tile<LM_C, SM_UOUT>(const os3d_bank*, const PassArgs&, bool, bool, hipStream_t);
template int launch_tile<LM_C, SM_REAL>(const os3d_bank*, const PassArgs&, bool, bool, hipStream_t);
template int launch_tile<LM_UIN, SM_C>(const os3d_bank*, const PassArgs&, bool, bool, hipStream_t);

}  // namespace os3d
