// 3D DFTs of the orientation-score transform (Eqs. 7-8) on gfx950: the order
// of the passes for every volume but 256^3 (kernels_fft4.hip), the scales of
// 16-bit scores and the per-kernel timer.
//
// Every 3D transform is a pass along z and a pass over (y, x) planes, so the
// intermediate makes one round trip through memory; planes larger than LDS
// take a y-line and an x-line pass instead (two round trips).  The per-voxel
// work of the method is fused into the passes:
//   * z lines (kernels_line.hip): the DFT of f along z, the spectral multiply
//     psi_hat_i F and the inverse DFT; the orientation sum
//     X += psi_hat_n DFT(.) over a batch of pairs, X / max(M, eps) and the
//     inverse DFT;
//   * planes (kernels_plane.hip for 64^2 and 128^2, kernels_tile.hip for the
//     others) and x lines (kernels_tile.hip): the antipodal pair store U_n and
//     U_{-n} = conj(U_n), the pair load U_n + conj(U_{-n}), Phi, the real part.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdlib>

#include "fft_pass.h"
#include "fft_tile.h"
#include "launch.h"
#include "layout4.h"

namespace os3d {

// Per-orientation power-of-two scale for 16-bit score storage from the
// bound max|U_i| <= (1/V) sum_k |psi_hat_i[k] F[k]|: fp16 maps the bound to
// at most 2^15, bf16 to at most 1.  Fixed-order FP64 sum (deterministic).
__global__ __launch_bounds__(256) void k_scales(const float* partial, int ntiles, PassArgs a, int dtype,
                                                float* scales) {
  __shared__ double red[256];
  const int j = blockIdx.x;
  double s = 0.0;
  for (int t = threadIdx.x; t < ntiles; t += 256) s += (double)partial[(long long)j * ntiles + t];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    double bound = red[0] / (double)a.V * (1.0 + 1e-5);
    float sc = 1.f;
    if (bound > 0.0) {
      int e;
      frexp(bound, &e);  // bound <= 2^e
      sc = (float)ldexp(1.0, dtype == OS3D_F16X2 ? e - 15 : e);
    }
    scales[a.oa[j]] = sc;
    if (a.ob[j] >= 0) scales[a.ob[j]] = sc;
  }
}

void launch_scales(const float* partial, int ntiles, const PassArgs& a, int dtype, float* scales, int nb,
                   hipStream_t st) {
  launch_k(k_scales, dim3(nb), dim3(256), 0, st, partial, ntiles, a, dtype, scales);
}

static int check_launch(const char* what) {
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) {
    set_error(std::string(what) + ": " + hipGetErrorString(e));
    return OS3D_EDEVICE;
  }
  return OS3D_OK;
}

// ---------------------------------------------------------------------------
// Optional per-kernel timing: a pair of HIP events per launch, stamped by the
// runtime with the kernel's start and end (launch_k), with the algorithmic
// bytes each launch must move; every launch, or only those of one slot (so
// that timing one kernel leaves the others' launches untouched).
// Process-wide and meant for one host thread (the benchmark); events are
// reused across enable calls.
// ---------------------------------------------------------------------------
static_assert((int)kProfBank == (int)PROF_BANK, "profiler slot of the bank kernel");
static const char* kKernelNames[kProfCount] = {
    "dft_f_first_real_in", "dft_f_mid", "dft_f_last", "fwd_first_mul_bank", "fwd_scales", "fwd_mid",
    "fwd_last_store_scores", "rec_first_load_scores", "rec_mid", "rec_last_accumulate", "inv_first_divide_M",
    "inv_mid", "inv_last_real_out", "bank_synth_mfma"};

struct ProfRec {
  int kid;
  hipEvent_t e0, e1;
  double alg_bytes, alg_flops;
  bool launched;
};
static int g_prof_mode = 0;  // 0 off, 1 every launch, 2 + k only the launches of slot k
static std::vector<ProfRec> g_prof;
static std::vector<hipEvent_t> g_event_pool;
static thread_local ProfRec* t_pending = nullptr;

static bool take_event(hipEvent_t* e) {
  if (!g_event_pool.empty()) {
    *e = g_event_pool.back();
    g_event_pool.pop_back();
    return true;
  }
  return hipEventCreate(e) == hipSuccess;
}

void* prof_start(void* stream, int kid) {
  (void)stream;
  if (g_prof_mode == 0 || (g_prof_mode >= 2 && kid != g_prof_mode - 2)) return nullptr;
  ProfRec* r = new ProfRec();
  r->launched = false;
  if (!take_event(&r->e0)) {
    delete r;
    return nullptr;
  }
  if (!take_event(&r->e1)) {
    g_event_pool.push_back(r->e0);
    delete r;
    return nullptr;
  }
  t_pending = r;
  return r;
}

bool prof_take(hipEvent_t* e0, hipEvent_t* e1) {
  ProfRec* r = t_pending;
  if (!r) return false;
  t_pending = nullptr;
  r->launched = true;
  *e0 = r->e0;
  *e1 = r->e1;
  return true;
}

void prof_stop(void* token, void* stream, int kid, double alg_bytes, double alg_flops) {
  (void)stream;
  if (!token) return;
  ProfRec* r = (ProfRec*)token;
  if (t_pending == r) t_pending = nullptr;
  if (r->launched) {
    r->kid = kid;
    r->alg_bytes = alg_bytes;
    r->alg_flops = alg_flops;
    g_prof.push_back(*r);
  } else {  // no launch between start and stop: nothing to time
    g_event_pool.push_back(r->e0);
    g_event_pool.push_back(r->e1);
  }
  delete r;
}

// Arguments of one pass over nb pairs.
static PassArgs pass_args(const os3d_bank* b, float sgn, int nb) {
  PassArgs a = {};
  a.Nz = (int)b->dims[0];
  a.Ny = (int)b->dims[1];
  a.Nx = (int)b->dims[2];
  a.V = b->V;
  a.tw = (const float2*)b->d.tw[2];
  a.sgn = sgn;
  a.nb = nb;
  return a;
}

static void set_pairs(const os3d_bank* b, PassArgs& a, int r0) {
  for (int j = 0; j < a.nb; ++j) {
    const int o = b->rep[r0 + j];
    a.rows[j] = r0 + j;
    a.oa[j] = o;
    a.ob[j] = b->partner[o];
  }
  a.psi = b->d.psi;
  a.kappa = (float)b->kappa;
}

// Algorithmic score bytes of one launch: every stored row stands for one
// orientation, or two with its antipode.
static double score_bytes(const PassArgs& a, size_t ubytes) {
  int n = 0;
  for (int j = 0; j < a.nb; ++j) n += (a.ob[j] >= 0) ? 2 : 1;
  return (double)n * (double)a.V * (double)ubytes;
}

// Launch f() timed under slot kid.
template <class F>
static int timed(hipStream_t st, int kid, double alg, F f) {
  void* tok = prof_start(st, kid);
  const int rc = f();
  prof_stop(tok, st, kid, alg, 0.0);
  return rc ? rc : check_launch(kKernelNames[kid]);
}

// The pass over (y, x) planes or x lines with the fused load LM and store SM;
// seq: in the sequential order of the forward transform into 16-bit scores.
template <int LM, int SM>
static int run_xy(const os3d_bank* b, int kid, double alg, const PassArgs& a, bool seq, hipStream_t st) {
  return timed(st, kid, alg, [&]() -> int {
    if (b->plane != kPlaneFixed) return launch_tile<LM, SM>(b, a, b->plane == kPlaneTile || a.split, seq, st);
    launch_plane<LM, SM>(a, a.nb, st);
    return OS3D_OK;
  });
}

static int run_y(const os3d_bank* b, int kid, const PassArgs& a, bool seq, hipStream_t st) {
  return timed(st, kid, 0.0, [&]() -> int { return launch_yline(b, a, seq, st); });
}

// Orientation pairs per launch: larger batches amortise the spectrum loads
// and the orientation-sum read-modify-write and keep more workgroups in
// flight; each pair costs one intermediate volume of workspace.  96 x 80 x 64 with
// 81 pairs takes 679 us a job in two launches (43 volumes) and 615 in one (83):
// the pairs stay at 64, so that a job that fits next to others in a memory
// budget goes on fitting.
static int pair_batch(const os3d_bank* b) {
  int nb = kMaxBatch;
  if (const char* e = getenv("OS3D_PAIR_BATCH")) nb = atoi(e);
  nb = std::max(1, std::min(std::min(nb, kMaxBatch), b->n_unique));
  // one complex intermediate volume per pair of a launch: at most 8 GiB of them
  nb = (int)std::max(1LL, std::min((long long)nb, (8LL << 30) / (b->V * (long long)sizeof(float2))));
  // the same number of pairs in every launch (no short last launch)
  const int launches = (b->n_unique + nb - 1) / nb;
  return (b->n_unique + launches - 1) / launches;
}

size_t workspace_bytes(const os3d_bank* b) {
  const int nb = pair_batch(b);
  // F or X, one intermediate per pair of the batch; processing via scores needs
  // F and X, and at 256^3 two buffers per pair of a half batch.  The scale
  // bounds of 16-bit scores (a float per pair and tile) have room of their own
  // at 256^3; elsewhere they go into the volume that is X in processing: a
  // tile holds Nz W values (W = 32 lines, fewer only where Nz > 32), so nb <= 64
  // pairs take at most 8 V + 4 nb bytes.
  const size_t bounds = b->layout == kLayoutFour256 ? (size_t)nb * 1024 * sizeof(float) : 0;
  return (size_t)(2 + std::max(nb, 2)) * b->V * sizeof(float2) + bounds + 256;
}

// f transformed along x and y into F (the z lines follow in the spectral multiply).
static int dft_planes_of_f(const os3d_bank* b, const float* f, float2* F, bool seq, hipStream_t st) {
  PassArgs a = pass_args(b, -1.f, 1);
  a.src_r = f;
  a.dst_c = F;
  int rc = run_xy<LM_REAL, SM_C>(b, kProfDftFirst, 4.0 * b->V, a, seq, st);
  if (rc || b->plane) return rc;
  a.src_c = F;
  return run_y(b, kProfDftMid, a, seq, st);
}

// X transformed along y and x, its real part into f_out.
static int planes_to_f(const os3d_bank* b, float2* X, float* f_out, hipStream_t st) {
  PassArgs a = pass_args(b, 1.f, 1);
  a.src_c = X;
  a.dst_c = X;
  int rc;
  if (!b->plane && (rc = run_y(b, kProfInvMid, a, false, st))) return rc;
  a.dst_r = f_out;
  a.out_scale = 1.f / (float)b->V;
  return run_xy<LM_C, SM_REAL>(b, kProfInvLast, 4.0 * b->V, a, false, st);
}

// The weighted orientation sum of the nb intermediates T (transformed along x
// and y; overwritten) into X; the last launch of a volume goes on to X / max(M,
// eps) (or X alone) transformed back along z.
static int sum_pairs(const os3d_bank* b, const PassArgs& pairs, float2* T, float2* X, bool first, bool last,
                     bool divide_M, hipStream_t st) {
  const int groups = zline_acc_groups(b, pairs.nb);
  PassArgs z = pairs;
  z.src_c = T;
  z.src_stride = b->V;
  z.dst_c = X;
  z.accumulate = first ? 0 : 1;
  z.M = b->d.M;
  z.eps = (float)b->params.eps;
  z.divide = divide_M ? 1 : 0;
  const bool finish = last && groups == 1;
  int rc = timed(st, kProfRecLast, 0.0,
                 [&]() -> int { return launch_zline_acc(b, z, T, groups, finish, st); });
  if (rc || groups == 1) return rc;
  z.src_c = X;
  z.split = 0;
  return timed(st, last ? kProfInvFirst : kProfRecLast, 0.0,
               [&]() -> int { return launch_zline_div(b, z, T, groups, last, st); });
}

int launch_forward(const os3d_bank* b, const float* f, int batch, void* U, int dtype, float* scales, void* ws,
                   void* stream) {
  if (b->layout == kLayoutFour256) return forward4(b, f, batch, U, dtype, scales, ws, pair_batch(b), stream);
  hipStream_t st = (hipStream_t)stream;
  const long long V = b->V;
  const int nbmax = pair_batch(b);
  float2* F = (float2*)ws;
  float2* T = F + V;
  float* partial = (float*)(T + (long long)nbmax * V);
  const size_t ubytes = (dtype == OS3D_C64) ? 8 : 4;
  const bool quant = dtype != OS3D_C64;
  int rc;
  for (int bi = 0; bi < batch; ++bi) {
    if ((rc = dft_planes_of_f(b, f + (long long)bi * V, F, quant, st))) return rc;
    float* sc = scales ? scales + (long long)bi * b->n_orients : nullptr;
    for (int r0 = 0; r0 < b->n_unique; r0 += nbmax) {
      PassArgs z = pass_args(b, 1.f, std::min(nbmax, b->n_unique - r0));
      set_pairs(b, z, r0);
      z.split = quant ? 0 : b->split;
      z.src_c = F;
      z.dst_c = T;
      z.dst_stride = V;
      z.partial = quant ? partial : nullptr;
      if ((rc = timed(st, kProfFwdFirst, 0.0, [&]() -> int { return launch_zline_mul(b, z, st); }))) return rc;
      if (quant) {
        rc = timed(st, kProfScales, 0.0, [&]() -> int {
          launch_scales(partial, zline_tiles(b), z, dtype, sc, z.nb, st);
          return OS3D_OK;
        });
        if (rc) return rc;
      }
      z.src_c = T;
      z.src_stride = V;
      if (!b->plane && !z.split && (rc = run_y(b, kProfFwdMid, z, quant, st))) return rc;
      // the pass before wrote T in ascending order: its last pairs are still in
      // the last-level cache (256 MB), so this one begins with them.  Forward +
      // reconstruction, oldest and newest first: 160 x 128 x 128 x 42 772 and 733 us,
      // 128^3 x 42 641 and 600, 96 x 80 x 64 x 162 690 and 679.  With a pass over y
      // between them reversing any of the passes gave nothing or lost 2 %.
      z.newest_first = b->plane || z.split ? 1 : 0;
      z.Uout = (char*)U + (size_t)bi * b->n_orients * V * ubytes;
      z.dtype = dtype;
      z.scales = quant ? sc : nullptr;
      z.out_scale = 1.f / (float)V;
      if ((rc = run_xy<LM_C, SM_UOUT>(b, kProfFwdLast, score_bytes(z, ubytes), z, quant, st))) return rc;
    }
  }
  return OS3D_OK;
}

int reduce_pair_batch(const os3d_bank* b, long long ws_bytes) {
  // X and one intermediate volume per pair of a launch
  const int nb = (int)std::min<long long>(pair_batch(b), ws_bytes / (b->V * (long long)sizeof(float2)) - 1);
  if (nb < 1) return 0;
  const int launches = (b->n_unique + nb - 1) / nb;
  return (b->n_unique + launches - 1) / launches;
}

int launch_reduce(const os3d_bank* b, const void* U, int dtype, const float* scales, int batch, float* f_out,
                  void* ws, bool divide_M, void* stream, int nb_limit) {
  const int nbmax = nb_limit > 0 ? nb_limit : pair_batch(b);
  if (b->layout == kLayoutFour256)
    return reduce4(b, U, dtype, scales, batch, f_out, ws, divide_M, nbmax, stream);
  hipStream_t st = (hipStream_t)stream;
  const long long V = b->V;
  float2* X = (float2*)ws;
  float2* T = X + V;
  const size_t ubytes = (dtype == OS3D_C64) ? 8 : 4;
  int rc;
  for (int bi = 0; bi < batch; ++bi) {
    for (int r0 = 0; r0 < b->n_unique; r0 += nbmax) {
      PassArgs x = pass_args(b, -1.f, std::min(nbmax, b->n_unique - r0));
      set_pairs(b, x, r0);
      x.split = b->split;
      x.U = (const char*)U + (size_t)bi * b->n_orients * V * ubytes;
      x.dtype = dtype;
      x.scales = (dtype == OS3D_C64) ? nullptr : scales + (long long)bi * b->n_orients;
      x.dst_c = T;
      x.dst_stride = V;
      if ((rc = run_xy<LM_UIN, SM_C>(b, kProfRecFirst, score_bytes(x, ubytes), x, false, st))) return rc;
      x.src_c = T;
      x.src_stride = V;
      if (!b->plane && !x.split && (rc = run_y(b, kProfRecMid, x, false, st))) return rc;
      if ((rc = sum_pairs(b, x, T, X, r0 == 0, r0 + nbmax >= b->n_unique, divide_M, st))) return rc;
    }
    if ((rc = planes_to_f(b, X, f_out + (long long)bi * V, st))) return rc;
  }
  return OS3D_OK;
}

// Processing via scores, Eq. (23) with the stabilised inverse: per pair batch
// the spectral multiply, Phi between the inverse and the forward DFT of the
// planes (in place, in LDS), and the orientation sum; planes larger than LDS
// take y-line passes around the x lines that apply Phi.
int launch_process(const os3d_bank* b, const float* f, int batch, int phi_kind, float phi_p, float* f_out, void* ws,
                   void* stream) {
  if (b->layout == kLayoutFour256)  // two intermediate volumes per pair
    return process4(b, f, batch, phi_kind, phi_p, f_out, ws, std::max(1, pair_batch(b) / 2), stream);
  const int nbp = pair_batch(b);
  hipStream_t st = (hipStream_t)stream;
  const long long V = b->V;
  float2* F = (float2*)ws;
  float2* X = F + V;
  float2* T = X + V;
  int rc;
  for (int bi = 0; bi < batch; ++bi) {
    if ((rc = dft_planes_of_f(b, f + (long long)bi * V, F, false, st))) return rc;
    for (int r0 = 0; r0 < b->n_unique; r0 += nbp) {
      PassArgs z = pass_args(b, 1.f, std::min(nbp, b->n_unique - r0));
      set_pairs(b, z, r0);
      z.split = b->split;
      z.src_c = F;
      z.dst_c = T;
      z.dst_stride = V;
      if ((rc = timed(st, kProfFwdFirst, 0.0, [&]() -> int { return launch_zline_mul(b, z, st); }))) return rc;
      z.src_c = T;
      z.src_stride = V;
      if (!b->plane && !z.split && (rc = run_y(b, kProfFwdMid, z, false, st))) return rc;
      z.out_scale = 1.f / (float)V;
      z.phi_kind = phi_kind;
      z.phi_p = phi_p;
      rc = timed(st, kProfFwdLast, 0.0, [&]() -> int {
        if (b->plane != kPlaneFixed) return launch_tile_phi(b, z, b->plane == kPlaneTile || z.split, st);
        launch_plane_phi(z, z.nb, st);
        return OS3D_OK;
      });
      if (rc) return rc;
      z.sgn = -1.f;
      if (!b->plane && !z.split && (rc = run_y(b, kProfRecMid, z, false, st))) return rc;
      if ((rc = sum_pairs(b, z, T, X, r0 == 0, r0 + nbp >= b->n_unique, true, st))) return rc;
    }
    if ((rc = planes_to_f(b, X, f_out + (long long)bi * V, st))) return rc;
  }
  return OS3D_OK;
}

int profile_enable(int on) {
  for (auto& r : g_prof) {
    g_event_pool.push_back(r.e0);
    g_event_pool.push_back(r.e1);
  }
  g_prof.clear();
  if (on < 0 || on >= 2 + kProfCount) return OS3D_EINVAL;
  g_prof_mode = on;
  return OS3D_OK;
}

int profile_get(int idx, const char** name, long long* launches, double* total_ms, double* alg_bytes,
                double* alg_flops) {
  if (idx < 0 || idx >= kProfCount) return OS3D_EINVAL;
  *name = kKernelNames[idx];
  long long n = 0;
  double ms = 0.0, by = 0.0, fl = 0.0;
  for (auto& r : g_prof) {
    if (r.kid != idx) continue;
    float t = 0.f;
    if (hipEventSynchronize(r.e1) != hipSuccess || hipEventElapsedTime(&t, r.e0, r.e1) != hipSuccess) return OS3D_EDEVICE;
    ++n;
    ms += t;
    by += r.alg_bytes;
    fl += r.alg_flops;
  }
  *launches = n;
  *total_ms = ms;
  *alg_bytes = by;
  *alg_flops = fl;
  return OS3D_OK;
}

int profile_count() { return kProfCount; }

}  // namespace os3d
