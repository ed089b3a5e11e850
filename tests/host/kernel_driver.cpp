// Runs the general transform (kernels_fft.hip, kernels_line.hip,
// kernels_tile.hip) on the CPU through the stand-in runtime of tests/host/emu,
// in ascending and in descending order of workgroups, waves and lanes.
//
//   kernel_driver NZ NY NX ROWS PAIRED ROUTE SPLIT BATCH [ONLY]
//
// ROUTE: 0 y and x lines, 2 whole planes; SPLIT: factor of y that goes with the
// z lines (ROUTE 0); ONLY: run the results whose names begin with it.  Prints one line per result: its name, the relative L2
// distance from 64-bit sums (16-bit scores: of the dequantised scores), whether
// the two orders agree bit for bit, and a checksum of its bytes.  The workspace
// has the size that workspace_bytes() asks for, with guard bytes behind it.
#include <complex>
#include <random>
#include <string>

#include "fft_pass.h"
#include "fft_tile.h"

dim3 threadIdx, blockIdx, blockDim, gridDim;
namespace emu {
int compute_units = 3;  // few, so that the persistent kernels loop
bool reversed = false;
Fibers fibers;
}  // namespace emu

namespace os3d {
alignas(256) float2 lds[(emu::kLds + emu::kGuard) / sizeof(float2)];
void set_error(const std::string& m) { emu::fail(m.c_str()); }
// not reached: 256^3 and the 64^2 and 128^2 planes
int forward4(const os3d_bank*, const float*, int, void*, int, float*, void*, int, void*) { emu::fail("256^3"); }
int reduce4(const os3d_bank*, const void*, int, const float*, int, float*, void*, bool, int, void*) {
  emu::fail("256^3");
}
int process4(const os3d_bank*, const float*, int, int, float, float*, void*, int, void*) { emu::fail("256^3"); }
template <int LM, int SM>
void launch_plane(const PassArgs&, int, hipStream_t) { emu::fail("64^2 and 128^2 planes"); }
template void launch_plane<LM_REAL, SM_C>(const PassArgs&, int, hipStream_t);
template void launch_plane<LM_C, SM_UOUT>(const PassArgs&, int, hipStream_t);
template void launch_plane<LM_C, SM_REAL>(const PassArgs&, int, hipStream_t);
template void launch_plane<LM_UIN, SM_C>(const PassArgs&, int, hipStream_t);
void launch_plane_phi(const PassArgs&, int, hipStream_t) { emu::fail("64^2 and 128^2 planes"); }
}  // namespace os3d

using namespace os3d;
typedef std::complex<double> cd;

static int dim[3];
static long long V;
static std::string only;

// DFT of a volume along the three axes, exponent sgn
static void dft3(std::vector<cd>& a, int sgn) {
  for (int ax = 0; ax < 3; ++ax) {
    const int N = dim[ax];
    long long st = 1;
    for (int k = ax + 1; k < 3; ++k) st *= dim[k];
    std::vector<cd> w(N), in(N);
    for (int i = 0; i < N; ++i) w[i] = std::polar(1.0, sgn * 2 * M_PI * i / N);
    for (long long o = 0; o < V; ++o) {
      if (o / st % N) continue;
      for (int i = 0; i < N; ++i) in[i] = a[o + i * st];
      for (int k = 0; k < N; ++k) {
        cd s = 0;
        for (int i = 0; i < N; ++i) s += in[i] * w[(long long)i * k % N];
        a[o + k * st] = s;
      }
    }
  }
}

struct Guarded {  // device memory: NaN, then guard bytes
  std::vector<unsigned char> m;
  size_t n;
  explicit Guarded(size_t bytes) : m(bytes + 4096, emu::kCanary), n(bytes) { std::fill(m.begin(), m.begin() + n, emu::kNaN); }
  template <class T>
  T* as() { return (T*)m.data(); }
  void check() const {
    for (size_t i = n; i < m.size(); ++i)
      if (m[i] != emu::kCanary) emu::fail("a write past a buffer");
  }
};

static unsigned long long checksum(const Guarded& g) {
  unsigned long long h = 1469598103934665603ull;  // FNV-1a
  for (size_t i = 0; i < g.n; ++i) h = (h ^ g.m[i]) * 1099511628211ull;
  return h;
}

template <class A, class B>
static double rel(const A& a, const B& b) {
  double d = 0, n = 0;
  for (size_t i = 0; i < b.size(); ++i) {
    d += std::norm(cd(a[i]) - cd(b[i]));
    n += std::norm(cd(b[i]));
  }
  return std::sqrt(d / n);
}

// call(ws) writes its outputs to the buffers out: run in both orders, print a line
template <class Call, class Err>
static void both(const char* name, size_t ws_bytes, std::vector<Guarded*> out, Call call, Err err) {
  if (std::string(name).compare(0, only.size(), only) != 0) return;
  unsigned long long sum[2] = {0, 0};
  double e = 0;
  for (int o = 0; o < 2; ++o) {
    emu::reversed = o == 1;
    for (Guarded* g : out) std::fill(g->m.begin(), g->m.begin() + g->n, emu::kNaN);
    Guarded ws(ws_bytes);
    if (call(ws.as<void>()) != OS3D_OK) emu::fail("status");
    ws.check();
    for (Guarded* g : out) {
      g->check();
      sum[o] = sum[o] * 31 + checksum(*g);
    }
    if (o == 0) e = err();
  }
  std::printf("%s %.3e %s %016llx\n", name, e, sum[0] == sum[1] ? "same" : "DIFFERS", sum[0]);
  std::fflush(stdout);
}

int main(int argc, char** argv) {
  if (argc < 9) return 2;
  for (int d = 0; d < 3; ++d) dim[d] = std::atoi(argv[1 + d]);
  const int rows = std::atoi(argv[4]), paired = std::atoi(argv[5]), route = std::atoi(argv[6]),
            split = std::atoi(argv[7]), batch = std::atoi(argv[8]);
  if (argc > 9) only = argv[9];
  V = (long long)dim[0] * dim[1] * dim[2];
  const int no = paired ? 2 * rows : rows;
  std::mt19937 gen(7);
  std::normal_distribution<float> normal;
  auto fill = [&](size_t n, float scale) {
    std::vector<float> v(n);
    for (float& x : v) x = scale * normal(gen);
    return v;
  };
  os3d_bank b = {};
  std::vector<float> tw[3];
  for (int d = 0; d < 3; ++d) {
    b.dims[d] = dim[d];
    for (int i = 0; i < dim[d]; ++i) {
      tw[d].push_back((float)std::cos(-2 * M_PI * i / dim[d]));
      tw[d].push_back((float)std::sin(-2 * M_PI * i / dim[d]));
    }
    b.d.tw[d] = tw[d].data();
  }
  b.V = V;
  b.n_orients = no;
  b.n_unique = rows;
  b.paired = paired;
  b.plane = route;
  b.split = split;
  b.kappa = 1.25;
  b.params.eps = 0.5;
  for (int i = 0; i < no; ++i) b.partner.push_back(!paired ? -1 : i < rows ? i + rows : i - rows);
  for (int i = 0; i < rows; ++i) b.rep.push_back(i);
  std::vector<float> psi = fill((size_t)rows * V, 1.f), M = fill(V, 1.f), f = fill(batch * V, 1.f);
  for (float& m : M) m = std::fabs(m);
  b.d.psi = psi.data();
  b.d.M = M.data();
  std::vector<float> Uf = fill((size_t)batch * no * V * 2, 1.f);  // a score of no forward transform
  const size_t ws = workspace_bytes(&b);
  std::printf("workspace %lld %lld\n", (long long)ws, (long long)(ws / (8 * V)));

  const float kappa = (float)b.kappa, eps = (float)b.params.eps;
  std::vector<cd> U((size_t)batch * no * V);
  for (int bi = 0; bi < batch; ++bi) {
    std::vector<cd> F(f.begin() + bi * V, f.begin() + (bi + 1) * V);
    dft3(F, -1);
    for (int r = 0; r < rows; ++r) {
      std::vector<cd> T(V);
      for (long long k = 0; k < V; ++k) T[k] = F[k] * (double)psi[r * V + k] * (double)kappa / (double)V;
      dft3(T, 1);
      cd* u = &U[((size_t)bi * no + r) * V];
      std::copy(T.begin(), T.end(), u);
      if (paired) std::transform(T.begin(), T.end(), u + rows * V, [](cd z) { return std::conj(z); });
    }
  }
  // Re IDFT of the orientation sum (divided by max(M, eps))
  auto sum = [&](auto score, bool divide) {
    std::vector<cd> out;
    for (int bi = 0; bi < batch; ++bi) {
      std::vector<cd> X(V);
      for (int r = 0; r < rows; ++r) {
        std::vector<cd> T(V);
        for (long long x = 0; x < V; ++x) {
          T[x] = score(((size_t)bi * no + r) * V + x);
          if (paired) T[x] += std::conj(score(((size_t)bi * no + r + rows) * V + x));
        }
        dft3(T, -1);
        for (long long k = 0; k < V; ++k) X[k] += T[k] * (double)psi[r * V + k] * (double)kappa;
      }
      if (divide)
        for (long long k = 0; k < V; ++k) X[k] /= (double)std::max(M[k], eps);
      dft3(X, 1);
      for (long long x = 0; x < V; ++x) out.push_back(X[x].real() / (double)V);
    }
    return out;
  };

  Guarded gU((size_t)batch * no * V * 8), gQ((size_t)batch * no * V * 4), gs((size_t)batch * no * 4),
      gr((size_t)batch * V * 4);
  both("forward_c64", ws, {&gU},
       [&](void* w) { return launch_forward(&b, f.data(), batch, gU.as<void>(), OS3D_C64, nullptr, w, nullptr); },
       [&]() {
         std::vector<cd> g;
         for (size_t i = 0; i < U.size(); ++i) g.push_back(cd(gU.as<float2>()[i].x, gU.as<float2>()[i].y));
         return rel(g, U);
       });
  auto real_err = [&](const std::vector<cd>& want) {
    return rel(std::vector<float>(gr.as<float>(), gr.as<float>() + batch * V), want);
  };
  auto given = [&](size_t i) { return cd(Uf[2 * i], Uf[2 * i + 1]); };
  for (int divide = 0; divide < 2; ++divide)
    both(divide ? "reconstruct_c64" : "adjoint_c64", ws, {&gr},
         [&](void* w) {
           return launch_reduce(&b, Uf.data(), OS3D_C64, nullptr, batch, gr.as<float>(), w, divide == 1, nullptr);
         },
         [&]() { return real_err(sum(given, divide == 1)); });
  // the least workspace of a reduction: the sum and one intermediate
  both("reconstruct_one_pair", 16 * V, {&gr},
       [&](void* w) {
         return launch_reduce(&b, Uf.data(), OS3D_C64, nullptr, batch, gr.as<float>(), w, true, nullptr,
                              reduce_pair_batch(&b, 16 * V));
       },
       [&]() { return real_err(sum(given, true)); });
  for (int kind = 0; kind < 2; ++kind) {
    const double p = 1.5;
    both(kind ? "process_soft" : "process_identity", ws, {&gr},
         [&](void* w) { return launch_process(&b, f.data(), batch, kind, (float)p, gr.as<float>(), w, nullptr); },
         [&]() {
           return real_err(
               sum([&](size_t i) { return kind ? U[i] * std::pow(std::abs(U[i]), p - 1.0) : U[i]; }, true));
         });
  }
  for (int dt : {OS3D_BF16X2, OS3D_F16X2}) {
    const std::string t = dt == OS3D_BF16X2 ? "bf16" : "fp16";
    auto value = [&](size_t i) {
      const float2 v = dt == OS3D_BF16X2 ? load_score<OS3D_BF16X2>(gQ.as<void>(), (long long)i, gs.as<float>()[i / V])
                                         : load_score<OS3D_F16X2>(gQ.as<void>(), (long long)i, gs.as<float>()[i / V]);
      return cd(v.x, v.y);
    };
    std::vector<cd> Uq;
    both(("forward_" + t).c_str(), ws, {&gQ, &gs},
         [&](void* w) { return launch_forward(&b, f.data(), batch, gQ.as<void>(), dt, gs.as<float>(), w, nullptr); },
         [&]() {
           Uq.clear();
           for (size_t i = 0; i < U.size(); ++i) Uq.push_back(value(i));
           return rel(Uq, U);
         });
    both(("reconstruct_" + t).c_str(), ws, {&gr},
         [&](void* w) {
           return launch_reduce(&b, gQ.as<void>(), dt, gs.as<float>(), batch, gr.as<float>(), w, true, nullptr);
         },
         [&]() { return real_err(sum([&](size_t i) { return value(i); }, true)); });
  }
  return 0;
}
