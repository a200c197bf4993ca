// Entry points of the CPU build for tests of single kernels and host functions.
#include <cmath>
#include <random>
#include <vector>

#include "common.h"
#include "engine.h"
#include "frag_kernels.h"

using namespace rtcc3;

extern "C" long emu_launches(const char* name);
extern "C" void emu_reset_launches();
extern "C" size_t emu_memory_in_use();
extern "C" void emu_trial_ms(double of_one_workgroup);

namespace {

template <class T>
T* device(size_t n) {
  T* p = nullptr;
  RTCC3_HIP(hipMalloc(&p, n * sizeof(T)));
  return p;
}
template <class T>
T* device(const std::vector<T>& x) {
  T* p = device<T>(x.size());
  std::memcpy(p, x.data(), x.size() * sizeof(T));
  return p;
}
std::vector<cplx> random(size_t n, unsigned seed) {
  std::mt19937 g(seed);
  std::normal_distribution<double> d;
  std::vector<cplx> x(n);
  for (auto& z : x) z = cplx{d(g), d(g)};
  return x;
}
void add(cplx& s, cplx a, cplx b) {
  s.re += a.re * b.re - a.im * b.im;
  s.im += a.re * b.im + a.im * b.re;
}

}  // namespace

// One block of a segmented product at window slot `slot`: the largest error of
// the block, in place of which nothing else is written.
extern "C" double drive_seg_slot(int v, int slot) {
  const int vp = (v + 7) / 8 * 8, len = 5;
  const int64_t va = (int64_t)v * vp, vb = va * v;
  const std::vector<cplx> A = random((size_t)v * len, 1), B = random((size_t)len * v * v, 2);
  cplx* C = device<cplx>((slot + 1) * vb);
  GemmDesc g;
  std::memset(&g, 0, sizeof(g));
  g.M = g.M0 = g.N0 = v;
  g.N = v * v;
  g.K = g.K0 = len;
  g.batch = 1;
  g.bl = device<int>({0, 0, 0, slot});
  g.alpha = cplx{1, 0};
  g.store = 1;
  g.nseg = 1;
  g.seg[0].len = len;
  g.seg[0].A = device(A);
  g.seg[0].sAm = len;
  g.seg[0].sAk = 1;
  g.seg[0].B = device(B);
  g.seg[0].sBk = v * v;
  g.seg[0].sBn = 1;
  g.C = C;
  g.sCm0 = va;
  g.sCn1 = vp;
  g.sCn0 = 1;
  g.cC[3] = vb;
  const int nt = (v + kFragRows - 1) / kFragRows;
  std::vector<int> rt;
  for (int t = 0; t < nt; ++t) rt.insert(rt.end(), {0, 1, 0, nt});
  frag_seg(g, device(rt), nt, nullptr);
  double err = 0;
  for (int a = 0; a < v; ++a)
    for (int n = 0; n < v * v; ++n) {
      cplx s{0, 0};
      for (int k = 0; k < len; ++k) add(s, A[a * len + k], B[k * v * v + n]);
      const cplx c = C[slot * vb + a * va + n / v * vp + n % v];
      err = std::max(err, std::hypot(c.re - s.re, c.im - s.im));
    }
  RTCC3_HIP(hipFree(C));
  return err;
}

// A derivative evaluation that ends in an error while its clearing is queued,
// then another one: how far the derivative is from alpha x'.
extern "C" double drive_dropped_queue(int of_gradient) {
  Engine e(nullptr);
  const int64_t n = 6;
  View x = e.tensor("x", {n}), y = e.tensor("y", {n});
  View out = y;
  if (of_gradient) {
    e.set_requires_grad(y.buf, true);
    out = e.grad(y);
  }
  e.enable_twins();
  e.set_tangent(true);
  cplx* xt = e.twin_out(x.p);
  for (int64_t i = 0; i < n; ++i) xt[i] = cplx{1.0 + i, -2.0};
  double err = 0;
  for (int pass = 0; pass < 3; ++pass) {
    try {
      Engine::Queue queued(e);
      e.start_queue();
      e.zero_later(out);
      if (pass == 1) throw Error(-3, "a device error");
      e.axpy(cplx{2, 0}, x, out);
      e.settle();
    } catch (const Error&) {
      continue;
    }
    const cplx* t = e.twin(out.p);
    for (int64_t i = 0; i < n; ++i)
      err = std::max(err, t ? std::hypot(t[i].re - 2 * xt[i].re, t[i].im - 2 * xt[i].im) : 1.0);
  }
  return err;
}

// Products C += A B and C += D E of M x K by K x N, tuned one by one and then
// queued into one level: launches of a product by itself and of several
// together, and the largest error.  ms: what the trial of one workgroup takes,
// of more of them less (0: not tuned).
extern "C" double drive_tuned_level(int M, int N, int K, double ms, long launches[2]) {
  Engine e(nullptr);
  View X[4], C = e.tensor("C", {M, N});
  std::vector<cplx> h[4];
  for (int q = 0; q < 4; ++q) {
    const int r = q % 2 == 0 ? M : K, c = q % 2 == 0 ? K : N;
    X[q] = e.tensor(std::string(1, 'p' + q), {r, c});
    h[q] = random((size_t)r * c, 7 + q);
    std::memcpy(X[q].p, h[q].data(), h[q].size() * sizeof(cplx));
  }
  Tuner* t = tuner_new();
  TunerScope scope(t);
  emu_trial_ms(ms);
  auto evaluate = [&]() {
    Engine::Queue queued(e);
    e.zero(C);
    e.start_queue();
    e.einsum("mk,kn->mn", cplx{1, 0}, X[0], X[1], C);
    e.einsum("mk,kn->mn", cplx{1, 0}, X[2], X[3], C);
    e.settle();
  };
  tuner_set_tuning(t, ms > 0);
  evaluate();
  tuner_set_tuning(t, false);
  emu_reset_launches();
  evaluate();
  launches[0] = emu_launches("frag_gemm_kernel");
  launches[1] = emu_launches("frag_group_kernel");
  double err = 0;
  for (int m = 0; m < M; ++m)
    for (int n = 0; n < N; ++n) {
      cplx s{0, 0};
      for (int q = 0; q < 4; q += 2)
        for (int k = 0; k < K; ++k) add(s, h[q][m * K + k], h[q + 1][k * N + n]);
      const cplx c = C.p[m * N + n];
      err = std::max(err, std::hypot(c.re - s.re, c.im - s.im));
    }
  tuner_delete(t);
  return err;
}

// A sum over three runs of indices, Y[i][a] = sum_bde Z[i][b][d][e] W[d][a][e][b]:
// the device memory it takes beside its operands, and the largest error.
extern "C" double drive_three_runs(int o, int v, size_t* extra) {
  Engine e(nullptr);
  View Z = e.tensor("Z", {o, v, v, v}), W = e.tensor("W", {v, v, v, v}), Y = e.tensor("Y", {o, v});
  const std::vector<cplx> z = random(Z.numel(), 3), w = random(W.numel(), 4);
  std::memcpy(Z.p, z.data(), z.size() * sizeof(cplx));
  std::memcpy(W.p, w.data(), w.size() * sizeof(cplx));
  const size_t before = emu_memory_in_use();
  e.einsum("ibde,daeb->ia", cplx{1, 0}, Z, W, Y);
  *extra = emu_memory_in_use() - before;
  double err = 0;
  for (int i = 0; i < o; ++i)
    for (int a = 0; a < v; ++a) {
      cplx s{0, 0};
      for (int b = 0; b < v; ++b)
        for (int d = 0; d < v; ++d)
          for (int x = 0; x < v; ++x) add(s, z[((i * v + b) * v + d) * v + x], w[((d * v + a) * v + x) * v + b]);
      err = std::max(err, std::hypot(Y.p[i * v + a].re - s.re, Y.p[i * v + a].im - s.im));
    }
  return err;
}
