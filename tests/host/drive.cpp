// Entry points of the CPU build for tests of single kernels and host functions.
#include <algorithm>
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

namespace {

// A plain product whose indices m, n and k are split in two levels each, with
// the dimensions of its operands in any order, dense or with gaps, several
// entries with an output each or one for all.
struct Product {
  GemmDesc g;
  std::vector<cplx> A, B, before;
  int64_t nC = 0;
  bool adds;
};

// Strides of the dimensions of x, the one listed first in `order` slowest, each
// slower one with `gap` more than it needs; returns the elements spanned.
int64_t lay(const int* x, int64_t* stride, const int* order, int nd, int gap) {
  int64_t s = 1;
  for (int q = nd - 1; q >= 0; --q) {
    stride[order[q]] = s;
    s *= x[order[q]] + (q > 0 ? gap : 0);
  }
  return s;
}

Product make(std::mt19937& r, const int* e, int batch, int form) {  // e: M1, M0, N1, N0, K1, K0
  Product p;
  GemmDesc& g = p.g;
  std::memset(&g, 0, sizeof(g));
  g.M = e[0] * e[1];
  g.M0 = e[1];
  g.N = e[2] * e[3];
  g.N0 = e[3];
  g.K = e[4] * e[5];
  g.K0 = e[5];
  g.batch = batch;
  auto order = [&](int* o) {
    for (int q = 0; q < 5; ++q) o[q] = q;
    std::shuffle(o, o + 5, r);
  };
  int o[5];
  int64_t s[5];
  const int a[5] = {e[0], e[1], e[4], e[5], batch}, b[5] = {e[4], e[5], e[2], e[3], batch};
  const bool one = form & 1;  // one output for all entries
  const int c[5] = {e[0], e[1], e[2], e[3], one ? 1 : batch};
  order(o);
  p.A = random(lay(a, s, o, 5, form >> 1 & 1), r());
  g.sAm1 = s[0], g.sAm0 = s[1], g.sAk1 = s[2], g.sAk0 = s[3], g.sAb = s[4];
  order(o);
  p.B = random(lay(b, s, o, 5, form >> 2 & 1), r());
  g.sBk1 = s[0], g.sBk0 = s[1], g.sBn1 = s[2], g.sBn0 = s[3], g.sBb = s[4];
  order(o);
  const bool fresh = form >> 3 & 1;
  p.nC = lay(c, s, o, 5, fresh ? 0 : form >> 4 & 1);
  g.sCm1 = s[0], g.sCm0 = s[1], g.sCn1 = s[2], g.sCn0 = s[3], g.sCb = one ? 0 : s[4];
  p.before = random(p.nC, r());
  if (fresh)
    for (auto& z : p.before) z = cplx{std::nan(""), std::nan("")};
  g.A = device(p.A);
  g.B = device(p.B);
  g.C = device(p.before);
  g.alpha = cplx{0.5, form & 32 ? -1.5 : 0.0};
  g.atomic = one && batch > 1;
  g.fresh = fresh;
  g.fresh_p = g.C;
  g.fresh_n = p.nC;
  g.prec = RTCC3_PREC_FP64;
  p.adds = !fresh;
  return p;
}

// The largest error of C in units of the bound on rounding; other elements of C stay.
double check(const Product& p) {
  const GemmDesc& g = p.g;
  std::vector<cplx> want(p.nC), size(p.nC);
  std::vector<char> mine(p.nC);
  for (int b = 0; b < g.batch; ++b)
    for (int m = 0; m < g.M; ++m)
      for (int n = 0; n < g.N; ++n) {
        const int64_t at = b * g.sCb + m / g.M0 * g.sCm1 + m % g.M0 * g.sCm0 + n / g.N0 * g.sCn1 + n % g.N0 * g.sCn0;
        cplx s{0, 0};
        for (int k = 0; k < g.K; ++k) {
          const cplx x = p.A[b * g.sAb + m / g.M0 * g.sAm1 + m % g.M0 * g.sAm0 + k / g.K0 * g.sAk1 + k % g.K0 * g.sAk0];
          const cplx y = p.B[b * g.sBb + n / g.N0 * g.sBn1 + n % g.N0 * g.sBn0 + k / g.K0 * g.sBk1 + k % g.K0 * g.sBk0];
          add(s, x, y);
          size[at].re += std::hypot(x.re, x.im) * std::hypot(y.re, y.im);
        }
        add(want[at], s, g.alpha);
        mine[at] = 1;
      }
  double worst = 0;
  for (int64_t i = 0; i < p.nC; ++i) {
    if (p.adds || !mine[i]) want[i].re += p.before[i].re, want[i].im += p.before[i].im;
    const double err = std::hypot(g.C[i].re - want[i].re, g.C[i].im - want[i].im);
    // each term passes as many roundings of sums of at most twice its size as
    // there are terms (three real products per complex one), and alpha's
    const double before = p.adds ? std::hypot(p.before[i].re, p.before[i].im) : 0.0;
    const double bound =
        mine[i] ? 8 * (g.K * g.batch + 8) * 2.3e-16 * (std::hypot(g.alpha.re, g.alpha.im) * size[i].re + before) : 0.0;
    if (!(err <= bound)) worst = std::max(worst, std::isfinite(err) && bound > 0 ? err / bound : 1e300);
  }
  return worst;
}

void drop(const Product& p) {
  (void)hipFree(const_cast<cplx*>(p.g.A));
  (void)hipFree(const_cast<cplx*>(p.g.B));
  (void)hipFree(p.g.C);
}

}  // namespace

// `count` products of random forms, one by one and four to a level; the largest error.
extern "C" double drive_products(int seed, int count) {
  std::mt19937 r(seed);
  const int outer[] = {1, 1, 2, 3, 5}, inner[] = {1, 2, 3, 4, 7, 8, 15, 16, 17, 33}, steps[] = {1, 2, 3, 4, 5, 8, 13, 32};
  double worst = 0;
  std::vector<Product> level;
  for (int i = 0; i < count; ++i) {
    const int e[6] = {outer[r() % 5], inner[r() % 10], outer[r() % 5], inner[r() % 10], outer[r() % 5], steps[r() % 8]};
    Product p = make(r, e, r() % 3 == 0 ? 2 + r() % 3 : 1, (int)(r() % 64));
    RTCC3_CHECK(frag_gemm_fits(p.g), "not a product for the kernel");
    if (i % 2) {
      level.push_back(std::move(p));
      if (level.size() < 4) continue;
      std::vector<GemmDesc> g;
      for (auto& q : level) g.push_back(q.g);
      gemm_group(g.data(), (int)g.size(), nullptr);
      for (auto& q : level) worst = std::max(worst, check(q)), drop(q);
      level.clear();
    } else {
      gemm(p.g, nullptr);
      worst = std::max(worst, check(p));
      drop(p);
    }
  }
  for (auto& q : level) drop(q);
  return worst;
}

// One product of given extents (M1, M0, N1, N0, K1, K0), split of k as given (0: the kernel's choice).
extern "C" double drive_product(const int* e, int batch, int form, int ksplit) {
  std::mt19937 r(17);
  Product p = make(r, e, batch, form);
  if (ksplit > 0)
    frag_gemm(p.g, ksplit, nullptr);
  else
    gemm(p.g, nullptr);
  const double worst = check(p);
  drop(p);
  return worst;
}

// Block products of four groups with traces, all groups in a launch and (reach
// of a panel) one group at a time; the launches and the largest error.
extern "C" double drive_block(int o, int v, int one_by_one, long* launches) {
  const int vp = (v + 7) / 8 * 8, nb = o * o * o;
  const int64_t v2 = (int64_t)v * v, vb = v2 * vp, ov2 = o * v2;
  std::vector<int> bl, part;
  for (int i = 0; i < o; ++i)
    for (int j = 0; j < o; ++j)
      for (int k = 0; k < o; ++k) {
        const int n = (int)bl.size() / 4;
        bl.insert(bl.end(), {i, j, k, n});
        for (int q = 0; q < 6; ++q) part.push_back((n + q) % nb);
      }
  const std::vector<cplx> X = random(nb * vb, 1), B0 = random(o * ov2, 2), B1 = random(o * ov2, 3);
  const cplx *d0 = device(B0), *d1 = device(B1);
  const int64_t nC = (int64_t)o * o * v * o;
  std::vector<cplx*> C;
  for (int q = 0; q < 4; ++q) C.push_back(device<cplx>(nC));
  cplx *t0 = device<cplx>(o * v), *t1 = device<cplx>(o * v);
  const int64_t vo = (int64_t)v * o, ovo = o * vo;
  const BlockCols groups[4] = {{d0, 0, ov2, v2, C[0], {0, ovo, vo}, o, 1, 1.0},
                               {d1, 1, ov2, v2, C[1], {vo, 0, ovo}, o, 1, -1.0},
                               {d0, 0, v2, ov2, C[2], {0, ovo, vo}, o, 1, 0.5},
                               {d0, 2, v2, ov2, C[3], {ovo, vo, 0}, o, 1, 2.0}};
  const BlockTrace traces[4] = {{1, 2, 0, t0, v, 1.0}, {1, 0, 2, t0, v, -1.0}, {3, 1, 0, t1, v, 0.25}, {3, 0, 1, t1, v, -1.0}};
  cplx* pack = device<cplx>(frag_block_pack(groups, 4, o, o, v));
  const int perm = 5;
  *launches = frag_block(groups, 4, o, traces, 4, device(X), perm, o, v, vp, device(part), device(bl), nb, pack, nullptr,
                         one_by_one ? 1 : (int64_t)1 << 32);
  std::vector<std::vector<cplx>> want(6, std::vector<cplx>(nC));
  for (int n = 0; n < nb; ++n)
    for (int g = 0; g < 4; ++g)
      for (int x = 0; x < o; ++x)
        for (int b = 0; b < v; ++b) {
          const int* q = &bl[4 * n];
          const BlockCols& c = groups[g];
          const std::vector<cplx>& src = c.B == d0 ? B0 : B1;
          cplx s{0, 0};
          for (int k = 0; k < v2; ++k) add(s, X[part[6 * n + perm] * vb + (int64_t)k * vp + b], src[q[c.key] * c.sKey + x * c.sB + k]);
          add(want[g][c.cC[0] * q[0] + c.cC[1] * q[1] + c.cC[2] * q[2] + b * c.sCm + x * c.sCx], s, cplx{c.alpha, 0});
          for (const BlockTrace& t : traces)
            if (t.group == g && x == q[t.col]) add(want[t.C == t0 ? 4 : 5][q[t.row] * t.sC + b], s, cplx{t.alpha, 0});
        }
  double err = 0;
  for (int g = 0; g < 6; ++g) {
    const cplx* c = g < 4 ? C[g] : g == 4 ? t0 : t1;
    for (int64_t i = 0; i < (g < 4 ? nC : o * v); ++i)
      err = std::max(err, std::hypot(c[i].re - want[g][i].re, c[i].im - want[g][i].im));
  }
  return err;
}

// The error code of a sum over three runs of indices of the given extents (0: none).
extern "C" int drive_three_runs_extent(int b, int d, int x) {
  Engine e(nullptr);
  View Z = e.tensor("Z", {1, b, d, x}), W = e.tensor("W", {d, 2, x, b}), Y = e.tensor("Y", {1, 2});
  try {
    e.einsum("ibde,daeb->ia", cplx{1, 0}, Z, W, Y);
  } catch (const Error& err) {
    return err.code;
  }
  return 0;
}
