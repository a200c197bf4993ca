// Generic kernels: batched complex GEMM on the matrix cores (FP32 MFMA with the
// complex product as four real products, bf16 slices; FP64 with three for what
// frag_kernels.hip does not take), strided axpy/permute, fill.
#include <algorithm>
#include <type_traits>
#include <unordered_map>
#include <vector>

#include "common.h"
#include "frag_kernels.h"

namespace rtcc3 {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));

namespace {

constexpr int BM = 64, NT = 256;
constexpr int GK_MAXSEG = 256;  // gathered blocks one workgroup's K range may touch

template <typename T>
struct Frag;
template <>
struct Frag<double> {
  typedef d4 acc;
  static __device__ __forceinline__ acc mfma(double a, double b, acc c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int lane, int r) { return 4 * r + (lane >> 4); }
};
template <>
struct Frag<float> {
  typedef f4 acc;
  static __device__ __forceinline__ acc mfma(float a, float b, acc c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int lane, int r) { return 4 * (lane >> 4) + r; }
};

__device__ __forceinline__ void atomic_add_cplx(cplx* p, double re, double im) {
  unsafeAtomicAdd(&p->re, re);
  unsafeAtomicAdd(&p->im, im);
}

// Split k = q*K0 + r for 0 <= k < 2^22 without an integer divide: the float
// estimate of the quotient is off by at most one, corrected either way.
__device__ __forceinline__ void split_k(int k, int K0, float inv, int& q, int& r) {
  q = (int)((float)k * inv);
  r = k - q * K0;
  q = r < 0 ? q - 1 : q;
  r = r < 0 ? r + K0 : r;
  q = r >= K0 ? q + 1 : q;
  r = r >= K0 ? r - K0 : r;
}

// Operands of one 64 x BN tile of C for one batch entry, brought into
// registers BK values of k at a time.  Element r of a thread sits at
// (akk[r], amm[r]) of the A tile and (bkk[r], bnn[r]) of the B tile.
// KFA: A is read with k as the fast thread index (unit stride in k), so all
// of a thread's A elements share one k; else they share one m.  NFB: B is read
// with n as the fast thread index, else k.  SEG: the operands come from the K
// segments of the descriptor (read with A k-fast, B n-fast).
// Every load is issued: an element outside the operand reads offset 0 of its
// entry (the empty asm keeps the compiler from turning the address select
// back into a branch around the load) and is then replaced by zero.
// CMB = 1 / 2: operand A / B is a combination of three blocks (GemmDesc::comb_*);
// CMB = 3: gathered K (GemmDesc::gk_*); CMB = 4: B is one block of a permuted
// occupied triple (comb_n = 1).
template <bool KFA, bool NFB, int BN, int BK, bool SEG, int CMB = 0>
struct TileLoader {
  static constexpr int NEA = BM * BK / NT, NEB = BN * BK / NT;
  static constexpr int NKA = KFA ? 1 : NEA, NMA = KFA ? NEA : 1;
  static constexpr int NKB = NFB ? NEB : 1, NNB = NFB ? 1 : NEB;
  int akk[NEA], amm[NEA], bkk[NEB], bnn[NEB];
  int64_t aoff[NMA], boff[NNB];
  bool aval[NMA], bval[NNB];
  const cplx* A;
  const cplx* B;
  const cplx* Ap[4];  // K-segment bases of this entry
  const cplx* Bp[4];
  const cplx* Xc[3];  // bases of the combined operand's blocks
  double wc[3];
  const cplx* Bq[NNB];   // column segments: B base of each loaded column, and its k stride
  int sbq[NNB];
  int gs;                // first gathered block of the entry
  int gq0;               // first gathered block of this workgroup's K range
  const int64_t* gofs;   // LDS: A and B offsets of the gathered blocks from gq0 on
  int kend, sk1, sk2, sk3, m0, n0;
  float invK0;
  cplx av[NEA], bv[NEB];
  // CMB = 1 / 2: the three loaded parts of each combined element, combined
  // only when the tile is stored (settle), so that the loads stay in flight
  // during the MFMAs instead of being waited for right away
  static constexpr int NX = CMB == 1 ? NEA : CMB == 2 ? NEB : 1;
  cplx xr[NX][3];
  bool xok[NX];

  // Returns the entry's C base.
  __device__ __forceinline__ cplx* init(const GemmDesc& d, int64_t b, int tm, int tn, int kend_) {
    kend = kend_;
    m0 = tm * BM;
    n0 = tn * BN;
    invK0 = 1.0f / (float)d.K0;
    cplx* C;
    A = B = nullptr;
#pragma unroll
    for (int s = 0; s < 4; ++s) Ap[s] = Bp[s] = nullptr;
    if (d.bl) {
      const int I = d.bl[4 * b], J = d.bl[4 * b + 1], K = d.bl[4 * b + 2], n = d.bl[4 * b + 3];
      C = d.C + d.cC[0] * I + d.cC[1] * J + d.cC[2] * K + d.cC[3] * n;
      if (SEG) {
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const GemmDesc::Seg& g = d.seg[s < d.nseg ? s : 0];
          Ap[s] = g.A + g.cA[0] * I + g.cA[1] * J + g.cA[2] * K + g.cA[3] * n;
          Bp[s] = g.B + g.cB[0] * I + g.cB[1] * J + g.cB[2] * K + g.cB[3] * n;
        }
      } else {
        A = d.A + d.cA[0] * I + d.cA[1] * J + d.cA[2] * K + d.cA[3] * n;
        B = d.B + d.cB[0] * I + d.cB[1] * J + d.cB[2] * K + d.cB[3] * n;
      }
      if (CMB == 3) {
        A = d.A;
        B = d.B;
        gs = d.gk_start[b];
      }
      if (CMB == 4) B = d.B + (int64_t)d.part[6 * n + d.comb_perm[0]] * d.comb_stride;
      if (CMB == 1 || CMB == 2) {
#pragma unroll
        for (int s = 0; s < 3; ++s) {
          Xc[s] = (CMB == 1 ? d.A : d.B) + (int64_t)d.part[6 * n + d.comb_perm[s]] * d.comb_stride;
          wc[s] = d.comb_w[s];
        }
        if (CMB == 1) A = Xc[0];
        if (CMB == 2) B = Xc[0];
      }
    } else {
      A = d.A + b * d.sAb;
      B = d.B + b * d.sBb;
      C = d.C + b * d.sCb;
    }
    // segment starts; unused segments start at INT_MAX
    sk1 = d.nseg > 1 ? d.seg[1].k0 : 0x7fffffff;
    sk2 = d.nseg > 2 ? d.seg[2].k0 : 0x7fffffff;
    sk3 = d.nseg > 3 ? d.seg[3].k0 : 0x7fffffff;
    const int tid = threadIdx.x;
#pragma unroll
    for (int r = 0; r < NEA; ++r) {
      const int e = tid + NT * r;
      amm[r] = KFA ? e / BK : e % BM;
      akk[r] = KFA ? e % BK : e / BM;
    }
#pragma unroll
    for (int r = 0; r < NEB; ++r) {
      const int e = tid + NT * r;
      bnn[r] = NFB ? e % BN : e / BK;
      bkk[r] = NFB ? e / BN : e % BK;
    }
#pragma unroll
    for (int r = 0; r < NMA; ++r) {
      const int m = m0 + amm[r];
      aval[r] = m < d.M;
      aoff[r] = aval[r] ? (int64_t)(m / d.M0) * d.sAm1 + (int64_t)(m % d.M0) * d.sAm0 : 0;
    }
#pragma unroll
    for (int r = 0; r < NNB; ++r) {
      const int n = n0 + bnn[r];
      bval[r] = n < d.N;
      boff[r] = bval[r] ? (int64_t)(n / d.N0) * d.sBn1 + (int64_t)(n % d.N0) * d.sBn0 : 0;
    }
    if (CMB == 5) {
      static_assert(CMB != 5 || (!NFB && BN == 64 && NNB == 4), "column segments: B k-fast, 64-wide tiles");
      // entry r of a thread is column bnn[r] = 16 r + tid / 16, i.e. column
      // tid / 16 of segment r; masked columns read the entry's own A base
      const int I = d.bl[4 * b], J = d.bl[4 * b + 1], K = d.bl[4 * b + 2], n = d.bl[4 * b + 3];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const GemmDesc::ColSeg& g = d.cs[r];
        const int c = bnn[r] - 16 * r;
        const bool tail = r < d.ncs && c == 15 && g.tB;
        bval[r] = r < d.ncs && (c < g.n || tail);
        Bq[r] = !bval[r] ? A
                : tail   ? g.tB + g.tcB[0] * I + g.tcB[1] * J + g.tcB[2] * K + g.tcB[3] * n
                         : g.B + g.cB[0] * I + g.cB[1] * J + g.cB[2] * K + g.cB[3] * n + (int64_t)c * g.sBn;
        sbq[r] = !bval[r] ? 0 : tail ? (int)g.tsBk : (int)g.sBk;
      }
    }
    return C;
  }

  static __device__ __forceinline__ cplx fetch(const cplx* p, bool ok, int64_t off) {
    int64_t o = ok ? off : 0;
    asm volatile("" : "+v"(o));
    const cplx x = p[o];
    return cplx{ok ? x.re : 0.0, ok ? x.im : 0.0};
  }
  __device__ __forceinline__ void fetch3(int e, bool ok, int64_t off) {
    int64_t o = ok ? off : 0;
    asm volatile("" : "+v"(o));
    xr[e][0] = Xc[0][o];
    xr[e][1] = Xc[1][o];
    xr[e][2] = Xc[2][o];
    xok[e] = ok;
  }
  // Combined elements of the last load into av (CMB = 1) or bv (CMB = 2).
  __device__ __forceinline__ void settle() {
    if constexpr (CMB == 1 || CMB == 2) {
#pragma unroll
      for (int e = 0; e < NX; ++e) {
        const double re = wc[0] * xr[e][0].re + wc[1] * xr[e][1].re + wc[2] * xr[e][2].re;
        const double im = wc[0] * xr[e][0].im + wc[1] * xr[e][1].im + wc[2] * xr[e][2].im;
        const cplx x{xok[e] ? re : 0.0, xok[e] ? im : 0.0};
        if constexpr (CMB == 1)
          av[e] = x;
        else
          bv[e] = x;
      }
    }
  }
  // Offset of the q-th gathered block of the entry in operand x (0 = A, 1 = B).
  __device__ __forceinline__ int64_t gather_off(int x, int q) const { return gofs[2 * (q - gq0) + x]; }
  __device__ __forceinline__ int segof(int k) const { return (int)(k >= sk1) + (int)(k >= sk2) + (int)(k >= sk3); }
  template <typename X>
  static __device__ __forceinline__ X pick(int s, X x0, X x1, X x2, X x3) {
    return s == 0 ? x0 : s == 1 ? x1 : s == 2 ? x2 : x3;
  }

  __device__ __forceinline__ void load(const GemmDesc& d, int k0) {
    if (SEG) {
      static_assert(!SEG || (KFA && NFB), "segments are read with A k-fast and B n-fast");
      // Segments start at multiples of BK: the whole step lies in one segment,
      // whose operands, strides and length are uniform across the workgroup.
      const int s = segof(k0);
      const int base = pick(s, 0, sk1, sk2, sk3);
      const int len = pick(s, d.seg[0].len, d.seg[1].len, d.seg[2].len, d.seg[3].len);
      const cplx* pa = pick(s, Ap[0], Ap[1], Ap[2], Ap[3]);
      const cplx* pb = pick(s, Bp[0], Bp[1], Bp[2], Bp[3]);
      const int sam = (int)pick(s, d.seg[0].sAm, d.seg[1].sAm, d.seg[2].sAm, d.seg[3].sAm);
      const int sak = (int)pick(s, d.seg[0].sAk, d.seg[1].sAk, d.seg[2].sAk, d.seg[3].sAk);
      const int sbk = (int)pick(s, d.seg[0].sBk, d.seg[1].sBk, d.seg[2].sBk, d.seg[3].sBk);
      const int sbn = (int)pick(s, d.seg[0].sBn, d.seg[1].sBn, d.seg[2].sBn, d.seg[3].sBn);
      const int ka = k0 + akk[0], ra = ka - base;
      const bool oka = ka < kend && ra < len;
#pragma unroll
      for (int t = 0; t < NEA; ++t) av[t] = fetch(pa, oka && aval[t], (int64_t)((m0 + amm[t]) * sam + ra * sak));
      const int ncol = n0 + bnn[0];
#pragma unroll
      for (int t = 0; t < NEB; ++t) {
        const int kb = k0 + bkk[t], rb = kb - base;
        bv[t] = fetch(pb, kb < kend && rb < len && bval[0], (int64_t)(rb * sbk + ncol * sbn));
      }
      return;
    }
#pragma unroll
    for (int s = 0; s < NKA; ++s) {
      const int k = k0 + akk[s];
      int q, r;
      split_k(k, d.K0, invK0, q, r);
      const int64_t ko = CMB == 3 ? gather_off(0, k < kend ? q : gq0) + (int64_t)r * d.sAk0
                                  : (int64_t)q * d.sAk1 + (int64_t)r * d.sAk0;
#pragma unroll
      for (int t = 0; t < NMA; ++t) {
        const int e = KFA ? t : s;
        const bool ok = k < kend && aval[KFA ? t : 0];
        if constexpr (CMB == 1)
          fetch3(e, ok, aoff[KFA ? t : 0] + ko);
        else
          av[e] = fetch(A, ok, aoff[KFA ? t : 0] + ko);
      }
    }
#pragma unroll
    for (int s = 0; s < NKB; ++s) {
      const int k = k0 + bkk[s];
      int q, r;
      split_k(k, d.K0, invK0, q, r);
      const int64_t ko = CMB == 3 ? gather_off(1, k < kend ? q : gq0) + (int64_t)r * d.sBk0
                                  : (int64_t)q * d.sBk1 + (int64_t)r * d.sBk0;
#pragma unroll
      for (int t = 0; t < NNB; ++t) {
        const int e = NFB ? s : t;
        const bool ok = k < kend && bval[NFB ? 0 : t];
        if constexpr (CMB == 5)
          bv[e] = fetch(Bq[t], ok, (int64_t)k * sbq[t]);
        else if constexpr (CMB == 2)
          fetch3(e, ok, boff[NFB ? 0 : t] + ko);
        else
          bv[e] = fetch(B, ok, boff[NFB ? 0 : t] + ko);
      }
    }
  }
};

// C[m][n] (+)= alpha * x for one element of the tile.
// Offset of row m (or column n) of C split as (x / X0, x % X0); -1 outside.
__device__ __forceinline__ int64_t c_off(int x, int X, int X0, int64_t s1, int64_t s0) {
  if (x >= X) return -1;
  int q, r;
  split_k(x, X0, 1.0f / (float)X0, q, r);
  return (int64_t)q * s1 + (int64_t)r * s0;
}

// C[row + col] (+)= alpha * x for one element of the tile (offsets from c_off).
template <bool ATOMIC>
__device__ __forceinline__ void put(const GemmDesc& d, cplx* C, int64_t ro, int64_t co, double xr, double xi) {
  if (ro < 0 || co < 0) return;
  const double alr = d.alpha.re, ali = d.alpha.im;
  const double vr = alr * xr - ali * xi, vi = alr * xi + ali * xr;
  cplx* p = C + ro + co;
  if (ATOMIC) {
    atomic_add_cplx(p, vr, vi);
  } else if (d.store) {
    // store mode writes each element once and nothing in the same product reads
    // it: a streaming store leaves the cache lines to the operands
    typedef double d2v __attribute__((ext_vector_type(2)));
    __builtin_nontemporal_store(d2v{vr, vi}, reinterpret_cast<d2v*>(p));
  } else {
    cplx c = *p;
    c.re += vr;
    c.im += vi;
    *p = c;
  }
}

// One workgroup computes a 64 x BN tile of C for one batch entry.  BN = 64:
// waves arranged 2x2, each owning a 32x32 sub-tile = 2x2 MFMA 16x16 blocks;
// BN = 16 (narrow N, e.g. one occupied index): waves stacked 4x1, each owning
// one 16x16 block.  Every block has a real and an imaginary accumulator,
//   Cre += Are*Bre - Aim*Bim,  Cim += Are*Bim + Aim*Bre,
// and in FP64 a third, for the three-product form below.
// MFMA 16x16x4 operand layout: lane l holds A[l%16][l/16] and B[l/16][l%16].
// Result layout: FP32 holds D[4*(l/16)+r][l%16] in register r, FP64 holds
// D[4*r+l/16][l%16] (Frag<T>::row).
// Tiles of A and B go through two LDS buffers: while the MFMAs consume one,
// the next tile is loaded into registers and then stored into the other, so
// each K step needs one barrier.
// FP64: the workgroups per CU that the LDS tiles allow (160 KB per CU; one
// wave per SIMD each), at most three, to which the register allocation is held
// so that the scheduler does not trade that occupancy for registers.  FP32: no
// bound.
template <typename T, int BN, bool SEG, int CMB>
constexpr int zgemm_waves() {
  constexpr int lds = (SEG ? 1 : 2) * 2 * 16 * ((BM + 1) + (BN + 1)) * (int)sizeof(T) + (CMB == 3 ? 4096 : 0);
  return std::is_same<T, double>::value ? std::min(3, 160 * 1024 / lds) : 1;
}
template <typename T, bool ATOMIC, bool KFA, bool NFB, int BN, bool SEG, int CMB = 0>
__global__ __launch_bounds__(NT, (zgemm_waves<T, BN, SEG, CMB>())) void zgemm_kernel(GemmDesc d, int ksplit,
                                                                                  int kchunk) {
  typedef typename Frag<T>::acc acc_t;
  constexpr int BK = 16;
  // Wave sub-tile: 32x32 (2x2 MFMA blocks) in a 64x64 tile, 16x16 in a 64x16
  // tile; with column segments each wave takes 16 rows and all 64 columns, so
  // that a launch with fewer than four segments skips the MFMAs of the unused
  // 16-column blocks in every wave alike.
  constexpr int WM = CMB == 5 ? 16 : BN == 64 ? 32 : 16, WN = CMB == 5 ? BN : BN == 64 ? 32 : 16;
  constexpr int IB = WM / 16, JB = WN / 16;  // MFMA blocks per wave
  typedef TileLoader<KFA, NFB, BN, BK, SEG, CMB> Loader;
  // Segmented products keep one LDS buffer (two barriers per K step) so that
  // three workgroups fit on a CU; the others double-buffer.
  constexpr int NBUF = SEG ? 1 : 2;
  __shared__ T sA[NBUF][2][BK][BM + 1];  // [buffer][re, im][k][m]
  __shared__ T sB[NBUF][2][BK][BN + 1];  // [buffer][re, im][k][n]

  const int tilesN = (d.N + BN - 1) / BN;
  const int kz = blockIdx.x % ksplit;
  const int tile = blockIdx.x / ksplit;
  const int tm = tile / tilesN, tn = tile % tilesN;
  const int64_t b = (int64_t)blockIdx.y + (int64_t)blockIdx.z * gridDim.y;
  if (b >= d.batch) return;
  const int kbeg = kz * kchunk;
  const int Kb = CMB == 3 ? (d.gk_start[b + 1] - d.gk_start[b]) * d.K0 : d.K;  // this entry's contraction length
  const int kend = min(Kb, kbeg + kchunk);
  if (kbeg >= kend) return;

  Loader ld;
  cplx* C = ld.init(d, b, tm, tn, kend);
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int wm = (wave / (BN / WN)) * WM, wn = (wave % (BN / WN)) * WN;
  if (CMB == 3) {
    // operand offsets of the gathered blocks this workgroup's K range touches
    __shared__ int64_t gofs[2 * GK_MAXSEG];
    const int q0 = kbeg / d.K0, q1 = (kend - 1) / d.K0;
    for (int q = q0 + tid; q <= q1; q += NT) {
      const int* e = d.gk_bl + 4 * (ld.gs + q);
      gofs[2 * (q - q0)] = d.cA[0] * e[0] + d.cA[1] * e[1] + d.cA[2] * e[2] + d.cA[3] * e[3];
      gofs[2 * (q - q0) + 1] = d.cB[0] * e[0] + d.cB[1] * e[1] + d.cB[2] * e[2] + d.cB[3] * e[3];
    }
    ld.gq0 = q0;
    ld.gofs = gofs;
    __syncthreads();
  }

  auto stash = [&](int buf) {
    ld.settle();
#pragma unroll
    for (int r = 0; r < Loader::NEA; ++r) {
      sA[buf][0][ld.akk[r]][ld.amm[r]] = (T)ld.av[r].re;
      sA[buf][1][ld.akk[r]][ld.amm[r]] = (T)ld.av[r].im;
    }
#pragma unroll
    for (int r = 0; r < Loader::NEB; ++r) {
      sB[buf][0][ld.bkk[r]][ld.bnn[r]] = (T)ld.bv[r].re;
      sB[buf][1][ld.bkk[r]][ld.bnn[r]] = (T)ld.bv[r].im;
    }
  };

  // FP64: the complex product as three real products (Gauss),
  //   P1 = (Ar + Ai) Br,  P2 = Ar (Bi - Br),  P3 = Ai (Br + Bi),
  //   Re = P1 - P3,  Im = P1 + P2,
  // accumulated in cre, cim and c3 and combined after the K loop.  With real
  // operands P2 = -P1 bit for bit, so the imaginary part stays exactly zero.
  // FP32 keeps the four products of the plain definition.
  constexpr bool M3 = std::is_same<T, double>::value;
  acc_t cre[IB][JB], cim[IB][JB], c3[M3 ? IB : 1][M3 ? JB : 1];
#pragma unroll
  for (int i = 0; i < IB; ++i)
#pragma unroll
    for (int j = 0; j < JB; ++j) {
      cre[i][j] = acc_t{0, 0, 0, 0};
      cim[i][j] = acc_t{0, 0, 0, 0};
      if constexpr (M3) c3[i][j] = acc_t{0, 0, 0, 0};
    }

  const int nsteps = (kend - kbeg + BK - 1) / BK;
  // the wave's 16-column blocks that carry a column segment (all of them otherwise)
  const int jlive = CMB == 5 ? min(JB, d.ncs - (wn >> 4)) : JB;
  auto live = [&](int j) { return CMB != 5 || j < jlive; };
  ld.load(d, kbeg);
  stash(0);
  __syncthreads();
  // The last step also loads and stores a (fully masked) next tile: the loop
  // body then has no branch, and the buffer it overwrites is no longer read.
  for (int it = 0; it < nsteps; ++it) {
    const int cur = NBUF == 2 ? it & 1 : 0;
    ld.load(d, kbeg + (it + 1) * BK);  // in flight during the MFMAs below
#pragma unroll
    for (int kk = 0; kk < BK; kk += 4) {
      const int kr = kk + (lane >> 4), c16 = lane & 15;
      T ar[IB], ai[IB], nai[IB], br[JB], bi[JB];
#pragma unroll
      for (int i = 0; i < IB; ++i) {
        ar[i] = sA[cur][0][kr][wm + 16 * i + c16];
        ai[i] = sA[cur][1][kr][wm + 16 * i + c16];
        nai[i] = -ai[i];
      }
#pragma unroll
      for (int j = 0; j < JB; ++j) {
        br[j] = sB[cur][0][kr][wn + 16 * j + c16];
        bi[j] = sB[cur][1][kr][wn + 16 * j + c16];
      }
      if constexpr (M3) {
        T sa[IB], db[JB], sb[JB];
#pragma unroll
        for (int i = 0; i < IB; ++i) sa[i] = ar[i] + ai[i];
#pragma unroll
        for (int j = 0; j < JB; ++j) {
          db[j] = bi[j] - br[j];
          sb[j] = br[j] + bi[j];
        }
#pragma unroll
        for (int i = 0; i < IB; ++i)
#pragma unroll
          for (int j = 0; j < JB; ++j)
            if (live(j)) cre[i][j] = Frag<T>::mfma(sa[i], br[j], cre[i][j]);
#pragma unroll
        for (int i = 0; i < IB; ++i)
#pragma unroll
          for (int j = 0; j < JB; ++j)
            if (live(j)) cim[i][j] = Frag<T>::mfma(ar[i], db[j], cim[i][j]);
#pragma unroll
        for (int i = 0; i < IB; ++i)
#pragma unroll
          for (int j = 0; j < JB; ++j)
            if (live(j)) c3[i][j] = Frag<T>::mfma(ai[i], sb[j], c3[i][j]);
      } else {
        // four independent MFMAs between two that update the same accumulator
#pragma unroll
        for (int i = 0; i < IB; ++i)
#pragma unroll
          for (int j = 0; j < JB; ++j)
            if (live(j)) cre[i][j] = Frag<T>::mfma(ar[i], br[j], cre[i][j]);
#pragma unroll
        for (int i = 0; i < IB; ++i)
#pragma unroll
          for (int j = 0; j < JB; ++j)
            if (live(j)) cim[i][j] = Frag<T>::mfma(ar[i], bi[j], cim[i][j]);
#pragma unroll
        for (int i = 0; i < IB; ++i)
#pragma unroll
          for (int j = 0; j < JB; ++j)
            if (live(j)) cre[i][j] = Frag<T>::mfma(nai[i], bi[j], cre[i][j]);
#pragma unroll
        for (int i = 0; i < IB; ++i)
#pragma unroll
          for (int j = 0; j < JB; ++j)
            if (live(j)) cim[i][j] = Frag<T>::mfma(ai[i], br[j], cim[i][j]);
      }
    }
    if (NBUF == 1) __syncthreads();  // every wave is done with the buffer
    stash(NBUF == 2 ? cur ^ 1 : 0);
    __syncthreads();
  }
  if constexpr (M3) {
#pragma unroll
    for (int i = 0; i < IB; ++i)
#pragma unroll
      for (int j = 0; j < JB; ++j) {
        const acc_t p1 = cre[i][j];
        cre[i][j] = p1 - c3[i][j];
        cim[i][j] = p1 + cim[i][j];
      }
  }

  if (CMB == 5) {
    // column segments: the wave's 16-column blocks are segments wn/16 + j
    const int I = d.bl[4 * b], J = d.bl[4 * b + 1], K = d.bl[4 * b + 2], n = d.bl[4 * b + 3];
#pragma unroll
    for (int j = 0; j < JB; ++j) {
      const int sg = (wn >> 4) + j;
      if (sg >= d.ncs) continue;
      const GemmDesc::ColSeg& g = d.cs[sg];
      const int c = lane & 15;
      const bool tail = c == 15 && g.tB != nullptr;
      if (c >= g.n && !tail) continue;
      cplx* Cs;
      int64_t base, sCm, sCn;
      double alr, ali;
      if (tail) {
        Cs = g.tC;
        base = g.tcC[0] * I + g.tcC[1] * J + g.tcC[2] * K + g.tcC[3] * n;
        sCm = g.tsCm;
        sCn = 0;
        alr = g.talpha.re;
        ali = g.talpha.im;
      } else {
        Cs = g.C;
        base = g.cC[0] * I + g.cC[1] * J + g.cC[2] * K + g.cC[3] * n;
        sCm = g.sCm;
        sCn = g.sCn;
        alr = g.alpha.re;
        ali = g.alpha.im;
      }
#pragma unroll
      for (int i = 0; i < IB; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = tm * BM + wm + 16 * i + Frag<T>::row(lane, r);
          if (row >= d.M) continue;
          const double xr = (double)cre[i][j][r], xi = (double)cim[i][j][r];
          atomic_add_cplx(Cs + base + row * sCm + c * sCn, alr * xr - ali * xi, alr * xi + ali * xr);
        }
    }
    return;
  }
  int64_t co[JB], ro[IB][4];
#pragma unroll
  for (int j = 0; j < JB; ++j) co[j] = c_off(tn * BN + wn + 16 * j + (lane & 15), d.N, d.N0, d.sCn1, d.sCn0);
#pragma unroll
  for (int i = 0; i < IB; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r)
      ro[i][r] = c_off(tm * BM + wm + 16 * i + Frag<T>::row(lane, r), d.M, d.M0, d.sCm1, d.sCm0);
#pragma unroll
  for (int i = 0; i < IB; ++i)
#pragma unroll
    for (int j = 0; j < JB; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) put<ATOMIC>(d, C, ro[i][r], co[j], (double)cre[i][j][r], (double)cim[i][j][r]);
}

// Workgroups are dispatched to the eight XCDs in turn (consecutive linear ids
// land on different XCDs, each with an L2 of its own).  xcd_contiguous() maps
// a workgroup's linear id p < total to a logical id such that each XCD takes
// a contiguous range of logical ids (XCD x gets the x-th eighth): work items
// that share operands then run on one XCD and can share its L2.  A bijection
// of [0, total).
__device__ __forceinline__ int64_t xcd_contiguous(int64_t p, int64_t total) {
  constexpr int NXCD = 8;
  const int64_t q = total / NXCD, r = total % NXCD;
  const int64_t x = p % NXCD, slot = p / NXCD;
  return (x < r ? x * (q + 1) : r * (q + 1) + (x - r) * q) + slot;
}

// Logical id lg < T * nent (T column tiles per batch entry, nent entries) to
// (tile, entry): entry-major, or with grp > 1 group-major over groups of grp
// consecutive entries, tile by tile within a group (the last group may be
// short).  A bijection.
__device__ __forceinline__ void tile_entry(int64_t lg, int64_t T, int64_t nent, int grp, int& tile, int64_t& entry) {
  if (grp > 1) {
    const int64_t g0 = lg / ((int64_t)grp * T) * grp;  // the group's first entry
    const int64_t gl = min((int64_t)grp, nent - g0);
    const int64_t r = lg - g0 * T;
    tile = (int)(r / gl);
    entry = g0 + r % gl;
  } else {
    tile = (int)(lg % T);
    entry = lg / T;
  }
}

// Split bf16 operands: x = s_0 + s_1 + ... + s_{NSL-1} + O(2^-8NSL |x|) with
// each s_p the bf16 rounding of what the earlier slices leave (every
// remainder is exact in FP32).
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
template <int NSL>
__device__ __forceinline__ void bf16_slices8(const double* v, bf16x8* s) {
  float x[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) x[e] = (float)v[e];
#pragma unroll
  for (int p = 0; p < NSL; ++p)
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const __bf16 h = (__bf16)x[e];
      s[p][e] = h;
      x[e] -= (float)h;
    }
}

// Operand rows of the split kernel: thread t owns row t % R of its tile and
// the eight consecutive k of chunk (t / R) % 4 (R = 64 rows, or 16 for a
// narrow B tile, where only the first 64 threads load).  m- or n-fast
// operands are then read by a wave as 64 consecutive rows per instruction.
template <int R, bool SEG, bool ISA>
struct SplitRows {
  int row, chunk;
  bool act, val;
  int64_t roff;  // offset of the row (not SEG)
  const cplx* P;  // entry base (not SEG)
  const cplx* Ps[4];
  __device__ __forceinline__ void init(const GemmDesc& d, int tid, int base, int ext, const cplx* p,
                                       const cplx* const* ps) {
    row = tid % R;
    chunk = (tid / R) % 4;
    act = tid < 4 * R;
    const int x = base + row;
    val = act && x < ext;
    const int64_t s1 = ISA ? d.sAm1 : d.sBn1, s0 = ISA ? d.sAm0 : d.sBn0;
    const int X0 = ISA ? d.M0 : d.N0;
    roff = SEG ? 0 : (val ? (int64_t)(x / X0) * s1 + (int64_t)(x % X0) * s0 : 0);
    P = p;
#pragma unroll
    for (int s = 0; s < 4; ++s) Ps[s] = ps[s];
  }
  // Loads the eight elements k0 + 8*chunk + e (re and im parts).
  __device__ __forceinline__ void load(const GemmDesc& d, int k0, int kend, int sk1, int sk2, int sk3, float invK0,
                                       int xabs, double* re, double* im) const {
    const int kb = k0 + 8 * chunk;
    if (SEG) {
      // segments start at multiples of 16, so a chunk of eight k lies in one
      const int s = (int)(kb >= sk1) + (int)(kb >= sk2) + (int)(kb >= sk3);
      const int r0 = kb - (s == 0 ? 0 : s == 1 ? sk1 : s == 2 ? sk2 : sk3);
      auto sel = [s](auto x0, auto x1, auto x2, auto x3) { return s == 0 ? x0 : s == 1 ? x1 : s == 2 ? x2 : x3; };
      const GemmDesc::Seg &g0 = d.seg[0], &g1 = d.seg[1], &g2 = d.seg[2], &g3 = d.seg[3];
      const cplx* p = sel(Ps[0], Ps[1], Ps[2], Ps[3]);
      const int len = sel(g0.len, g1.len, g2.len, g3.len);
      const int sx = (int)(ISA ? sel(g0.sAm, g1.sAm, g2.sAm, g3.sAm) : sel(g0.sBn, g1.sBn, g2.sBn, g3.sBn));
      const int sk = (int)(ISA ? sel(g0.sAk, g1.sAk, g2.sAk, g3.sAk) : sel(g0.sBk, g1.sBk, g2.sBk, g3.sBk));
      const int xo = xabs * sx;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int r = r0 + e;
        const bool ok = val && kb + e < kend && r < len;
        int64_t o = ok ? (int64_t)(xo + r * sk) : 0;
        asm volatile("" : "+v"(o));
        const cplx v = p[o];
        re[e] = ok ? v.re : 0.0;
        im[e] = ok ? v.im : 0.0;
      }
      return;
    }
    const int64_t k1 = ISA ? d.sAk1 : d.sBk1, k0s = ISA ? d.sAk0 : d.sBk0;
    int q, r;
    split_k(kb, d.K0, invK0, q, r);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const bool ok = val && kb + e < kend;
      int64_t o = ok ? roff + (int64_t)q * k1 + (int64_t)r * k0s : 0;
      asm volatile("" : "+v"(o));
      const cplx v = P[o];
      re[e] = ok ? v.re : 0.0;
      im[e] = ok ? v.im : 0.0;
      // next k
      ++r;
      q = r == d.K0 ? q + 1 : q;
      r = r == d.K0 ? 0 : r;
    }
  }
};

// The same tile product on the bf16 matrix cores (16x16x32 MFMA, FP32
// accumulate) with each real operand split into NSL bf16 slices; the real
// products keep the slice pairs (p, q) with p + q < NSL (3 pairs for two
// slices, 6 for three), dropping terms of relative size 2^-8NSL.  The real
// part accumulates Re*Re and Im*Im separately and subtracts at the end.
// MFMA 16x16x32 bf16 operand layout: lane l holds A[l%16][8*(l/16) + 0..7] and
// B[8*(l/16) + 0..7][l%16]; the result layout is that of the FP32 MFMAs.
// LDS holds each slice as [row][k] (A rows m, B rows n) in rows of 32 bf16 =
// four 16-byte chunks, chunk index xor (row/4)%4, so that the 16 rows of one
// fragment read cover all banks once.  One buffer and two barriers per K
// step; several workgroups per CU overlap one's loads with another's MFMAs.
template <bool ATOMIC, bool KFA, bool NFB, int BN, bool SEG, int NSL>
__global__ __launch_bounds__(NT) void zgemm_split_kernel(GemmDesc d, int ksplit, int kchunk) {
  constexpr int BK = 32;
  constexpr int WM = BN == 64 ? 32 : 16, WN = BN == 64 ? 32 : 16;
  constexpr int IB = WM / 16, JB = WN / 16;
  __shared__ __attribute__((aligned(16))) bf16x8 sA[2][NSL][BM][BK / 8];  // [re, im][slice][m][k chunk]
  __shared__ __attribute__((aligned(16))) bf16x8 sB[2][NSL][BN][BK / 8];  // [re, im][slice][n][k chunk]

  const int tilesN = (d.N + BN - 1) / BN;
  int bx = blockIdx.x;
  int64_t b = (int64_t)blockIdx.y + (int64_t)blockIdx.z * gridDim.y;
  if (d.grp > 1 && ksplit == 1) {  // grouped entries, each XCD a contiguous range
    const int64_t nent = (int64_t)gridDim.y * gridDim.z;
    tile_entry(xcd_contiguous((int64_t)blockIdx.x + (int64_t)gridDim.x * b, (int64_t)gridDim.x * nent), gridDim.x,
               nent, d.grp, bx, b);
  }
  const int kz = bx % ksplit;
  const int tile = bx / ksplit;
  const int tm = tile / tilesN, tn = tile % tilesN;
  if (b >= d.batch) return;
  const int kbeg = kz * kchunk;
  const int kend = min(d.K, kbeg + kchunk);
  if (kbeg >= kend) return;

  // entry bases
  const cplx* A = nullptr;
  const cplx* B = nullptr;
  const cplx* Ap[4] = {nullptr, nullptr, nullptr, nullptr};
  const cplx* Bp[4] = {nullptr, nullptr, nullptr, nullptr};
  cplx* C;
  if (d.bl) {
    const int I = d.bl[4 * b], J = d.bl[4 * b + 1], K = d.bl[4 * b + 2], n = d.bl[4 * b + 3];
    C = d.C + d.cC[0] * I + d.cC[1] * J + d.cC[2] * K + d.cC[3] * n;
    if (SEG) {
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const GemmDesc::Seg& g = d.seg[s < d.nseg ? s : 0];
        Ap[s] = g.A + g.cA[0] * I + g.cA[1] * J + g.cA[2] * K + g.cA[3] * n;
        Bp[s] = g.B + g.cB[0] * I + g.cB[1] * J + g.cB[2] * K + g.cB[3] * n;
      }
    } else {
      A = d.A + d.cA[0] * I + d.cA[1] * J + d.cA[2] * K + d.cA[3] * n;
      B = d.B + d.cB[0] * I + d.cB[1] * J + d.cB[2] * K + d.cB[3] * n;
    }
  } else {
    A = d.A + b * d.sAb;
    B = d.B + b * d.sBb;
    C = d.C + b * d.sCb;
  }
  const int sk1 = d.nseg > 1 ? d.seg[1].k0 : 0x7fffffff;
  const int sk2 = d.nseg > 2 ? d.seg[2].k0 : 0x7fffffff;
  const int sk3 = d.nseg > 3 ? d.seg[3].k0 : 0x7fffffff;
  const float invK0 = 1.0f / (float)d.K0;

  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int wm = (wave / (BN / WN)) * WM, wn = (wave % (BN / WN)) * WN;
  SplitRows<BM, SEG, true> ra;
  SplitRows<BN, SEG, false> rb;
  ra.init(d, tid, tm * BM, d.M, A, Ap);
  rb.init(d, tid, tn * BN, d.N, B, Bp);
  auto cswz = [](int row, int c) { return (c ^ (row >> 2)) & 3; };

  f4 crr[IB][JB], cii[IB][JB], cim[IB][JB];
#pragma unroll
  for (int i = 0; i < IB; ++i)
#pragma unroll
    for (int j = 0; j < JB; ++j) {
      crr[i][j] = f4{0, 0, 0, 0};
      cii[i][j] = f4{0, 0, 0, 0};
      cim[i][j] = f4{0, 0, 0, 0};
    }

  const int nsteps = (kend - kbeg + BK - 1) / BK;
  const int c16 = lane & 15, kc = lane >> 4;
  for (int it = 0; it < nsteps; ++it) {
    const int k0 = kbeg + it * BK;
    double xr[8], xi[8];
    bf16x8 sr[NSL], si[NSL];
    ra.load(d, k0, kend, sk1, sk2, sk3, invK0, tm * BM + ra.row, xr, xi);
    bf16_slices8<NSL>(xr, sr);
    bf16_slices8<NSL>(xi, si);
    double yr[8], yi[8];
    bf16x8 tr[NSL], ti[NSL];
    if (rb.act) {
      rb.load(d, k0, kend, sk1, sk2, sk3, invK0, tn * BN + rb.row, yr, yi);
      bf16_slices8<NSL>(yr, tr);
      bf16_slices8<NSL>(yi, ti);
    }
    __syncthreads();  // the previous step's fragment reads are done
#pragma unroll
    for (int p = 0; p < NSL; ++p) {
      sA[0][p][ra.row][cswz(ra.row, ra.chunk)] = sr[p];
      sA[1][p][ra.row][cswz(ra.row, ra.chunk)] = si[p];
    }
    if (rb.act) {
#pragma unroll
      for (int p = 0; p < NSL; ++p) {
        sB[0][p][rb.row][cswz(rb.row, rb.chunk)] = tr[p];
        sB[1][p][rb.row][cswz(rb.row, rb.chunk)] = ti[p];
      }
    }
    __syncthreads();
#pragma unroll
    for (int p = 0; p < NSL; ++p) {
      bf16x8 ar[IB], ai[IB];
#pragma unroll
      for (int i = 0; i < IB; ++i) {
        const int row = wm + 16 * i + c16;
        ar[i] = sA[0][p][row][cswz(row, kc)];
        ai[i] = sA[1][p][row][cswz(row, kc)];
      }
#pragma unroll
      for (int q = 0; q + p < NSL; ++q) {
        bf16x8 br[JB], bi[JB];
#pragma unroll
        for (int j = 0; j < JB; ++j) {
          const int row = wn + 16 * j + c16;
          br[j] = sB[0][q][row][cswz(row, kc)];
          bi[j] = sB[1][q][row][cswz(row, kc)];
        }
#pragma unroll
        for (int i = 0; i < IB; ++i)
#pragma unroll
          for (int j = 0; j < JB; ++j) {
            crr[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ar[i], br[j], crr[i][j], 0, 0, 0);
            cim[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ar[i], bi[j], cim[i][j], 0, 0, 0);
            cii[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ai[i], bi[j], cii[i][j], 0, 0, 0);
            cim[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ai[i], br[j], cim[i][j], 0, 0, 0);
          }
      }
    }
  }

  int64_t co[JB], ro[IB][4];
#pragma unroll
  for (int j = 0; j < JB; ++j) co[j] = c_off(tn * BN + wn + 16 * j + (lane & 15), d.N, d.N0, d.sCn1, d.sCn0);
#pragma unroll
  for (int i = 0; i < IB; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r)
      ro[i][r] = c_off(tm * BM + wm + 16 * i + Frag<float>::row(lane, r), d.M, d.M0, d.sCm1, d.sCm0);
#pragma unroll
  for (int i = 0; i < IB; ++i)
#pragma unroll
    for (int j = 0; j < JB; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        put<ATOMIC>(d, C, ro[i][r], co[j], (double)crr[i][j][r] - (double)cii[i][j][r], (double)cim[i][j][r]);
}

// Y = alpha X (+ Y) over up to 8 index runs; INT the type indexes are formed in.
template <typename INT>
__device__ __forceinline__ void axpy_range(const AxpyDesc& d, int64_t first, int64_t step, int64_t total) {
  for (int64_t e = first; e < total; e += step) {
    INT r = (INT)e;
    int64_t ox = 0, oy = 0;
    for (int k = d.nd - 1; k > 0; --k) {
      const INT h = r / (INT)d.shape[k], q = r - h * (INT)d.shape[k];
      r = h;
      ox += q * d.sx[k];
      oy += q * d.sy[k];
    }
    ox += r * d.sx[0];
    oy += r * d.sy[0];
    const cplx x = d.X[ox];
    cplx y = d.store ? cplx{0, 0} : d.Y[oy];
    y.re += d.alpha.re * x.re - d.alpha.im * x.im;
    y.im += d.alpha.re * x.im + d.alpha.im * x.re;
    d.Y[oy] = y;
  }
}
template <typename INT>
__global__ void axpy_kernel(AxpyDesc d, int64_t total) {
  axpy_range<INT>(d, (int64_t)blockIdx.x * blockDim.x + threadIdx.x, (int64_t)gridDim.x * blockDim.x, total);
}
constexpr int kAxpyGroup = 12;
struct AxpyGroup {
  AxpyDesc d[kAxpyGroup];
  uint32_t total[kAxpyGroup];
  int end[kAxpyGroup];  // workgroups up to and with axpy i
  int n;
};
static_assert(sizeof(AxpyGroup) <= 4096, "kernel arguments");
__global__ void axpy_group_kernel(AxpyGroup d) {
  int i = 0;
  while (i + 1 < d.n && (int)blockIdx.x >= d.end[i]) ++i;
  const int b0 = i > 0 ? d.end[i - 1] : 0;
  axpy_range<uint32_t>(d.d[i], (int64_t)((int)blockIdx.x - b0) * blockDim.x + threadIdx.x,
                       (int64_t)(d.end[i] - b0) * blockDim.x, d.total[i]);
}

__global__ void zero_many_kernel(ZeroList z) {
  cplx* p = z.p[blockIdx.y];
  const int64_t n = z.n[blockIdx.y];
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x)
    p[e] = cplx{0, 0};
}

__global__ void fill_kernel(cplx* p, int64_t n, cplx v) {
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x)
    p[e] = v;
}

__global__ void fill_int_kernel(int* p, int64_t n, int v) {
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x)
    p[e] = v;
}

// cand = y + alpha * a, and the first step whose candidate has a non-finite
// element into pst[PST_FLAG] (as step + 1)
__global__ void update_candidate_kernel(const cplx* __restrict__ y, const cplx* __restrict__ a, cplx alpha,
                                        cplx* __restrict__ cand, int64_t n, int* pst) {
  bool bad = false;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x) {
    const cplx x = a[e];
    cplx c = y[e];
    c.re += alpha.re * x.re - alpha.im * x.im;
    c.im += alpha.re * x.im + alpha.im * x.re;
    cand[e] = c;
    bad = bad || !isfinite(c.re) || !isfinite(c.im);
  }
  if (bad) atomicCAS(pst + PST_FLAG, 0, pst[PST_BASE] + pst[PST_STEP] + 1);
}

// y = cand unless a step has diverged
__global__ void update_apply_kernel(cplx* __restrict__ y, const cplx* __restrict__ cand, int64_t n,
                                    const int* pst) {
  if (pst[PST_FLAG] != 0) return;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x)
    y[e] = cand[e];
}

__global__ void build_h_kernel(cplx* __restrict__ h, const cplx* __restrict__ h0, const cplx* __restrict__ mu,
                               int64_t nn, const double* Edev, double ex, double ey, double ez) {
  const double E0 = Edev ? Edev[0] : ex, E1 = Edev ? Edev[1] : ey, E2 = Edev ? Edev[2] : ez;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < nn; e += (int64_t)gridDim.x * blockDim.x) {
    cplx x = h0[e];
    const cplx m0 = mu[e], m1 = mu[nn + e], m2 = mu[2 * nn + e];
    x.re -= E0 * m0.re;
    x.im -= E0 * m0.im;
    x.re -= E1 * m1.re;
    x.im -= E1 * m1.im;
    x.re -= E2 * m2.re;
    x.im -= E2 * m2.im;
    h[e] = x;
  }
}

__global__ void stage_fields_kernel(const double* __restrict__ table, const int* __restrict__ pst,
                                    double* __restrict__ estage) {
  const int t = threadIdx.x;
  if (t >= 12) return;
  const int c = pst[PST_STEP], stage = t / 3, x = t % 3;
  const int k = 2 * c + (stage == 0 ? 0 : stage == 3 ? 2 : 1);
  estage[t] = table[3 * k + x];
}

__global__ void store_dipole_kernel(cplx* __restrict__ mus, const cplx* __restrict__ m3, const int* __restrict__ pst) {
  const int t = threadIdx.x;
  if (t < 3) mus[3 * pst[PST_STEP] + t] = m3[t];
}

__global__ void step_kernel(int* pst, int reset, int base) {
  if (threadIdx.x != 0) return;
  if (reset) {
    pst[PST_STEP] = 0;
    pst[PST_BASE] = base;
  } else {
    pst[PST_STEP] += 1;
  }
}

__global__ void copy_kernel(cplx* __restrict__ dst, const cplx* __restrict__ src, int64_t n) {
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x)
    dst[e] = src[e];
}

inline unsigned grid_for(int64_t n, int bs) {
  int64_t g = (n + bs - 1) / bs;
  if (g > 65536) g = 65536;
  if (g < 1) g = 1;
  return (unsigned)g;
}

// Kernel choice: precision (FP64, FP32, bf16 split with 3 or 2 slices),
// atomic epilogue, operand layouts, tile width and K segments.
template <int MODE, bool ATOMIC, bool KFA, bool NFB, int BN, bool SEG>
void launch_one(const GemmDesc& d, dim3 grid, hipStream_t s, int ksplit, int kchunk) {
  if constexpr (MODE == RTCC3_PREC_FP64 && SEG)
    RTCC3_CHECK(false, "gemm: FP64 segmented products have a kernel of their own");
  else if (MODE == RTCC3_PREC_FP64)
    hipLaunchKernelGGL((zgemm_kernel<double, ATOMIC, KFA, NFB, BN, SEG>), grid, dim3(NT), 0, s, d, ksplit, kchunk);
  else if (MODE == RTCC3_PREC_FP32)
    hipLaunchKernelGGL((zgemm_kernel<float, ATOMIC, KFA, NFB, BN, SEG>), grid, dim3(NT), 0, s, d, ksplit, kchunk);
  else if (MODE == RTCC3_PREC_BF16X3)
    hipLaunchKernelGGL((zgemm_split_kernel<ATOMIC, KFA, NFB, BN, SEG, 3>), grid, dim3(NT), 0, s, d, ksplit, kchunk);
  else
    hipLaunchKernelGGL((zgemm_split_kernel<ATOMIC, KFA, NFB, BN, SEG, 2>), grid, dim3(NT), 0, s, d, ksplit, kchunk);
}

// Combined-operand products (A k-fast, B k-fast), FP32.
template <bool ATOMIC, int BN>
void launch_comb_gemm(const GemmDesc& d, dim3 grid, hipStream_t s, int ksplit, int kchunk) {
  typedef float T;
  if (d.comb_n == 1)
    hipLaunchKernelGGL((zgemm_kernel<T, ATOMIC, true, false, BN, false, 4>), grid, dim3(NT), 0, s, d, ksplit, kchunk);
  else if (d.comb_on == 0)
    hipLaunchKernelGGL((zgemm_kernel<T, ATOMIC, true, false, BN, false, 1>), grid, dim3(NT), 0, s, d, ksplit, kchunk);
  else
    hipLaunchKernelGGL((zgemm_kernel<T, ATOMIC, true, false, BN, false, 2>), grid, dim3(NT), 0, s, d, ksplit, kchunk);
}

// Gathered-K products, FP32, for the layouts they are used with.
template <bool ATOMIC>
void launch_gather_gemm(const GemmDesc& d, dim3 grid, hipStream_t s, int ksplit, int kchunk, bool kfa, bool nfb,
                        int bn) {
  typedef float T;
  if (kfa && nfb) {
    if (bn == 16)
      hipLaunchKernelGGL((zgemm_kernel<T, ATOMIC, true, true, 16, false, 3>), grid, dim3(NT), 0, s, d, ksplit, kchunk);
    else
      hipLaunchKernelGGL((zgemm_kernel<T, ATOMIC, true, true, 64, false, 3>), grid, dim3(NT), 0, s, d, ksplit, kchunk);
    return;
  }
  RTCC3_CHECK(!nfb, "gemm: no gathered-K kernel for this operand layout");
  if (kfa) {
    if (bn == 16)
      hipLaunchKernelGGL((zgemm_kernel<T, ATOMIC, true, false, 16, false, 3>), grid, dim3(NT), 0, s, d, ksplit, kchunk);
    else
      hipLaunchKernelGGL((zgemm_kernel<T, ATOMIC, true, false, 64, false, 3>), grid, dim3(NT), 0, s, d, ksplit, kchunk);
  } else {
    if (bn == 16)
      hipLaunchKernelGGL((zgemm_kernel<T, ATOMIC, false, false, 16, false, 3>), grid, dim3(NT), 0, s, d, ksplit, kchunk);
    else
      hipLaunchKernelGGL((zgemm_kernel<T, ATOMIC, false, false, 64, false, 3>), grid, dim3(NT), 0, s, d, ksplit, kchunk);
  }
}

template <int MODE, bool ATOMIC>
void launch_layout(const GemmDesc& d, dim3 grid, hipStream_t s, int ksplit, int kchunk, bool kfa, bool nfb, int bn) {
  if (d.ncs > 0) {
    if constexpr (ATOMIC && MODE == RTCC3_PREC_FP32) {
      hipLaunchKernelGGL((zgemm_kernel<float, true, true, false, 64, false, 5>), grid, dim3(NT), 0, s, d, ksplit, kchunk);
    } else {
      RTCC3_CHECK(false, "gemm: column segments run in FP32 with atomics");
    }
    return;
  }
  if (d.gk_start) {
    if constexpr (MODE == RTCC3_PREC_FP32)
      launch_gather_gemm<ATOMIC>(d, grid, s, ksplit, kchunk, kfa, nfb, bn);
    else
      RTCC3_CHECK(false, "gemm: gathered products run in FP32");
  } else if (d.comb_n > 0) {
    if constexpr (MODE == RTCC3_PREC_FP32) {
      if (bn == 16)
        launch_comb_gemm<ATOMIC, 16>(d, grid, s, ksplit, kchunk);
      else
        launch_comb_gemm<ATOMIC, 64>(d, grid, s, ksplit, kchunk);
    } else {
      RTCC3_CHECK(false, "gemm: combined operands run in FP32");
    }
  } else if (d.nseg > 0)
    launch_one<MODE, ATOMIC, true, true, 64, true>(d, grid, s, ksplit, kchunk);
  else if (bn == 16) {
    if (kfa && nfb)
      launch_one<MODE, ATOMIC, true, true, 16, false>(d, grid, s, ksplit, kchunk);
    else if (kfa)
      launch_one<MODE, ATOMIC, true, false, 16, false>(d, grid, s, ksplit, kchunk);
    else if (nfb)
      launch_one<MODE, ATOMIC, false, true, 16, false>(d, grid, s, ksplit, kchunk);
    else
      launch_one<MODE, ATOMIC, false, false, 16, false>(d, grid, s, ksplit, kchunk);
  } else {
    if (kfa && nfb)
      launch_one<MODE, ATOMIC, true, true, 64, false>(d, grid, s, ksplit, kchunk);
    else if (kfa)
      launch_one<MODE, ATOMIC, true, false, 64, false>(d, grid, s, ksplit, kchunk);
    else if (nfb)
      launch_one<MODE, ATOMIC, false, true, 64, false>(d, grid, s, ksplit, kchunk);
    else
      launch_one<MODE, ATOMIC, false, false, 64, false>(d, grid, s, ksplit, kchunk);
  }
}

template <int MODE>
void launch_mode(const GemmDesc& d, dim3 grid, hipStream_t s, int ksplit, int kchunk, bool atomic, bool kfa, bool nfb,
                 int bn) {
  if (atomic)
    launch_layout<MODE, true>(d, grid, s, ksplit, kchunk, kfa, nfb, bn);
  else
    launch_layout<MODE, false>(d, grid, s, ksplit, kchunk, kfa, nfb, bn);
}

// The same product with the roles of A and B exchanged: C^T = B^T A^T.
GemmDesc transposed(const GemmDesc& d) {
  GemmDesc t = d;
  t.M = d.N;
  t.N = d.M;
  t.M0 = d.N0;
  t.N0 = d.M0;
  t.A = d.B;
  t.sAm1 = d.sBn1;
  t.sAm0 = d.sBn0;
  t.sAk1 = d.sBk1;
  t.sAk0 = d.sBk0;
  t.sAb = d.sBb;
  t.B = d.A;
  t.sBk1 = d.sAk1;
  t.sBk0 = d.sAk0;
  t.sBn1 = d.sAm1;
  t.sBn0 = d.sAm0;
  t.sBb = d.sAb;
  t.sCm1 = d.sCn1;
  t.sCm0 = d.sCn0;
  t.sCn1 = d.sCm1;
  t.sCn0 = d.sCm0;
  t.comb_on = 1 - d.comb_on;
  std::copy(d.cB, d.cB + 4, t.cA);
  std::copy(d.cA, d.cA + 4, t.cB);
  return t;
}

}  // namespace

struct Tuner {
  std::unordered_map<uint64_t, int> best;  // descriptor key -> K split
  std::unordered_map<uint64_t, int> heur;  // the heuristic's split for the same products
  std::unordered_map<uint64_t, TuneRecord> rec;
  std::unordered_map<uint64_t, float> gain;  // ms that the split saves against none
  bool tuning = false;
  hipEvent_t e0 = nullptr, e1 = nullptr;
};

namespace {
thread_local Tuner* g_tuner = nullptr;

// FNV-1a over the fields that define a product's work and layout (not its pointers, nor
// what runs beside it).
struct KeyHash {
  uint64_t h = 1469598103934665603ull;
  void add(int64_t x) {
    for (int i = 0; i < 8; ++i) {
      h ^= (uint64_t)((x >> (8 * i)) & 0xff);
      h *= 1099511628211ull;
    }
  }
};
uint64_t desc_key(const GemmDesc& d) {
  KeyHash k;
  for (int64_t x : {(int64_t)d.M, (int64_t)d.N, (int64_t)d.K, (int64_t)d.batch, (int64_t)d.M0, (int64_t)d.N0,
                    (int64_t)d.K0, d.sAm1, d.sAm0, d.sAk1, d.sAk0, d.sAb, d.sBk1, d.sBk0, d.sBn1, d.sBn0, d.sBb,
                    d.sCm1, d.sCm0, d.sCn1, d.sCn0, d.sCb, (int64_t)d.atomic, (int64_t)d.prec, (int64_t)d.store,
                    (int64_t)d.fresh, (int64_t)d.nseg, (int64_t)d.ncs, (int64_t)d.comb_n, (int64_t)d.comb_on,
                    (int64_t)(d.gk_start != nullptr), (int64_t)(d.bl != nullptr), (int64_t)d.force_prec})
    k.add(x);
  for (int i = 0; i < d.ncs; ++i) {
    k.add(d.cs[i].n);
    k.add(d.cs[i].sBk);
    k.add(d.cs[i].sBn);
    k.add(d.cs[i].tB != nullptr);
  }
  return k.h;
}
}  // namespace

Tuner* tuner_new() {
  Tuner* t = new Tuner();
  if (hipEventCreate(&t->e0) != hipSuccess || hipEventCreate(&t->e1) != hipSuccess) {
    tuner_delete(t);
    throw Error(-3, "tuner: event creation failed");
  }
  return t;
}
void tuner_delete(Tuner* t) {
  if (!t) return;
  if (t->e0) (void)hipEventDestroy(t->e0);
  if (t->e1) (void)hipEventDestroy(t->e1);
  delete t;
}
void tuner_set_tuning(Tuner* t, bool on) { t->tuning = on; }
bool tuning_now() { return g_tuner && g_tuner->tuning; }
void tuner_clear(Tuner* t) {
  t->best.clear();
  t->heur.clear();
  t->gain.clear();
}
int tuner_records(const Tuner* t, TuneRecord* out, int cap) {
  int n = 0;
  for (auto& kv : t->rec) {
    if (n < cap && out) out[n] = kv.second;
    ++n;
  }
  return n;
}
void tuner_counts(const Tuner* t, int& sites, int& changed) {
  sites = (int)t->best.size();
  changed = 0;
  for (auto& kv : t->best) {
    auto it = t->heur.find(kv.first);
    if (it != t->heur.end() && it->second != kv.second) ++changed;
  }
}
TunerScope::TunerScope(Tuner* t) : prev(g_tuner) { g_tuner = t; }
TunerScope::~TunerScope() { g_tuner = prev; }

int gemm(const GemmDesc& d_in, hipStream_t s) {
  // A bf16-split run takes the split kernel for its segmented products only;
  // its other products that come here run in FP32.
  GemmDesc dsel = d_in;
  if ((dsel.prec == RTCC3_PREC_BF16X3 || dsel.prec == RTCC3_PREC_BF16X2) &&
      !((dsel.nseg > 0 || dsel.force_prec) && !dsel.comb_n && !dsel.gk_start && !dsel.ncs))
    dsel.prec = RTCC3_PREC_FP32;
  const GemmDesc& d0 = dsel;
  if (d0.M <= 0 || d0.N <= 0 || d0.batch <= 0) return 0;
  if (d0.K <= 0) return 0;
  RTCC3_CHECK(d0.M0 >= 1 && d0.N0 >= 1 && d0.K0 >= 1, "gemm: inner extents must be >= 1");
  if (d0.comb_n > 0) {
    RTCC3_CHECK((d0.comb_n == 3 || (d0.comb_n == 1 && d0.comb_on == 1)) && d0.bl && d0.part && d0.nseg == 0 &&
                    (d0.comb_on == 0 || d0.comb_on == 1),
                "gemm: bad combined operand");
  }
  if (d0.ncs > 0) {
    RTCC3_CHECK(d0.ncs <= 4 && d0.bl && d0.nseg == 0 && d0.comb_n == 0 && !d0.gk_start && !d0.store &&
                    d0.atomic && d0.M0 == d0.M && d0.sAk0 == 1,
                "gemm: bad column segments");
    for (int s = 0; s < d0.ncs; ++s) {
      const GemmDesc::ColSeg& g = d0.cs[s];
      RTCC3_CHECK(g.n >= 1 && g.n <= 16 && g.B && g.C && g.sBk >= 0 && g.sBn >= 0 && g.sCm >= 0 && g.sCn >= 0 &&
                      (int64_t)d0.K * g.sBk < (1LL << 31),
                  "gemm: bad column segment");
      RTCC3_CHECK(!g.tB || (g.n <= 15 && g.tC && g.tsBk >= 0 && g.tsCm >= 0 && (int64_t)d0.K * g.tsBk < (1LL << 31)),
                  "gemm: bad tail column");
    }
  }
  if (d0.gk_start) {
    RTCC3_CHECK(d0.gk_bl && d0.bl && d0.nseg == 0 && d0.comb_n == 0 && d0.K % d0.K0 == 0 && d0.sAk1 == 0 &&
                    d0.sBk1 == 0,
                "gemm: bad gathered K");
  }
  if (d0.nseg > 0) {
    RTCC3_CHECK(d0.nseg <= 4 && d0.bl && d0.seg[0].k0 == 0 && d0.M0 == d0.M, "gemm: bad K segments");
    for (int s = 0; s < d0.nseg; ++s) {
      const GemmDesc::Seg& g = d0.seg[s];
      const int end = s + 1 < d0.nseg ? d0.seg[s + 1].k0 : d0.K;
      RTCC3_CHECK(g.A && g.B && g.len >= 1 && g.k0 % 16 == 0 && g.k0 + g.len <= end, "gemm: bad K segments");
      // element offsets inside a segment operand are formed in 32 bits
      RTCC3_CHECK((int64_t)(d0.M + 63) * g.sAm + (int64_t)g.len * g.sAk < (1LL << 31) &&
                      (int64_t)g.len * g.sBk + (int64_t)(d0.N + 63) * g.sBn < (1LL << 31),
                  "gemm: segment operand too large");
    }
  }
  RTCC3_CHECK(d0.K < (1 << 22) && d0.M < (1 << 22) && d0.N < (1 << 22), "gemm: extent too long");
  RTCC3_CHECK(!(d0.store || d0.fresh) || !d0.shared, "gemm: an output written over has one product");
  RTCC3_CHECK(!d0.store || !d0.atomic, "gemm: store mode cannot be atomic");
  // A narrow side (at most 16, e.g. one occupied index) goes on N with 64x16
  // tiles; a narrow M is moved there by transposing the product.
  const bool tr = d0.M <= 16 && d0.N > 16 && d0.nseg == 0 && !d0.gk_start && d0.ncs == 0;
  GemmDesc d = tr ? transposed(d0) : d0;
  if (d.ncs > 0) d.N = d.N0 = 64;  // one 64-wide tile of four 16-column segments
  // The segmented kernel has 64-wide tiles.  A gathered product up to 32 wide
  // (an occupied index of 17 to 32) takes two 16-wide tiles rather than one
  // 64-wide tile that would be mostly padding.
  const int bn = (d.N <= 16 || (d.gk_start && d.N <= 32)) && d.nseg == 0 ? 16 : 64;
  const int64_t tiles = (int64_t)((d.M + BM - 1) / BM) * ((d.N + bn - 1) / bn);
  // Split K across workgroups when the grid is too small to fill the chip and
  // K is long; the partial products are then added with atomics.
  int ksplit = 1;
  const int64_t wgs = tiles * d.batch;
  constexpr int BKMAX = 32;  // K chunks are multiples of every kernel's K step
  // A gathered product has few entries with long K: aim at a fuller chip.  A
  // plain product with a handful of tiles splits K down to chunks of 64 for
  // about 512 workgroups; one that already has half a workgroup per CU splits
  // only into chunks of at least 512 (short chunks cost more in atomics and
  // loop overhead than the extra workgroups gain).
  int64_t kmin = 1;  // the accumulation limits below
  if (!d.store && d.K >= 4 * BKMAX) {
    int64_t want = 1, maxs = 1;
    if (d.gk_start) {
      if (wgs < 2048) want = (2048 + wgs - 1) / wgs, maxs = d.K / (2 * BKMAX);
    } else if (wgs < 128) {
      want = (512 + wgs - 1) / wgs, maxs = d.K / (2 * BKMAX);
    } else if (wgs < 512) {
      want = (1024 + wgs - 1) / wgs, maxs = d.K / 512;
    }
    ksplit = (int)std::max<int64_t>(1, std::min<int64_t>(want, maxs));
  }
  if (d.prec != RTCC3_PREC_FP64 && !d.store && !d.gk_start) {
    // FP32 accumulation: no workgroup sums more than 4096 terms (partial sums
    // are added in FP64)
    kmin = std::max<int64_t>(kmin, (d.K + 4095) / 4096);
    ksplit = (int)std::max<int64_t>(ksplit, kmin);
  }
  if (d.gk_start) {  // a workgroup's FP32 sum spans at most 16 gathered blocks
    const int64_t span_k = std::max<int64_t>(BKMAX, 16 * (int64_t)d.K0 / BKMAX * BKMAX);
    kmin = std::max<int64_t>(kmin, (d.K + span_k - 1) / span_k);
    ksplit = (int)std::max<int64_t>(ksplit, kmin);
  }
  const bool kfa = d.sAk0 == 1, nfb = d.sBn0 == 1;
  RTCC3_CHECK(!d.comb_n || (kfa && !nfb), "gemm: a combined operand needs A and B read k-fast");
  // The bf16 split pays off only where the matrix cores bound the product (the
  // long segmented builds); the other products of a split-precision run use
  // FP32, which is at least as accurate.
  const bool split = d.prec == RTCC3_PREC_BF16X3 || d.prec == RTCC3_PREC_BF16X2;
  const int prec = split && ((d.nseg == 0 && !d.force_prec) || d.comb_n || d.gk_start || d.ncs) ? RTCC3_PREC_FP32 : d.prec;
  // Plain FP64 products go to the fragment kernel wherever its 32-bit offsets
  // reach (o=15, v=57: 110 products of a right-hand side 8.2 ms through LDS tiles,
  // 6.1 from fragments; o=5, v=18: 2.0 and 0.6).
  const bool frag = prec == RTCC3_PREC_FP64 && frag_gemm_fits(d);
  if (frag) ksplit = frag_gemm_split(d);
  int launches = 0;
  auto launch = [&](int ks, bool trial = false) {
    ++launches;
    // In FP32 the trials add in any case: which split is the fastest by itself
    // decides, since the split is also how far the sums are formed in FP32.
    d.store = d_in.store;
    if (d.fresh && (frag || !trial)) {
      if (ks == 1 && !d.atomic)
        d.store = 1;
      else
        fill(d.fresh_p, d.fresh_n, cplx{0, 0}, s), ++launches;
    }
    if (frag) return frag_gemm(d, ks, s);
    const int kchunk = (int)((((int64_t)d.K + ks - 1) / ks + BKMAX - 1) / BKMAX * BKMAX);
    RTCC3_CHECK(tiles * ks < (1LL << 31), "gemm: too many tiles");
    RTCC3_CHECK(!d.gk_start || kchunk / d.K0 + 2 <= GK_MAXSEG, "gemm: gathered K range too long for one workgroup");
    int64_t by = d.batch, bz = 1;
    while (by > 65535) {
      by = (by + 1) / 2;
      bz *= 2;
    }
    dim3 grid((unsigned)(tiles * ks), (unsigned)by, (unsigned)bz);
    const bool atomic = d.atomic || d.shared || ks > 1;
    switch (prec) {
      case RTCC3_PREC_FP64:
        launch_mode<RTCC3_PREC_FP64>(d, grid, s, ks, kchunk, atomic, kfa, nfb, bn);
        break;
      case RTCC3_PREC_FP32:
        launch_mode<RTCC3_PREC_FP32>(d, grid, s, ks, kchunk, atomic, kfa, nfb, bn);
        break;
      case RTCC3_PREC_BF16X3:
        launch_mode<RTCC3_PREC_BF16X3>(d, grid, s, ks, kchunk, atomic, kfa, nfb, bn);
        break;
      case RTCC3_PREC_BF16X2:
        launch_mode<RTCC3_PREC_BF16X2>(d, grid, s, ks, kchunk, atomic, kfa, nfb, bn);
        break;
      default:
        RTCC3_CHECK(false, "gemm: unknown precision");
    }
    RTCC3_HIP(hipGetLastError());
  };
  Tuner* tu = g_tuner;
  const bool tunable = tu && !d.store && wgs < 1024 &&
                       d.K >= 4 * BKMAX;
  if (tunable) {
    const uint64_t key = desc_key(d);
    if (tu->tuning) {
      // candidates: the heuristic's split and powers of two from kmin up to chunks of 64
      std::vector<int> cand{ksplit};
      const int64_t kmax = std::max<int64_t>(kmin, d.K / 64);
      for (int64_t ks = kmin; ks <= kmax && ks <= 64; ks *= 2)
        if (ks != ksplit) cand.push_back((int)ks);
      // An FP32 product rounds differently with another split: twice the trials, so
      // that nearly equal ones (o=5, v=36: 112.8 and 109.3 us) are not told apart by
      // chance.
      const int reps = frag ? 2 : 4;
      const float margin = frag ? 0.97f : 0.975f;
      launch(ksplit, true);  // warm the caches
      float best_ms = 1e30f, heur_ms = 0.f, one_ms = 1e30f;
      int best = ksplit;
      for (int ks : cand) {
        float ms = 1e30f;
        for (int rep = 0; rep < reps; ++rep) {
          RTCC3_HIP(hipEventRecord(tu->e0, s));
          launch(ks, true);
          RTCC3_HIP(hipEventRecord(tu->e1, s));
          RTCC3_HIP(hipEventSynchronize(tu->e1));
          float t = 0.f;
          RTCC3_HIP(hipEventElapsedTime(&t, tu->e0, tu->e1));
          ms = std::min(ms, t);
        }
        if (ks == ksplit) heur_ms = ms;
        if (ks == 1) one_ms = ms;
        if (ms < margin * best_ms) {  // a new choice must win by more than the noise
          best_ms = ms;
          best = ks;
        }
      }
      tu->best[key] = best;
      tu->heur[key] = ksplit;
      tu->gain[key] = one_ms - best_ms;
      tu->rec[key] = TuneRecord{d.M, d.N, d.K, d.batch, ksplit, best, heur_ms, best_ms};
      ksplit = best;
    } else {
      auto it = tu->best.find(key);
      if (it != tu->best.end()) ksplit = std::max<int>(it->second, (int)kmin);
    }
  }
  launch(ksplit);
  return launches;
}

namespace {
// Index runs that are contiguous in both operands counted as one; returns the
// number of elements.
int64_t axpy_runs(const AxpyDesc& d_in, AxpyDesc& d) {
  d = d_in;
  d.nd = 0;
  int64_t total = 1;
  for (int k = 0; k < d_in.nd; ++k) {
    total *= d_in.shape[k];
    if (d_in.shape[k] == 1) continue;
    if (d.nd > 0 && d.sx[d.nd - 1] == d_in.sx[k] * d_in.shape[k] && d.sy[d.nd - 1] == d_in.sy[k] * d_in.shape[k]) {
      d.shape[d.nd - 1] *= d_in.shape[k];
      d.sx[d.nd - 1] = d_in.sx[k];
      d.sy[d.nd - 1] = d_in.sy[k];
    } else {
      d.shape[d.nd] = d_in.shape[k];
      d.sx[d.nd] = d_in.sx[k];
      d.sy[d.nd] = d_in.sy[k];
      ++d.nd;
    }
  }
  if (d.nd == 0) {
    d.nd = 1;
    d.shape[0] = 1;
    d.sx[0] = d.sy[0] = 0;
  }
  return total;
}
}  // namespace

void axpy_strided(const AxpyDesc& d_in, hipStream_t s) {
  AxpyDesc d;
  const int64_t total = axpy_runs(d_in, d);
  if (total <= 0) return;
  if (total < (1LL << 32))
    hipLaunchKernelGGL(axpy_kernel<uint32_t>, dim3(grid_for(total, 256)), dim3(256), 0, s, d, total);
  else
    hipLaunchKernelGGL(axpy_kernel<int64_t>, dim3(grid_for(total, 256)), dim3(256), 0, s, d, total);
  RTCC3_HIP(hipGetLastError());
}

void axpy_group(const AxpyDesc* a, int n, hipStream_t s) {
  AxpyGroup g;
  g.n = 0;
  auto launch = [&]() {
    if (g.n == 0) return;
    hipLaunchKernelGGL(axpy_group_kernel, dim3((unsigned)g.end[g.n - 1]), dim3(256), 0, s, g);
    RTCC3_HIP(hipGetLastError());
    g.n = 0;
  };
  for (int i = 0; i < n; ++i) {
    AxpyDesc d;
    const int64_t total = axpy_runs(a[i], d);
    if (total <= 0) continue;
    if (n == 1 || total > (1 << 20)) {
      axpy_strided(a[i], s);
      continue;
    }
    g.d[g.n] = d;
    g.total[g.n] = (uint32_t)total;
    g.end[g.n] = (g.n > 0 ? g.end[g.n - 1] : 0) + (int)grid_for(total, 256);
    if (++g.n == kAxpyGroup) launch();
  }
  launch();
}

void gemm_group(const GemmDesc* g, int n, hipStream_t s) {
  std::vector<GemmDesc> small;
  for (int i = 0; i < n; ++i) {
    const GemmDesc& d = g[i];
    bool in = n > 1 && d.prec == RTCC3_PREC_FP64 && d.M > 0 && d.N > 0 && d.K > 0 && d.batch > 0 && frag_gemm_small(d);
    if (in) {
      // the split that gemm() would take (it forms the key of the product as it runs it)
      GemmDesc x = d.M <= 16 && d.N > 16 ? transposed(d) : d;
      int ks = frag_gemm_split(x);
      if (g_tuner) {
        const uint64_t key = desc_key(x);
        auto it = g_tuner->best.find(key);
        if (it != g_tuner->best.end()) ks = it->second;
        // Products that add to one output come several to a level: one stays
        // unless its split, timed by itself, saves more than the launch of its own
        // that it then takes (10 steps at o=5, v=19: 27.5 ms with none of these
        // splits, 30.0 with all of them, 27.8 with those that save 4 us).
        if (ks > 1 && d.shared && it != g_tuner->best.end() && g_tuner->gain[key] < 0.004f) ks = 1;
      }
      in = ks == 1 && !(d.fresh && d.atomic);
    }
    if (!in) {
      gemm(d, s);
      continue;
    }
    small.push_back(d);
    if (d.fresh) small.back().store = 1;
  }
  // one by itself in the kernel of its own shape (5.3 us against 6.2)
  if (small.size() == 1) {
    gemm(small[0], s);
  } else if (!small.empty()) {
    frag_gemm_group(small.data(), (int)small.size(), s);
  }
}

void zero_many(const ZeroList& z, hipStream_t s) {
  int64_t most = 0;
  for (int k = 0; k < z.count; ++k) most = std::max(most, z.n[k]);
  if (most <= 0) return;
  const dim3 grid(grid_for(most, 256), (unsigned)z.count);
  hipLaunchKernelGGL(zero_many_kernel, grid, dim3(256), 0, s, z);
  RTCC3_HIP(hipGetLastError());
}

void fill(cplx* p, int64_t n, cplx val, hipStream_t s) {
  if (n <= 0) return;
  hipLaunchKernelGGL(fill_kernel, dim3(grid_for(n, 256)), dim3(256), 0, s, p, n, val);
  RTCC3_HIP(hipGetLastError());
}

void fill_int(int* p, int64_t n, int val, hipStream_t s) {
  if (n <= 0) return;
  hipLaunchKernelGGL(fill_int_kernel, dim3(grid_for(n, 256)), dim3(256), 0, s, p, n, val);
  RTCC3_HIP(hipGetLastError());
}

void guarded_update(cplx* y, const cplx* a, cplx alpha, cplx* cand, int64_t n, int* pst, hipStream_t s) {
  if (n <= 0) return;
  RTCC3_CHECK(cand != y && cand != a, "guarded_update: candidate buffer aliases an operand");
  hipLaunchKernelGGL(update_candidate_kernel, dim3(grid_for(n, 256)), dim3(256), 0, s, y, a, alpha, cand, n, pst);
  RTCC3_HIP(hipGetLastError());
  hipLaunchKernelGGL(update_apply_kernel, dim3(grid_for(n, 256)), dim3(256), 0, s, y, cand, n, pst);
  RTCC3_HIP(hipGetLastError());
}

void build_h(cplx* h, const cplx* h0, const cplx* mu, int64_t nn, const double* Edev, const double* Ehost,
             hipStream_t s) {
  RTCC3_CHECK(Edev || Ehost, "build_h: no field");
  const double ex = Edev ? 0.0 : Ehost[0], ey = Edev ? 0.0 : Ehost[1], ez = Edev ? 0.0 : Ehost[2];
  hipLaunchKernelGGL(build_h_kernel, dim3(grid_for(nn, 256)), dim3(256), 0, s, h, h0, mu, nn, Edev, ex, ey, ez);
  RTCC3_HIP(hipGetLastError());
}

void stage_fields(const double* table, const int* pst, double* estage, hipStream_t s) {
  hipLaunchKernelGGL(stage_fields_kernel, dim3(1), dim3(64), 0, s, table, pst, estage);
  RTCC3_HIP(hipGetLastError());
}

void store_dipole(cplx* mus, const cplx* m3, const int* pst, hipStream_t s) {
  hipLaunchKernelGGL(store_dipole_kernel, dim3(1), dim3(64), 0, s, mus, m3, pst);
  RTCC3_HIP(hipGetLastError());
}

void advance_step(int* pst, hipStream_t s) {
  hipLaunchKernelGGL(step_kernel, dim3(1), dim3(64), 0, s, pst, 0, 0);
  RTCC3_HIP(hipGetLastError());
}

void reset_step(int* pst, int base, hipStream_t s) {
  hipLaunchKernelGGL(step_kernel, dim3(1), dim3(64), 0, s, pst, 1, base);
  RTCC3_HIP(hipGetLastError());
}

void copy(cplx* dst, const cplx* src, int64_t n, hipStream_t s) {
  if (n <= 0) return;
  hipLaunchKernelGGL(copy_kernel, dim3(grid_for(n, 256)), dim3(256), 0, s, dst, src, n);
  RTCC3_HIP(hipGetLastError());
}

}  // namespace rtcc3
