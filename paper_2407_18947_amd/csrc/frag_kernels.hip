// FP64 complex products on the matrix cores with fragments loaded straight
// from memory into registers.
//
// On gfx950 an FP64 MFMA and vector-ALU instructions do not overlap, also not
// across the waves of a SIMD: 12 v_mfma_f64_16x16x4 alone run at 78 TFLOP/s,
// with 24 integer adds between them at 66, with 24 f64 adds at 60.  Staging
// tiles through LDS costs such instructions (addresses, range masks, the
// planes of the three-product form, moves between prefetch registers), so the
// kernels here have none of it in their loops: a lane loads its own fragment
// elements (16 bytes each) with buffer loads whose k offset is a scalar
// register, rows and columns outside the product read a valid row or column
// and are not stored, two register sets take turns as the step in flight, and
// per 12 MFMAs only the six sums of the three-product form are left.  Waves do
// not wait for one another; the L1 cache serves the fragments that the waves of
// a workgroup share.
#include "frag_kernels.h"

#include <algorithm>
#include <cmath>
#include <vector>

namespace rtcc3 {

namespace {

typedef double d2v __attribute__((ext_vector_type(2)));
typedef double d4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
constexpr int kRsrcWord3 = 0x00020000;

__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(const cplx* p, int64_t elements) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)p, 0, (int)(elements * (int64_t)sizeof(cplx)), kRsrcWord3);
}
// The element at byte offset voff + soff (soff uniform) of a resource.
__device__ __forceinline__ d2v frag_load(__amdgpu_buffer_rsrc_t r, int voff, int soff) {
  const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0);
  d2v x;
  __builtin_memcpy(&x, &v, sizeof(x));
  return x;
}

// IB x JB blocks of 16 x 16 as three real products each (P1 = (Ar + Ai) Br,
// P2 = Ar (Bi - Br), P3 = Ai (Br + Bi); Re = P1 - P3, Im = P1 + P2).
// MFMA 16x16x4 operands: lane l holds A[l%16][l/16] and B[l/16][l%16]; result
// register r holds D[4r + l/16][l%16].
template <int IB, int JB>
struct Acc {
  d4 p1[IB][JB], p2[IB][JB], p3[IB][JB];
  __device__ __forceinline__ void clear(int i) {
#pragma unroll
    for (int j = 0; j < JB; ++j) p1[i][j] = p2[i][j] = p3[i][j] = d4{0, 0, 0, 0};
  }
  __device__ __forceinline__ void clear() {
#pragma unroll
    for (int i = 0; i < IB; ++i) clear(i);
  }
  __device__ __forceinline__ void step(const d2v* a, const d2v* b) {
    double as[IB], bd[JB], bs[JB];
#pragma unroll
    for (int i = 0; i < IB; ++i) as[i] = a[i][0] + a[i][1];
#pragma unroll
    for (int j = 0; j < JB; ++j) {
      bd[j] = b[j][1] - b[j][0];
      bs[j] = b[j][0] + b[j][1];
    }
#pragma unroll
    for (int i = 0; i < IB; ++i)
#pragma unroll
      for (int j = 0; j < JB; ++j) p1[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(as[i], b[j][0], p1[i][j], 0, 0, 0);
#pragma unroll
    for (int i = 0; i < IB; ++i)
#pragma unroll
      for (int j = 0; j < JB; ++j) p2[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i][0], bd[j], p2[i][j], 0, 0, 0);
#pragma unroll
    for (int i = 0; i < IB; ++i)
#pragma unroll
      for (int j = 0; j < JB; ++j) p3[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i][1], bs[j], p3[i][j], 0, 0, 0);
  }
  __device__ __forceinline__ d2v value(int i, int j, int r) const {
    const double x = p1[i][j][r];
    return d2v{x - p3[i][j][r], x + p2[i][j][r]};
  }
};

// acc += sum over k < len of A[.][k] B[k][.]: lane offsets ao, bo (bytes, at
// k = l/16) into ra (one resource per row block), rb; sak, sbk bytes per k.  Two register sets alternate as
// the step in flight.  A last partial step of four reads its missing k at the
// last valid one and multiplies by a zero A.
template <int IB, int JB>
__device__ __forceinline__ void contract(Acc<IB, JB>& acc, const __amdgpu_buffer_rsrc_t* ra, const int* ao, int sak,
                                         __amdgpu_buffer_rsrc_t rb, const int* bo, int sbk, int len, int kl) {
  d2v a0[IB], b0[JB], a1[IB], b1[JB];
  int sa = 0, sb = 0;
  auto load = [&](d2v* a, d2v* b) {
#pragma unroll
    for (int i = 0; i < IB; ++i) a[i] = frag_load(ra[i], ao[i], sa);
#pragma unroll
    for (int j = 0; j < JB; ++j) b[j] = frag_load(rb, bo[j], sb);
    sa += 4 * sak;
    sb += 4 * sbk;
  };
  const int nf = len >> 2;
  int q = 0;
  if (nf > 0) load(a0, b0);
  for (; q + 2 <= nf; q += 2) {
    // the barriers keep each step's loads ahead of the other set's products
    load(a1, b1);
    __builtin_amdgcn_sched_barrier(0);
    acc.step(a0, b0);
    __builtin_amdgcn_sched_barrier(0);
    if (q + 2 < nf) load(a0, b0);
    __builtin_amdgcn_sched_barrier(0);
    acc.step(a1, b1);
    __builtin_amdgcn_sched_barrier(0);
  }
  if (q < nf) acc.step(a0, b0);
  const int rest = len & 3;
  if (rest) {
    const int back = min(kl, rest - 1) - kl;  // 0 where the lane's k is valid
#pragma unroll
    for (int i = 0; i < IB; ++i) {
      const d2v z = frag_load(ra[i], ao[i] + back * sak, sa);
      a1[i] = d2v{back == 0 ? z[0] : 0.0, back == 0 ? z[1] : 0.0};
    }
#pragma unroll
    for (int j = 0; j < JB; ++j) b1[j] = frag_load(rb, bo[j] + back * sbk, sb);
    acc.step(a1, b1);
  }
}

// x / d for 0 <= x < 2^22, d >= 1, with inv = 1.0f / d.
__device__ __forceinline__ int quot(int x, int d, float inv) {
  int q = (int)((float)x * inv);
  const int r = x - q * d;
  q = r < 0 ? q - 1 : q;
  return r >= d ? q + 1 : q;
}

// Workgroups go to the eight XCDs in turn; logical ids are dealt so that each
// XCD gets a contiguous range of them (as in kernels.hip).
__device__ __forceinline__ int xcd_contiguous(int p, int total) {
  const int q = total / 8, r = total % 8, x = p % 8, slot = p / 8;
  return (x < r ? x * (q + 1) : r * (q + 1) + (x - r) * q) + slot;
}

struct FragSeg {
  GemmDesc::Seg seg[4];
  int nseg, v, N, vp;
  cplx* C;
  int64_t vb;  // block stride of C
  const int* bl;
  const int4* rt;
  int ncol;
};

// The builds of t3 and lambda3 (o=15, v=57: t3 6.9 -> 6.3 ms, lambda3 12.3 ->
// 10.1 ms a launch, alone; 0.77 -> 0.40 ms for t3 at o=10, v=38, where an
// entry's 38 rows filled a tile of 64).  What bounds them: the matrix cores,
// then the stores (10 GB of 256-byte pieces of rows that are padded to whole
// lines, 4.1 ms alone).  A workgroup computes 64 rows by 64 columns, a wave 32 by
// 32.  The rows of all entries of a run (which share B) are numbered through,
// so only a run's last tile has rows to spare.  Workgroups run over a run's
// row tiles first, so its 64-column slice of B stays in the XCD's L2.  Three
// waves per SIMD: 96 accumulator registers and two sets of 16 for loads.
template <bool ATOMIC>
__global__ __launch_bounds__(256, 3) void frag_seg_kernel(FragSeg d) {
  constexpr int IB = 2, JB = 2;
  __shared__ int64_t ebase[kFragRun];   // first element of the entry's block in C
  __shared__ int eoff[4][kFragRun];     // byte offset of the entry's A operand from the run's first, per segment
  const int lg = xcd_contiguous((int)blockIdx.x, (int)gridDim.x);
  const int4 rt = d.rt[lg / d.ncol];
  const int rem = lg - rt.z * d.ncol;
  const int ct = rem / rt.w, tile = rem % rt.w;
  const int* e0 = d.bl + 4 * (int64_t)rt.x;
  const int I0 = e0[0], J0 = e0[1], K0 = e0[2];
  const int tid = threadIdx.x;
  if (tid < rt.y) {
    const int dI = e0[4 * tid] - I0, dJ = e0[4 * tid + 1] - J0, dK = e0[4 * tid + 2] - K0;
    ebase[tid] = e0[4 * tid + 3] * d.vb;
#pragma unroll
    for (int s = 0; s < 4; ++s)
      if (s < d.nseg) {
        const int64_t* c = d.seg[s].cA;
        eoff[s][tid] = (int)(c[0] * dI + c[1] * dJ + c[2] * dK) * (int)sizeof(cplx);
      }
  }
  __syncthreads();
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l16 = lane & 15, kl = lane >> 4;
  const int v = d.v, rows = rt.y * v;
  const float inv = 1.0f / (float)v;
  const int m0 = tile * kFragRows + (wave >> 1) * 16 * IB, n0 = ct * 64 + (wave & 1) * 16 * JB;
  if (m0 >= rows || n0 >= d.N) return;
  int me[IB], ma[IB], nc[JB];
#pragma unroll
  for (int i = 0; i < IB; ++i) {
    const int m = min(m0 + 16 * i + l16, rows - 1);
    me[i] = quot(m, v, inv);
    ma[i] = m - me[i] * v;
  }
#pragma unroll
  for (int j = 0; j < JB; ++j) nc[j] = min(n0 + 16 * j + l16, d.N - 1);
  Acc<IB, JB> acc;
  acc.clear();
  for (int s = 0; s < d.nseg; ++s) {
    const GemmDesc::Seg& g = d.seg[s];
    const int sak = (int)g.sAk * (int)sizeof(cplx), sbk = (int)g.sBk * (int)sizeof(cplx);
    int ao[IB], bo[JB];
#pragma unroll
    for (int i = 0; i < IB; ++i) ao[i] = eoff[s][me[i]] + ma[i] * (int)g.sAm * (int)sizeof(cplx) + kl * sak;
#pragma unroll
    for (int j = 0; j < JB; ++j) bo[j] = nc[j] * (int)sizeof(cplx) + kl * sbk;
    // resources from the run's first operand blocks on; every offset is inside
    // the operands (host-checked below 2^31 bytes)
    const auto r0 = rsrc(g.A + g.cA[0] * I0 + g.cA[1] * J0 + g.cA[2] * K0, (1 << 27) - 1);
    const __amdgpu_buffer_rsrc_t ra[IB] = {r0, r0};
    const auto rb = rsrc(g.B + g.cB[0] * I0 + g.cB[1] * J0 + g.cB[2] * K0, (1 << 27) - 1);
    contract<IB, JB>(acc, ra, ao, sak, rb, bo, sbk, g.len, kl);
  }
  unsigned co[JB];
#pragma unroll
  for (int j = 0; j < JB; ++j) co[j] = (unsigned)(quot(nc[j], v, inv) * (d.vp - v) + nc[j]);
  const bool cok[JB] = {n0 + l16 < d.N, n0 + 16 + l16 < d.N};
  const unsigned va = (unsigned)v * (unsigned)d.vp;
  int m = m0 + kl, e = quot(m, v, inv), a = m - e * v;
  unsigned off = (unsigned)a * va;
#pragma unroll
  for (int i = 0; i < IB; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      if (m < rows) {
        cplx* c = d.C + ebase[e];
#pragma unroll
        for (int j = 0; j < JB; ++j)
          if (cok[j]) {
            const d2v z = acc.value(i, j, r);
            cplx* p = c + (off + co[j]);
            if (ATOMIC) {
              unsafeAtomicAdd(&p->re, z[0]);
              unsafeAtomicAdd(&p->im, z[1]);
            } else {
              // written once, read by a later kernel: a streaming store leaves the caches to the operands
              __builtin_nontemporal_store(z, reinterpret_cast<d2v*>(p));
            }
          }
      }
      m += 4;
      a += 4;
      off += 4 * va;
      while (a >= v) {  // at most once unless v < 4
        a -= v;
        off -= (unsigned)v * va;
        ++e;
      }
    }
}

// A wave's share of frag_gather: two 16-row blocks by 32 columns, or one by 64.
struct FragUnit {
  int job[2], row[2];  // row blocks (job, first row); row[1] unused when single
  int single;
  int half;  // which 32 of the workgroup's 64 columns (pairs)
};
constexpr int kMaxUnits = 64;
struct FragGather {
  FragJob job[2];
  const cplx* B;
  const int* bl;
  int v, vp, nblk, chunk, ncol, nunit;
  FragUnit unit[kMaxUnits];
};

template <int IB, int JB>
__device__ __forceinline__ void gather_unit(const FragGather& d, const FragUnit& u, int n0, int p0, int p1) {
  typedef const __attribute__((address_space(4))) int cint;  // the table is read-only: scalar loads
  cint* bl = (cint*)(uintptr_t)d.bl;
  const int lane = threadIdx.x & 63, l16 = lane & 15, kl = lane >> 4;
  const int v = d.v, N = v * v;
  const int64_t va = (int64_t)v * d.vp, vb = va * v;
  const float inv = 1.0f / (float)v;
  const FragJob* jb[IB];
  int ao[IB], bo[JB], row[IB], la[IB];
  bool nok[JB];
#pragma unroll
  for (int i = 0; i < IB; ++i) {
    jb[i] = &d.job[u.job[i]];
    row[i] = u.row[i];
    la[i] = (int)jb[i]->lA;
    asm volatile("" : "+s"(la[i]));  // held in a register, not loaded again at each use
    ao[i] = (min(row[i] + l16, jb[i]->M - 1) * (int)jb[i]->sAm + kl) * (int)sizeof(cplx);
  }
#pragma unroll
  for (int j = 0; j < JB; ++j) {
    const int n = n0 + 16 * j + l16, nn = min(n, N - 1);
    nok[j] = n < N;
    bo[j] = (quot(nn, v, inv) * (d.vp - v) + nn + kl * (int)va) * (int)sizeof(cplx);
  }
  Acc<IB, JB> acc;
  acc.clear();
  // The next D steps (of four c) in registers: the blocks stream from HBM, and
  // D steps are about 3000 cycles of products per wave.  A slot is refilled as
  // soon as its step is done, with the block's step D further on or, past its
  // end, with the next block's step that belongs into the slot: one load with
  // scalar selects, so that it never waits.  Rows c >= v of B lie beyond the
  // block's resource and read as zero; A is masked there.  The scalar
  // offset has to begin inside the resource (the range check takes it off
  // the size without a sign), so it is always that of a step of the block: where
  // a block has fewer than D, the slots without one hold the last.
  constexpr int D = 4;
  const int ns = (v + 3) >> 2, rest = v & 3;
  d2v a[D][IB], b[D][JB];
  const cplx *pa[IB], *qa[IB], *pb, *qb;  // this block's and the next one's operands
  auto block = [&](int p, const cplx** xa, const cplx*& xb) {
#pragma unroll
    for (int i = 0; i < IB; ++i)
      xa[i] = jb[i]->A + jb[i]->cA[0] * bl[4 * p] + jb[i]->cA[1] * bl[4 * p + 1] + jb[i]->cA[2] * bl[4 * p + 2];
    xb = d.B + bl[4 * p + 3] * vb;
  };
  auto load = [&](int u, const cplx* const* xa, const cplx* xb, int q) {
#pragma unroll
    for (int i = 0; i < IB; ++i) a[u][i] = frag_load(rsrc(xa[i], la[i]), ao[i], q * 4 * (int)sizeof(cplx));
    const auto rb = rsrc(xb, vb);
#pragma unroll
    for (int j = 0; j < JB; ++j) b[u][j] = frag_load(rb, bo[j], q * 4 * (int)va * (int)sizeof(cplx));
  };
  block(p0, pa, pb);
#pragma unroll
  for (int u = 0; u < D; ++u) load(u, pa, pb, min(u, ns - 1));
  for (int p = p0; p < p1; ++p) {
    const bool last = p + 1 == p1;
    const int q = last ? p : p + 1;
    block(q, qa, qb);
    for (int k = 0; k < ns; k += D) {
#pragma unroll
      for (int u = 0; u < D; ++u) {
        if (k + u >= ns) break;
        if (k + u + 1 == ns && rest) {
#pragma unroll
          for (int i = 0; i < IB; ++i) {
            a[u][i] = d2v{kl < rest ? a[u][i][0] : 0.0, kl < rest ? a[u][i][1] : 0.0};
            asm volatile("" : "+v"(a[u][i]));  // a branch: these selects belong to one step of a block only
          }
        }
        acc.step(a[u], b[u]);
        __builtin_amdgcn_sched_barrier(0);  // the refill follows the products of its slot
        const bool in = k + u + D < ns;
        const cplx* xa[IB];
#pragma unroll
        for (int i = 0; i < IB; ++i) xa[i] = in ? pa[i] : qa[i];
        load(u, xa, in ? pb : qb, in ? k + u + D : u);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
#pragma unroll
    for (int i = 0; i < IB; ++i) pa[i] = qa[i];
    pb = qb;
    const int I = bl[4 * p], J = bl[4 * p + 1], K = bl[4 * p + 2];
    const int dI = bl[4 * q] - I, dJ = bl[4 * q + 1] - J, dK = bl[4 * q + 2] - K;
#pragma unroll
    for (int i = 0; i < IB; ++i) {
      const FragJob& g = *jb[i];
      if (!last && g.cC[0] * dI + g.cC[1] * dJ + g.cC[2] * dK == 0) continue;  // the next block has the same output
      cplx* C = g.C + g.cC[0] * I + g.cC[1] * J + g.cC[2] * K;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = row[i] + 4 * r + kl;
        if (m >= g.M) continue;
#pragma unroll
        for (int j = 0; j < JB; ++j)
          if (nok[j]) {
            const d2v z = acc.value(i, j, r);
            cplx* c = C + m * g.sCm + (n0 + 16 * j + l16);
            unsafeAtomicAdd(&c->re, g.alpha * z[0]);
            unsafeAtomicAdd(&c->im, g.alpha * z[1]);
          }
      }
      acc.clear(i);
    }
  }
}

// The waves of a chunk of the block list and 64 columns are its units: the
// 16-row blocks of all jobs, two and two by 32 columns or a last one by 64 (12
// MFMAs a step either way).  They read the same rows of B, which come from HBM
// once and from the caches for the other units; waves are numbered through, so
// that four of them fill a workgroup whatever the number of units (as
// workgroups of a chunk's units, five at o=15, v=57, only one would fit on a
// CU: 8.5 ms).  At o=15, v=57 Z_i and the Y2 product, 6.9 ms apart, take 5.8 ms,
// the two X2 products 2.9 instead of 3.85 ms; 0.71 -> 0.49 and 0.39 -> 0.28 ms at
// o=10, v=38.  Bound by the matrix cores (4.0 ms of MFMAs) and, for the X2
// pair, by the 10 GB it reads.
__global__ __launch_bounds__(256, 2) void frag_gather_kernel(FragGather d) {
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int64_t w = (int64_t)xcd_contiguous((int)blockIdx.x, (int)gridDim.x) * 4 + wave;
  const int lg = (int)(w / d.nunit);
  const FragUnit& u = d.unit[w % d.nunit];
  const int p0 = lg / d.ncol * d.chunk, p1 = min(d.nblk, p0 + d.chunk);
  const int n0 = lg % d.ncol * 64 + (u.single ? 0 : 32 * u.half);
  if (p0 >= p1 || n0 >= d.v * d.v) return;
  if (u.single)
    gather_unit<1, 4>(d, u, n0, p0, p1);
  else
    gather_unit<2, 2>(d, u, n0, p0, p1);
}

// A operands of frag_cols in the order the waves read them: the panel of K and
// row block i holds, step of four k by step, the 64 lanes' elements (l%16 the
// row, l/16 the k), zero beyond the operand.
struct ColsPack {
  ColsJob job[2];
  int nrb[2], njob, n, steps;  // row blocks per job, extent of K, steps with the partial one
  int64_t v2;
  cplx* dst;
};
__global__ __launch_bounds__(256) void cols_pack_kernel(ColsPack d) {
  const int nrb = d.nrb[0] + d.nrb[1];
  const int64_t total = (int64_t)d.n * nrb * d.steps * 64;
  for (int64_t x = (int64_t)blockIdx.x * 256 + threadIdx.x; x < total; x += (int64_t)gridDim.x * 256) {
    const int l = (int)(x & 63);
    const int64_t t = x >> 6;
    const int q = (int)(t % d.steps);
    const int64_t p = t / d.steps;
    const int i = (int)(p % nrb), K = (int)(p / nrb);
    const ColsJob& g = d.job[i < d.nrb[0] ? 0 : 1];
    const int m = 16 * (i < d.nrb[0] ? i : i - d.nrb[0]) + (l & 15);
    const int64_t k = 4 * (int64_t)q + (l >> 4);
    d.dst[x] = m < g.M && k < d.v2 ? g.A[g.cAK * K + m * g.sAm + k] : cplx{0, 0};
  }
}

// A wave's row blocks in frag_cols.
struct ColsUnit {
  int nb;
  int job[5], row[5], panel[5];
};
constexpr int kMaxColsUnits = 32;
struct FragCols {
  ColsJob job[2];
  const cplx* B;
  const int* bl;
  const int* part;
  const int4* frag;
  const cplx* pack;  // panels of the row blocks, npanel per K
  int npanel;
  int perm[3];
  int v, vp, nfrag, nunit, steps, nsplit;  // full steps of four k in all, and per split
  ColsUnit unit[kMaxColsUnits];
};

template <int IB, int NS>
__device__ __forceinline__ void cols_unit(const FragCols& d, const ColsUnit& u, int f, int split) {
  constexpr int D = NS == 3 && IB <= 4 ? 4 : 3;
  const int lane = threadIdx.x & 63, l16 = lane & 15, kl = lane >> 4;
  const int v = d.v;
  const int64_t vb = (int64_t)v * v * d.vp;
  const int4 fr = d.frag[f];
  const bool ok = l16 < fr.z;
  int e = fr.x, b = fr.y + (ok ? l16 : 0);
  while (b >= v) {
    b -= v;
    ++e;
  }
  const int I = d.bl[4 * e], J = d.bl[4 * e + 1], n = d.bl[4 * e + 3];
  const int K = __builtin_amdgcn_readfirstlane(d.bl[4 * e + 2]);  // the same for all columns of a fragment
  // B: one resource per stream from the lowest of the lanes' blocks on (the
  // table keeps a fragment's blocks within 2^31 bytes of each other)
  __amdgpu_buffer_rsrc_t rb[NS];
  int bo[NS];
#pragma unroll
  for (int w = 0; w < NS; ++w) {
    const int slot = d.part[6 * n + d.perm[w]];
    int lo = slot;
#pragma unroll
    for (int x = 1; x < 16; x <<= 1) lo = min(lo, __shfl_xor(lo, x));
    lo = __builtin_amdgcn_readfirstlane(lo);
    rb[w] = __builtin_amdgcn_make_buffer_rsrc((void*)(d.B + lo * vb), 0, -1, kRsrcWord3);
    bo[w] = (int)(((uint32_t)(slot - lo) * (uint32_t)vb + (uint32_t)(b + kl * d.vp)) * (uint32_t)sizeof(cplx));
  }
  __amdgpu_buffer_rsrc_t ra[IB];
  int ao[IB];
#pragma unroll
  for (int i = 0; i < IB; ++i) {
    const int64_t len = (int64_t)((v * v + 3) / 4) * 64;
    ra[i] = rsrc(d.pack + ((int64_t)K * d.npanel + u.panel[i]) * len, len);
    ao[i] = lane * (int)sizeof(cplx);
  }
  const int sbk = 4 * d.vp * (int)sizeof(cplx);
  Acc<IB, 1> acc;
  acc.clear();
  d2v a[D][IB], x[D][NS];
  auto load = [&](int r, int q) {
#pragma unroll
    for (int i = 0; i < IB; ++i) a[r][i] = frag_load(ra[i], ao[i], q * 64 * (int)sizeof(cplx));
#pragma unroll
    for (int w = 0; w < NS; ++w) x[r][w] = frag_load(rb[w], bo[w], q * sbk);
  };
  auto step = [&](const d2v* ar, const d2v* xr) {
    d2v z = xr[0];
    if constexpr (NS == 3) {
      const d2v t{xr[1][0] + xr[2][0], xr[1][1] + xr[2][1]};
      z = d2v{__builtin_fma(2.0, xr[0][0], -t[0]), __builtin_fma(2.0, xr[0][1], -t[1])};
    }
    acc.step(ar, &z);
  };
  const int q0 = split * d.steps / d.nsplit, q1 = (split + 1) * d.steps / d.nsplit;
  if (q0 < q1) {
#pragma unroll
    for (int r = 0; r < D; ++r) load(r, min(q0 + r, q1 - 1));
    for (int q = q0; q < q1; q += D) {
#pragma unroll
      for (int r = 0; r < D; ++r) {
        if (q + r >= q1) break;
        step(a[r], x[r]);
        __builtin_amdgcn_sched_barrier(0);  // the refill follows the products of its slot
        load(r, min(q + r + D, q1 - 1));
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  const int rest = (v * v) & 3;
  if (rest && split + 1 == d.nsplit) {  // the last k: A is zero at the missing ones, B reads a valid k
    const int back = min(kl, rest - 1) - kl;
    d2v at[IB], xt[NS];
#pragma unroll
    for (int i = 0; i < IB; ++i) at[i] = frag_load(ra[i], ao[i], d.steps * 64 * (int)sizeof(cplx));
#pragma unroll
    for (int w = 0; w < NS; ++w) xt[w] = frag_load(rb[w], bo[w] + back * d.vp * (int)sizeof(cplx), d.steps * sbk);
    step(at, xt);
  }
  if (!ok) return;
#pragma unroll
  for (int i = 0; i < IB; ++i) {
    const ColsJob& g = d.job[u.job[i]];
    cplx* C = g.C + g.cC[0] * I + g.cC[1] * J + b * g.sCb;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int m = u.row[i] + 4 * r + kl;
      if (m >= g.M) continue;
      const d2v z = acc.value(i, 0, r);
      cplx* c = C + m * g.sCm;
      unsafeAtomicAdd(&c->re, z[0]);
      unsafeAtomicAdd(&c->im, z[1]);
    }
  }
}

// X2 (three streams) and Y2 with R8 (one).  Bound by the matrix cores (Y2: MFMA
// busy 0.88 of the SIMD cycles) and, for X2, by the three orderings of each
// block that pass through the L2.  o=15, v=57, alone: X2 5.9 -> 5.2 ms, Y2 and R8
// 7.6 -> 5.3; o=10, v=38: 0.73 -> 0.46 and 0.85 -> 0.51, since columns of all
// entries of a K are numbered through and rows come in blocks of 16.  A read
// straight from the integrals (64-byte pieces of rows 52 KB apart) instead of
// packed panels made that 9.6 and 7.8 ms.
// One wave per 16 columns, group of row blocks and split of k, four to a
// workgroup as they come (splits outermost, so that the waves that run
// together read the same stretch of k of blocks they share).
template <int NS>
__global__ __launch_bounds__(256, 2) void frag_cols_kernel(FragCols d) {
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int64_t w = (int64_t)xcd_contiguous((int)blockIdx.x, (int)gridDim.x) * 4 + wave;
  const int split = (int)(w / ((int64_t)d.nfrag * d.nunit));
  if (split >= d.nsplit) return;
  const int f = (int)(w / d.nunit % d.nfrag);
  const ColsUnit& u = d.unit[w % d.nunit];
  switch (u.nb) {
    case 1:
      cols_unit<1, NS>(d, u, f, split);
      break;
    case 2:
      cols_unit<2, NS>(d, u, f, split);
      break;
    case 3:
      cols_unit<3, NS>(d, u, f, split);
      break;
    case 4:
      cols_unit<4, NS>(d, u, f, split);
      break;
    default:
      cols_unit<5, NS>(d, u, f, split);
  }
}

// Column operands of frag_block in the order the waves read them: the panel of
// an operand and key holds, step of four k by step, the columns' four elements,
// zero beyond the last k.
struct BlockPack {
  struct {
    const cplx* B;
    int64_t sKey, sB;
  } src[kMaxBlockCols];
  int64_t v2;
  int nsrc, n, o, steps;
  cplx* dst;
};
__global__ __launch_bounds__(256) void block_pack_kernel(BlockPack d) {
  const int64_t total = (int64_t)d.nsrc * d.o * d.steps * d.n * 4;
  for (int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x; t < total; t += (int64_t)gridDim.x * 256) {
    const int x = (int)((t >> 2) % d.n);
    const int64_t r = (t >> 2) / d.n;
    const int panel = (int)(r / d.steps);
    const int64_t k = 4 * (r % d.steps) + (t & 3);
    const auto& g = d.src[panel / d.o];
    d.dst[t] = k < d.v2 ? g.B[g.sKey * (panel % d.o) + x * g.sB + k] : cplx{0, 0};
  }
}

struct FragBlock {
  BlockCols g[kMaxBlockCols];
  int panel[kMaxBlockCols];  // a group's first panel
  BlockTrace tr[kMaxBlockCols];
  int ng, n, ntr;
  const cplx* X;
  const cplx* pack;
  const int* bl;
  const int* part;
  int perm, v, vp, nblk, nfrag, nrg, steps, nsplit;
  int row0[8], nb[8];  // groups of row blocks: first row and number
};

template <int IB>
__device__ __forceinline__ void block_unit(const FragBlock& d, int e, int f, int row0, int split) {
  constexpr int D = 3;
  const int lane = threadIdx.x & 63, l16 = lane & 15, kl = lane >> 4;
  const int v = d.v;
  const int64_t vb = (int64_t)v * v * d.vp;
  const int ijk[3] = {d.bl[4 * e], d.bl[4 * e + 1], d.bl[4 * e + 2]};
  const int slot = __builtin_amdgcn_readfirstlane(d.part[6 * d.bl[4 * e + 3] + d.perm]);
  auto pick = [&](int w) { return w == 0 ? ijk[0] : w == 1 ? ijk[1] : ijk[2]; };
  // the lane's column: its group and its place there; one resource from the
  // lowest of the lanes' panels on
  const int c = 16 * f + l16;
  const bool ok = c < d.ng * d.n;
  const int gi = ok ? c / d.n : 0, x = ok ? c % d.n : 0;
  const BlockCols& g = d.g[gi];
  const int panel = d.panel[gi] + pick(g.key);
  int lo = panel;
#pragma unroll
  for (int m = 1; m < 16; m <<= 1) lo = min(lo, __shfl_xor(lo, m));
  lo = __builtin_amdgcn_readfirstlane(lo);
  const int plen = (v * v + 3) / 4 * 4 * d.n;
  const auto rb = __builtin_amdgcn_make_buffer_rsrc((void*)(d.pack + (int64_t)lo * plen), 0, -1, kRsrcWord3);
  const int bo = (int)(((uint32_t)(panel - lo) * (uint32_t)plen + (uint32_t)(4 * x + kl)) * (uint32_t)sizeof(cplx));
  const auto ra = rsrc(d.X + slot * vb, vb);
  int ao[IB];
#pragma unroll
  for (int i = 0; i < IB; ++i) ao[i] = (min(row0 + 16 * i + l16, v - 1) + kl * d.vp) * (int)sizeof(cplx);
  const int sak = 4 * d.vp * (int)sizeof(cplx), sbk = 4 * d.n * (int)sizeof(cplx);
  Acc<IB, 1> acc;
  acc.clear();
  d2v a[D][IB], b[D];
  auto load = [&](int r, int q) {
#pragma unroll
    for (int i = 0; i < IB; ++i) a[r][i] = frag_load(ra, ao[i], q * sak);
    b[r] = frag_load(rb, bo, q * sbk);
  };
  const int q0 = split * d.steps / d.nsplit, q1 = (split + 1) * d.steps / d.nsplit;
  if (q0 < q1) {
#pragma unroll
    for (int r = 0; r < D; ++r) load(r, min(q0 + r, q1 - 1));
    for (int q = q0; q < q1; q += D) {
#pragma unroll
      for (int r = 0; r < D; ++r) {
        if (q + r >= q1) break;
        acc.step(a[r], &b[r]);
        __builtin_amdgcn_sched_barrier(0);  // the refill follows the products of its slot
        load(r, min(q + r + D, q1 - 1));
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  const int rest = (v * v) & 3;
  if (rest && split + 1 == d.nsplit) {  // the last k: B is zero at the missing ones, A reads a valid k
    const int back = min(kl, rest - 1) - kl;
    d2v at[IB];
#pragma unroll
    for (int i = 0; i < IB; ++i) at[i] = frag_load(ra, ao[i] + back * d.vp * (int)sizeof(cplx), d.steps * sak);
    const d2v bt = frag_load(rb, bo, d.steps * sbk);
    acc.step(at, &bt);
  }
  if (!ok) return;
  auto add = [&](cplx* C, int64_t sCm, double alpha) {
#pragma unroll
    for (int i = 0; i < IB; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = row0 + 16 * i + 4 * r + kl;
        if (m >= v) continue;
        const d2v z = acc.value(i, 0, r);
        cplx* q = C + m * sCm;
        unsafeAtomicAdd(&q->re, alpha * z[0]);
        unsafeAtomicAdd(&q->im, alpha * z[1]);
      }
  };
  add(g.C + g.cC[0] * ijk[0] + g.cC[1] * ijk[1] + g.cC[2] * ijk[2] + x * g.sCx, g.sCm, g.alpha);
  for (int t = 0; t < d.ntr; ++t) {
    const BlockTrace& u = d.tr[t];
    if (u.group == gi && x == pick(u.col)) add(u.C + u.sC * pick(u.row), 1, u.alpha);
  }
}

// Terms 1, 2, 5 and 6 of Y1 with X1 and terms 3 and 4 as traces of them.  Bound
// by the matrix cores.  o=15, v=57, alone: 5.95 -> 4.7 ms; o=10, v=38: 0.76 ->
// 0.49; o=16, v=66: 26.4 (16-wide columns of each segment, X1 and terms 3 and 4
// in a sweep of their own) -> 8.7.  The columns of all groups are numbered
// through (4 o of them, so that little of the 16-wide fragments is padding) and
// packed: read where they lie, as 16 pieces of 64 bytes v^2 apart each step, they
// made that 6.6, 0.78 and 14.2 ms.
// One wave per block, 16 columns, group of row blocks and split of k; the
// waves of a block follow each other, so that they share its rows in the L1.
__global__ __launch_bounds__(256, 2) void frag_block_kernel(FragBlock d) {
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int64_t w = (int64_t)xcd_contiguous((int)blockIdx.x, (int)gridDim.x) * 4 + wave;
  const int per = d.nfrag * d.nrg;
  const int64_t t = w / per;
  const int r = (int)(w % per), f = r % d.nfrag, rg = r / d.nfrag;
  const int e = (int)(t / d.nsplit), split = (int)(t % d.nsplit);
  if (e >= d.nblk) return;
  switch (d.nb[rg]) {
    case 1:
      block_unit<1>(d, e, f, d.row0[rg], split);
      break;
    case 2:
      block_unit<2>(d, e, f, d.row0[rg], split);
      break;
    case 3:
      block_unit<3>(d, e, f, d.row0[rg], split);
      break;
    case 4:
      block_unit<4>(d, e, f, d.row0[rg], split);
      break;
    default:
      block_unit<5>(d, e, f, d.row0[rg], split);
  }
}

// x / d for 0 <= x < 2^31 by a multiplication: with 2^(s-1) < d <= 2^s, m =
// floor(2^(31+s) / d) + 1 is at most 2^32 - 1 and too large by less than 2^-s of
// 2^31 (an integer division takes some 35 instructions, which is what a small
// product waits for).
struct Divisor {
  uint32_t d = 1, m = 0x80000001u, s = 0;
  Divisor() = default;
  explicit Divisor(int64_t x) : d((uint32_t)x) {
    while ((1ll << s) < x) ++s;
    m = (uint32_t)((1ull << (31 + s)) / d + 1);
  }
  __device__ __forceinline__ int quot(int x) const { return (int)(__umulhi(2u * (uint32_t)x, m) >> s); }
};

struct FragGemm {
  const cplx* A;
  const cplx* B;
  cplx* C;
  int M, N, M0, N0;
  Divisor per, fast, split, dM0, dN0, drun;  // workgroups of an entry and split, those of its fast index, ksplit, M0, N0, run
  int64_t sAm1, sAm0, sBn1, sBn0, sCm1, sCm0, sCn1, sCn0, sAb, sBb, sCb;
  const int* bl;
  int64_t cA[4], cB[4], cC[4];
  int64_t nA, nB;              // elements from an entry's first to past its last
  int K0, steps;               // inner extent of k; steps of four in all (one level: full ones)
  int sak1, sak0, sbk1, sbk0;  // bytes per k
  int mt, nt, wm, wn, gm, gn;  // wave tiles; a workgroup's tiles; workgroups along M and N
  int mfast;                   // consecutive workgroups walk along M
  int ksplit;
  int mode;                    // 0: C += , 1: C = , 2: atomic C +=
  double are, aim;
};

// C[m][n] (+)= alpha sum_k A[m][k] B[k][n] of one entry, tile of 16 IB x 16 JB
// and split of k.  KW = 1: a workgroup's four waves take neighbouring tiles;
// else its KW waves split the k of one tile and add up through the LDS.
// Steps are of four k; two are loaded at a time, so that an operand stored
// k-fast is read in whole lines.  k of one level (TAIL < 0): the last K % 4 go
// first, in a step that reads zeros past the last.  k of two levels, inner runs
// of K0: such a step ends each run (TAIL = 1), or K0 % 4 is zero (TAIL = 0).
//
// The plain products of the einsum engine.  Bound by the matrix cores where the
// contraction is long (o=4, v=96, the two ladders over 9216 virtual pairs with
// 300 rows: 51 and 75 TFLOP/s, k-fast against n-fast columns), by C where it is
// short (3249 x 3249 x 216: 338 MB of C, 0.33 ms at 55 TFLOP/s), by latency and
// launch below some 10^8 terms.  A right-hand side's products, kernel time, one
// launch each: o=15, v=57 8.2 -> 6.1 ms, o=4, v=96 16.5 -> 15.1, o=5, v=18 2.0 ->
// 0.69 (an 18 us LDS-tiled product with its split added by atomics becomes one
// of 6 us: a workgroup's waves split k down to a few steps each); queued in
// levels 6.0, 14.3 and, at o=5, v=19, 0.30.  Steps in pairs with k
// next to each other (8u + 2 (l/16) + 0, 1) made k-fast operands read half lines
// twice as often: 6.6 ms at o=15.  Where a workgroup has one block, its thread's
// element of C is loaded before the product and indexes are divided by
// multiplications: o=5, v=18 0.67 -> 0.56 ms.
template <int IB, int JB, int KW, int TAIL>
__device__ __forceinline__ void frag_gemm_tile(const FragGemm& d, const int g, d2v* red) {
  constexpr int R = IB * JB > 1 || KW > 4 ? 4 : 6;  // steps in flight
  const int lane = threadIdx.x & 63, l16 = lane & 15, kl = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int ge = d.per.quot(g), t = g - ge * (int)d.per.d;
  const int e = d.split.quot(ge), ks = ge - e * (int)d.split.d;
  const int slow = d.fast.quot(t), fast = t - slow * (int)d.fast.d;
  int ti = d.mfast ? fast : slow, tj = d.mfast ? slow : fast;
  if constexpr (KW == 1) {
    ti = ti * d.wm + wave % d.wm;
    tj = tj * d.wn + wave / d.wm;
    if (ti >= d.mt || tj >= d.nt) return;
  }
  const cplx* pA = d.A;
  const cplx* pB = d.B;
  cplx* pC = d.C;
  if (d.bl) {
    const int* q = d.bl + 4 * (int64_t)e;
    const int q0 = q[0], q1 = q[1], q2 = q[2], q3 = q[3];
    pA += d.cA[0] * q0 + d.cA[1] * q1 + d.cA[2] * q2 + d.cA[3] * q3;
    pB += d.cB[0] * q0 + d.cB[1] * q1 + d.cB[2] * q2 + d.cB[3] * q3;
    pC += d.cC[0] * q0 + d.cC[1] * q1 + d.cC[2] * q2 + d.cC[3] * q3;
  } else {
    pA += d.sAb * e;
    pB += d.sBb * e;
    pC += d.sCb * e;
  }
  auto off = [](int x, int X, const Divisor& X0, int64_t s1, int64_t s0) {
    if ((int)X0.d == X) return x * s0;
    const int h = X0.quot(x);
    return h * s1 + (x - h * (int)X0.d) * s0;
  };
  const auto ra = rsrc(pA, d.nA), rb = rsrc(pB, d.nB);
  auto at_c = [&](int m, int n) {
    return pC + off(m, d.M, d.dM0, d.sCm1, d.sCm0) + off(n, d.N, d.dN0, d.sCn1, d.sCn0);
  };
  // one block a workgroup: the thread's element of C, on its way as long as the
  // product is formed
  [[maybe_unused]] cplx* c1 = nullptr;
  [[maybe_unused]] d2v old = {0, 0};
  if constexpr (IB * JB == 1) {
    const int x = threadIdx.x, m = 16 * ti + 4 * (x >> 6) + kl, n = 16 * tj + l16;
    if (x < 256 && m < d.M && n < d.N) {
      c1 = at_c(m, n);
      if (d.mode == 0) old = *reinterpret_cast<const d2v*>(c1);
    }
  }
  constexpr int kOut = 0x7ffffff0;  // beyond every operand (spans below 2^31 bytes)
  // row and column offsets, and those of the lane's first k
  constexpr bool TWO = TAIL >= 0;
  int ao[IB], bo[JB], al[IB], bl[JB];
  const int rest = d.K0 & 3;
#pragma unroll
  for (int i = 0; i < IB; ++i) {
    ao[i] = (int)off(min(16 * (ti * IB + i) + l16, d.M - 1), d.M, d.dM0, d.sAm1, d.sAm0) * (int)sizeof(cplx) + kl * d.sak0;
    al[i] = kl < rest ? ao[i] : kOut;
  }
#pragma unroll
  for (int j = 0; j < JB; ++j) {
    bo[j] = (int)off(min(16 * (tj * JB + j) + l16, d.N - 1), d.N, d.dN0, d.sBn1, d.sBn0) * (int)sizeof(cplx) + kl * d.sbk0;
    bl[j] = kl < rest ? bo[j] : kOut;
  }
  // the wave's steps
  const int nsp = d.ksplit * KW, sp = KW == 1 ? ks : ks * KW + wave;
  const int t0 = (int)((int64_t)d.steps * sp / nsp), t1 = (int)((int64_t)d.steps * (sp + 1) / nsp);
  Acc<IB, JB> acc;
  acc.clear();
  d2v a[R][IB], b[R][JB];
  [[maybe_unused]] d2v at[IB], bt[JB];
  [[maybe_unused]] const bool tail = !TWO && rest > 0 && sp + 1 == nsp;
  if constexpr (!TWO) {
    if (tail) {
#pragma unroll
      for (int i = 0; i < IB; ++i) at[i] = frag_load(ra, al[i], d.steps * 4 * d.sak0);
#pragma unroll
      for (int j = 0; j < JB; ++j) bt[j] = frag_load(rb, bl[j], d.steps * 4 * d.sbk0);
    }
  }
  [[maybe_unused]] const int run = (d.K0 + 3) >> 2;  // steps of an inner run
  [[maybe_unused]] int k1 = 0, q = 0;
  if constexpr (TWO) {
    k1 = d.drun.quot(t0);
    q = t0 - k1 * run;
  }
  auto load = [&](int r, int t) {
    if constexpr (TWO) {
      const int sa = k1 * d.sak1 + 4 * q * d.sak0, sb = k1 * d.sbk1 + 4 * q * d.sbk0;
      const bool last = q + 1 == run;
#pragma unroll
      for (int i = 0; i < IB; ++i) a[r][i] = frag_load(ra, TAIL && last ? al[i] : ao[i], sa);
#pragma unroll
      for (int j = 0; j < JB; ++j) b[r][j] = frag_load(rb, TAIL && last ? bl[j] : bo[j], sb);
      if (t + 1 < t1) {
        q = last ? 0 : q + 1;
        k1 = last ? k1 + 1 : k1;
      }
    } else {
      const int x = 4 * min(t, t1 - 1);
#pragma unroll
      for (int i = 0; i < IB; ++i) a[r][i] = frag_load(ra, ao[i], x * d.sak0);
#pragma unroll
      for (int j = 0; j < JB; ++j) b[r][j] = frag_load(rb, bo[j], x * d.sbk0);
    }
  };
  if (t0 < t1) {
#pragma unroll
    for (int r = 0; r < R; ++r) load(r, t0 + r);
  }
  if constexpr (!TWO) {
    if (tail) acc.step(at, bt);
  }
  if (t0 < t1) {
    for (int t = t0; t < t1; t += R) {
#pragma unroll
      for (int r = 0; r < R; r += 2) {
        if (t + r >= t1) break;
        acc.step(a[r], b[r]);
        if (t + r + 1 >= t1) break;
        acc.step(a[r + 1], b[r + 1]);
        __builtin_amdgcn_sched_barrier(0);  // the refill follows the products of its slots
        load(r, t + r + R);
        load(r + 1, t + r + 1 + R);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  auto put = [&](int m, int n, d2v z) {
    cplx* c = at_c(m, n);
    const double re = d.are * z[0] - d.aim * z[1], im = d.are * z[1] + d.aim * z[0];
    if (d.mode == 2) {
      unsafeAtomicAdd(&c->re, re);
      unsafeAtomicAdd(&c->im, im);
    } else if (d.mode == 1) {
      *c = cplx{re, im};
    } else {
      *c = cplx{c->re + re, c->im + im};
    }
  };
  if constexpr (KW == 1) {
#pragma unroll
    for (int i = 0; i < IB; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int j = 0; j < JB; ++j) {
          const int m = 16 * (ti * IB + i) + 4 * r + kl, n = 16 * (tj * JB + j) + l16;
          if (m < d.M && n < d.N) put(m, n, acc.value(i, j, r));
        }
  } else {
#pragma unroll
    for (int i = 0; i < IB; ++i)
#pragma unroll
      for (int j = 0; j < JB; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) red[((wave * IB * JB + i * JB + j) * 4 + r) * 64 + lane] = acc.value(i, j, r);
    __syncthreads();
    if constexpr (IB * JB == 1) {
      if (!c1) return;
      d2v z = red[threadIdx.x];
#pragma unroll
      for (int w = 1; w < KW; ++w) z += red[w * 256 + threadIdx.x];
      const double re = d.are * z[0] - d.aim * z[1], im = d.are * z[1] + d.aim * z[0];
      if (d.mode == 2) {
        unsafeAtomicAdd(&c1->re, re);
        unsafeAtomicAdd(&c1->im, im);
      } else {
        *c1 = cplx{old[0] + re, old[1] + im};
      }
      return;
    }
    for (int x = threadIdx.x; x < IB * JB * 256; x += KW * 64) {
      d2v z = red[x];
#pragma unroll
      for (int w = 1; w < KW; ++w) z += red[w * IB * JB * 256 + x];
      const int l = x & 63, r = (x >> 6) & 3, ij = x >> 8;
      const int m = 16 * (ti * IB + ij / JB) + 4 * r + (l >> 4), n = 16 * (tj * JB + ij % JB) + (l & 15);
      if (m < d.M && n < d.N) put(m, n, z);
    }
  }
}

template <int IB, int JB, int KW, int TAIL>
__global__ __launch_bounds__((KW == 1 ? 4 : KW) * 64, (IB * JB > 1 ? 2 : 4)) void frag_gemm_kernel(FragGemm d) {
  __shared__ d2v red[KW == 1 ? 1 : KW * IB * JB * 256];
  frag_gemm_tile<IB, JB, KW, TAIL>(d, xcd_contiguous((int)blockIdx.x, (int)gridDim.x), red);
}

// Several small products that do not depend on each other in one launch, one
// block of 16 x 16 a workgroup and its k split over eight waves.  A launch of a
// small product is 4 to 8 us of latency whatever its size.
constexpr int kGroup = 8;
struct FragGroup {
  FragGemm g[kGroup];
  int end[kGroup];   // workgroups up to and with product i
  int tail[kGroup];  // TAIL of its tile
  int n;
};
static_assert(sizeof(FragGroup) <= 4096, "kernel arguments");
__global__ __launch_bounds__(512, 4) void frag_group_kernel(FragGroup d) {
  __shared__ d2v red[8 * 256];
  int i = 0;
  while (i + 1 < d.n && (int)blockIdx.x >= d.end[i]) ++i;
  const FragGemm& g = d.g[i];
  const int x = (int)blockIdx.x - (i > 0 ? d.end[i - 1] : 0);
  if (d.tail[i] < 0)
    frag_gemm_tile<1, 1, 8, -1>(g, x, red);
  else if (d.tail[i] > 0)
    frag_gemm_tile<1, 1, 8, 1>(g, x, red);
  else
    frag_gemm_tile<1, 1, 8, 0>(g, x, red);
}

template <int IB, int JB, int KW>
void launch_frag_gemm(FragGemm& d, int batch, bool two, hipStream_t s) {
  const int64_t wg = (int64_t)d.gm * d.gn * d.ksplit * batch;
  RTCC3_CHECK(wg < (1LL << 31), "frag: product too large");
  const dim3 grid((unsigned)wg), block((KW == 1 ? 4 : KW) * 64);
  if (!two)
    hipLaunchKernelGGL((frag_gemm_kernel<IB, JB, KW, -1>), grid, block, 0, s, d);
  else if (d.K0 & 3)
    hipLaunchKernelGGL((frag_gemm_kernel<IB, JB, KW, 1>), grid, block, 0, s, d);
  else
    hipLaunchKernelGGL((frag_gemm_kernel<IB, JB, KW, 0>), grid, block, 0, s, d);
  RTCC3_HIP(hipGetLastError());
}

}  // namespace

namespace {

// First panel of each group's operand, groups with the same one sharing it;
// returns the number of panels.
int block_panels(const BlockCols* g, int ng, int o, int* panel) {
  int np = 0;
  for (int q = 0; q < ng; ++q) {
    panel[q] = -1;
    for (int p = 0; p < q && panel[q] < 0; ++p)
      if (g[p].B == g[q].B && g[p].sKey == g[q].sKey && g[p].sB == g[q].sB) panel[q] = panel[p];
    if (panel[q] >= 0) continue;
    panel[q] = np;
    np += o;
  }
  return np;
}

}  // namespace

int64_t frag_block_pack(const BlockCols* groups, int ng, int n, int o, int v) {
  int panel[kMaxBlockCols];
  RTCC3_CHECK(ng <= kMaxBlockCols, "frag: too many column groups");
  return (int64_t)block_panels(groups, ng, o, panel) * (((int64_t)v * v + 3) / 4 * 4 * n);
}

int frag_block(const BlockCols* groups, int ng, int n, const BlockTrace* tr, int ntr, const cplx* X, int perm, int o,
               int v, int vp, const int* part, const int* bl, int nblk, cplx* pack, hipStream_t s, int64_t reach) {
  if (nblk <= 0 || ng <= 0) return 0;
  RTCC3_CHECK(ng <= kMaxBlockCols && ntr <= kMaxBlockCols && n >= 1 && v >= 1 && vp >= v &&
                  (int64_t)v * v * vp < (1LL << 27) && ((int64_t)v * v + 3) * n < (1LL << 27),
              "frag: bad block product");
  FragBlock d;
  const int64_t plen = ((int64_t)v * v + 3) / 4 * 4 * n;
  if (ng > 1 && (block_panels(groups, ng, o, d.panel) + 1) * plen * (int64_t)sizeof(cplx) > reach) {
    // a fragment's panels have to lie within reach: with one group it has one
    int launches = 0;
    for (int q = 0; q < ng; ++q) {
      std::vector<BlockTrace> own;
      for (int t = 0; t < ntr; ++t)
        if (tr[t].group == q) {
          own.push_back(tr[t]);
          own.back().group = 0;
        }
      launches += frag_block(groups + q, 1, n, own.data(), (int)own.size(), X, perm, o, v, vp, part, bl, nblk, pack, s);
    }
    return launches;
  }
  block_panels(groups, ng, o, d.panel);
  d.ng = ng;
  d.n = n;
  d.ntr = ntr;
  for (int t = 0; t < ntr; ++t) d.tr[t] = tr[t];
  BlockPack pk;
  pk.v2 = (int64_t)v * v;
  pk.n = n;
  pk.o = o;
  pk.steps = (v * v + 3) / 4;
  pk.nsrc = 0;
  pk.dst = pack;
  for (int q = 0; q < ng; ++q) {
    d.g[q] = groups[q];
    if (d.panel[q] == pk.nsrc * o) pk.src[pk.nsrc++] = {groups[q].B, groups[q].sKey, groups[q].sB};
  }
  const int64_t packed = (int64_t)pk.nsrc * o * plen;
  hipLaunchKernelGGL(block_pack_kernel, dim3((unsigned)std::min<int64_t>((packed + 255) / 256, 65536)), dim3(256), 0, s,
                     pk);
  RTCC3_HIP(hipGetLastError());
  int launches = 1;
  d.X = X;
  d.pack = pack;
  d.bl = bl;
  d.part = part;
  d.perm = perm;
  d.v = v;
  d.vp = vp;
  d.nblk = nblk;
  d.nfrag = (ng * n + 15) / 16;
  d.steps = v * v / 4;
  const int nrb = (v + 15) / 16, nrg = (nrb + 4) / 5;
  for (int g0 = 0; g0 < nrg; g0 += 8) {
    d.nrg = std::min(8, nrg - g0);
    for (int g = 0; g < d.nrg; ++g) {
      const int r0 = nrb * (g0 + g) / nrg, r1 = nrb * (g0 + g + 1) / nrg;
      d.row0[g] = 16 * r0;
      d.nb[g] = r1 - r0;
    }
    // splits of k for at least four rounds of the chip's 2048 waves, of 32 steps or more
    const int64_t waves = (int64_t)nblk * d.nfrag * d.nrg;
    d.nsplit = (int)std::max<int64_t>(1, std::min<int64_t>((4 * 2048 + waves - 1) / waves, d.steps / 32));
    const int64_t nw = waves * d.nsplit;
    RTCC3_CHECK(nw < (1LL << 31), "frag: product too large");
    hipLaunchKernelGGL(frag_block_kernel, dim3((unsigned)((nw + 3) / 4)), dim3(256), 0, s, d);
    RTCC3_HIP(hipGetLastError());
    ++launches;
  }
  return launches;
}

namespace {

// The largest offset of a two-level index plus one.
int64_t reach(int64_t X, int64_t X0, int64_t s1, int64_t s0) { return (X / X0 - 1) * s1 + (X0 - 1) * s0; }

// A wave's tile, the waves that split the k of one (1: none), two levels of k.
struct FragTile {
  int ib, jb, kw;
  bool two;
};

// The product with n as the index along which C is contiguous, if any, and its
// k levels in the order the kernel takes; false: not one for the kernel.
bool frag_gemm_plan(const GemmDesc& g, FragGemm& d, FragTile& tile) {
  if (g.gk_start || g.ncs || g.nseg || g.comb_n || g.M % g.M0 || g.N % g.N0 || g.K % g.K0) return false;
  struct Level {
    int64_t n, a, b;
  } in{g.K0, g.sAk0, g.sBk0}, out{g.K / g.K0, g.sAk1, g.sBk1};
  if (in.n == 1) std::swap(in, out);
  if (out.n == 1) out.a = out.b = 0;
  if (in.n == 1) in.a = in.b = 0;
  if (out.n > 1 && out.a == in.n * in.a && out.b == in.n * in.b) {
    in.n *= out.n;
    out = Level{1, 0, 0};
  }
  // fewer padded steps with the other level inside
  if (out.n > 1 && in.n * ((out.n + 3) / 4) < out.n * ((in.n + 3) / 4)) std::swap(in, out);
  const bool two = tile.two = out.n > 1;
  d.K0 = (int)in.n;
  d.steps = two ? (int)(out.n * ((in.n + 3) / 4)) : (int)(in.n / 4);
  const int64_t spanA = reach(g.M, g.M0, g.M0 == g.M ? 0 : g.sAm1, g.M0 == 1 ? 0 : g.sAm0) + (out.n - 1) * out.a + (in.n - 1) * in.a + 1;
  const int64_t spanB = reach(g.N, g.N0, g.N0 == g.N ? 0 : g.sBn1, g.N0 == 1 ? 0 : g.sBn0) + (out.n - 1) * out.b + (in.n - 1) * in.b + 1;
  // offsets are formed in 32 bits, for k up to eight past the last
  if (spanA + 8 * in.a >= (1LL << 27) || spanB + 8 * in.b >= (1LL << 27)) return false;
  if (in.a < 0 || in.b < 0 || out.a < 0 || out.b < 0 || spanA < 1 || spanB < 1) return false;
  d.sak1 = (int)(out.a * sizeof(cplx));
  d.sak0 = (int)(in.a * sizeof(cplx));
  d.sbk1 = (int)(out.b * sizeof(cplx));
  d.sbk0 = (int)(in.b * sizeof(cplx));
  d.A = g.A;
  d.B = g.B;
  d.C = g.C;
  d.M = g.M;
  d.N = g.N;
  d.M0 = g.M0;
  d.N0 = g.N0;
  d.sAm1 = g.sAm1, d.sAm0 = g.sAm0, d.sAb = g.sAb;
  d.sBn1 = g.sBn1, d.sBn0 = g.sBn0, d.sBb = g.sBb;
  d.sCm1 = g.sCm1, d.sCm0 = g.sCm0, d.sCn1 = g.sCn1, d.sCn0 = g.sCn0, d.sCb = g.sCb;
  d.bl = g.bl;
  std::copy(g.cA, g.cA + 4, d.cA);
  std::copy(g.cB, g.cB + 4, d.cB);
  std::copy(g.cC, g.cC + 4, d.cC);
  d.nA = spanA;
  d.nB = spanB;
  d.are = g.alpha.re;
  d.aim = g.alpha.im;
  if (g.sCm0 == 1 && g.sCn0 != 1 && g.M0 > 1) {  // C^T = B^T A^T
    std::swap(d.A, d.B);
    std::swap(d.M, d.N);
    std::swap(d.M0, d.N0);
    std::swap(d.sAm1, d.sBn1);
    std::swap(d.sAm0, d.sBn0);
    std::swap(d.sAb, d.sBb);
    std::swap(d.sCm1, d.sCn1);
    std::swap(d.sCm0, d.sCn0);
    std::swap(d.cA, d.cB);
    std::swap(d.nA, d.nB);
    std::swap(d.sak1, d.sbk1);
    std::swap(d.sak0, d.sbk0);
  }
  // rows whose outer level is contiguous in A: numbered the other way round, so
  // that a fragment reads whole lines (of C, the columns are)
  if (d.M0 > 1 && d.M0 < d.M && d.sAm1 == 1 && d.sAm0 != 1 && d.sak0 != (int)sizeof(cplx)) {
    d.M0 = d.M / d.M0;
    std::swap(d.sAm1, d.sAm0);
    std::swap(d.sCm1, d.sCm0);
  }
  // Tiles of four 16 x 16 blocks a wave in the shape with the least padding
  // where they fill the chip's 2048 such waves, then (a long enough k) as
  // workgroups of four waves that split it; else one block and as many waves
  // for its k as that takes.
  auto up = [](int64_t x, int64_t y) { return (x + y - 1) / y; };
  const int64_t mb = up(d.M, 16), nb = up(d.N, 16);
  const int64_t p22 = up(mb, 2) * up(nb, 2), p14 = mb * up(nb, 4), p41 = up(mb, 4) * nb;
  const int64_t wide = std::min(p22, std::min(p14, p41));
  if (wide * g.batch >= 2048 || (wide * g.batch >= 64 && wide * g.batch * d.steps >= 16384)) {
    tile.kw = wide * g.batch >= 2048 ? 1 : 4;
    tile.ib = wide == p22 ? 2 : wide == p14 ? 1 : 4;
    tile.jb = 4 / tile.ib;
  } else {
    const int64_t w = mb * nb * g.batch;
    tile.kw = w * 4 >= 2048 || d.steps < 16 ? 4 : w * 8 >= 2048 || d.steps < 32 ? 8 : 16;
    tile.ib = tile.jb = 1;
  }
  d.mt = (int)up(mb, tile.ib);
  d.nt = (int)up(nb, tile.jb);
  d.wm = tile.kw > 1 || d.mt == 1 ? 1 : d.nt == 1 ? 4 : 2;
  d.wn = tile.kw > 1 ? 1 : 4 / d.wm;
  d.gm = (int)up(d.mt, d.wm);
  d.gn = (int)up(d.nt, d.wn);
  d.mfast = d.gm <= d.gn;
  d.per = Divisor((int64_t)d.gm * d.gn);
  d.fast = Divisor(d.mfast ? d.gm : d.gn);
  d.dM0 = Divisor(d.M0);
  d.dN0 = Divisor(d.N0);
  d.drun = Divisor((d.K0 + 3) / 4);
  return true;
}

}  // namespace

bool frag_gemm_fits(const GemmDesc& g) {
  FragGemm d;
  FragTile t;
  return frag_gemm_plan(g, d, t);
}

// The split of k with the least time by a simple account: rounds of workgroups
// on the chip, each its steps at the matrix cores' rate and 2 us to begin and
// end, and the atomic adds of a split product at 1 TB/s.
int frag_gemm_split(const GemmDesc& g) {
  FragGemm d;
  FragTile t;
  if (!frag_gemm_plan(g, d, t) || g.store) return 1;
  const int blocks = t.ib * t.jb, waves = t.kw == 1 ? 4 : t.kw;
  const int per_cu = blocks > 1 ? 2 : std::max(1, 20 / waves);
  const double step = blocks * 192 / 2400.0 * std::max(1.0, per_cu * waves / 4.0);  // us, a wave's
  const double wgs = (double)d.gm * d.gn * g.batch;
  int best = 1;
  double tbest = 0;
  for (int ks = 1; ks <= 16 && d.steps >= 8 * ks * t.kw / (t.kw == 1 ? 1 : 2); ++ks) {
    const double x = std::ceil(wgs * ks / (256.0 * per_cu)) * (std::ceil((double)d.steps / (ks * t.kw)) * step + 2.0) +
                     (ks > 1 ? (double)d.M * d.N * g.batch * ks * sizeof(cplx) / 1e6 : 0.0);
    if (ks == 1 || x < 0.9 * tbest) {
      best = ks;
      tbest = x;
    }
  }
  return best;
}

void frag_gemm(const GemmDesc& g, int ksplit, hipStream_t s) {
  FragGemm d;
  FragTile t;
  RTCC3_CHECK(frag_gemm_plan(g, d, t), "frag: bad product");
  d.ksplit = ksplit;
  d.split = Divisor(ksplit);
  d.mode = g.atomic || g.shared || ksplit > 1 ? 2 : g.store ? 1 : 0;
  if (t.ib == 2)
    t.kw == 1 ? launch_frag_gemm<2, 2, 1>(d, g.batch, t.two, s) : launch_frag_gemm<2, 2, 4>(d, g.batch, t.two, s);
  else if (t.jb == 4)
    t.kw == 1 ? launch_frag_gemm<1, 4, 1>(d, g.batch, t.two, s) : launch_frag_gemm<1, 4, 4>(d, g.batch, t.two, s);
  else if (t.ib == 4)
    t.kw == 1 ? launch_frag_gemm<4, 1, 1>(d, g.batch, t.two, s) : launch_frag_gemm<4, 1, 4>(d, g.batch, t.two, s);
  else if (t.kw == 4)
    launch_frag_gemm<1, 1, 4>(d, g.batch, t.two, s);
  else if (t.kw == 8)
    launch_frag_gemm<1, 1, 8>(d, g.batch, t.two, s);
  else
    launch_frag_gemm<1, 1, 16>(d, g.batch, t.two, s);
}

bool frag_gemm_small(const GemmDesc& g) {
  FragGemm d;
  FragTile t;
  // (with the eight waves that a group gives to each)
  return frag_gemm_plan(g, d, t) && t.ib * t.jb == 1 && d.steps <= 512 && (int64_t)d.gm * d.gn * g.batch < (1 << 20);
}

void frag_gemm_group(const GemmDesc* g, int n, hipStream_t s) {
  for (int i0 = 0; i0 < n; i0 += kGroup) {
    FragGroup d;
    d.n = std::min(kGroup, n - i0);
    int wg = 0;
    for (int i = 0; i < d.n; ++i) {
      FragTile t;
      const GemmDesc& q = g[i0 + i];
      RTCC3_CHECK(frag_gemm_plan(q, d.g[i], t) && t.ib * t.jb == 1, "frag: not a small product");
      d.g[i].ksplit = 1;
      d.g[i].split = Divisor(1);
      d.g[i].mode = q.atomic || q.shared ? 2 : q.store ? 1 : 0;
      d.tail[i] = !t.two ? -1 : (d.g[i].K0 & 3) != 0;
      wg += d.g[i].gm * d.g[i].gn * q.batch;
      d.end[i] = wg;
    }
    hipLaunchKernelGGL(frag_group_kernel, dim3((unsigned)wg), dim3(512), 0, s, d);
    RTCC3_HIP(hipGetLastError());
  }
}

int64_t frag_cols_pack(const int* rows, int njob, int o, int v) {
  int64_t nrb = 0;
  for (int j = 0; j < njob; ++j) nrb += (rows[j] + 15) / 16;
  return o * nrb * (((int64_t)v * v + 3) / 4) * 64;
}

int frag_cols(const ColsJob* jobs, int njob, const cplx* B, const int* perm, int nstream, int v, int vp,
               const int* part, const int* bl, const int* frags, int nfrag, int o, cplx* pack, hipStream_t s) {
  if (nfrag <= 0 || njob <= 0) return 0;
  RTCC3_CHECK(njob <= 2 && (nstream == 1 || nstream == 3) && v >= 1 && vp >= v, "frag: bad column product");
  RTCC3_CHECK((int64_t)v * v * vp < (1LL << 27), "frag: product too large");
  FragCols d;
  d.B = B;
  d.bl = bl;
  d.part = part;
  d.frag = reinterpret_cast<const int4*>(frags);
  for (int w = 0; w < 3; ++w) d.perm[w] = w < nstream ? perm[w] : 0;
  d.v = v;
  d.vp = vp;
  d.nfrag = nfrag;
  d.steps = v * v / 4;
  struct RowBlock {
    int job, row;
  };
  std::vector<RowBlock> rb;
  for (int j = 0; j < njob; ++j) {
    RTCC3_CHECK(jobs[j].M >= 1, "frag: bad column operand");
    d.job[j] = jobs[j];
    for (int m = 0; m < jobs[j].M; m += 16) rb.push_back({j, m});
  }
  ColsPack pk;
  for (int j = 0; j < 2; ++j) {
    pk.job[j] = jobs[std::min(j, njob - 1)];
    pk.nrb[j] = j < njob ? (jobs[j].M + 15) / 16 : 0;
  }
  pk.njob = njob;
  pk.n = o;
  pk.steps = (v * v + 3) / 4;
  pk.v2 = (int64_t)v * v;
  pk.dst = pack;
  RTCC3_CHECK((int64_t)pk.steps * 64 < (1LL << 27), "frag: product too large");
  const int64_t packed = (int64_t)o * (int64_t)rb.size() * pk.steps * 64;
  hipLaunchKernelGGL(cols_pack_kernel, dim3((unsigned)std::min<int64_t>((packed + 255) / 256, 65536)), dim3(256), 0, s,
                     pk);
  RTCC3_HIP(hipGetLastError());
  int launches = 1;
  d.pack = pack;
  d.npanel = (int)rb.size();
  // Row blocks in groups as large as the registers allow (the sums of a B
  // fragment and, with three streams, its combination serve all of a group's
  // rows), of about the same size.  Five blocks in one group where four would
  // make two: X2 at o=16, v=66 26.2 -> 11.8 ms.
  const int most = 5;
  const int ng = ((int)rb.size() + most - 1) / most;
  auto launch = [&]() {
    // Splits of k for at least four rounds of the chip's 2048 waves, of 32 steps
    // or more; and of 256 to 511 steps, at whose ends the waves that share blocks
    // meet again (X2 at o=16, v=66 12.4 -> 11.0 ms, o=15, v=57 5.46 -> 5.28; of 33
    // steps at o=10, v=38 0.43 -> 0.53).
    const int64_t waves = (int64_t)nfrag * d.nunit;
    d.nsplit = (int)std::max<int64_t>(1, std::max<int64_t>(std::min<int64_t>((4 * 2048 + waves - 1) / waves, d.steps / 32),
                                                           d.steps / 256));
    const int64_t nw = waves * d.nsplit;
    RTCC3_CHECK(nw < (1LL << 31), "frag: product too large");
    const dim3 grid((unsigned)((nw + 3) / 4));
    if (nstream == 1)
      hipLaunchKernelGGL(frag_cols_kernel<1>, grid, dim3(256), 0, s, d);
    else
      hipLaunchKernelGGL(frag_cols_kernel<3>, grid, dim3(256), 0, s, d);
    RTCC3_HIP(hipGetLastError());
    ++launches;
    d.nunit = 0;
  };
  d.nunit = 0;
  for (int g = 0; g < ng; ++g) {
    const int r0 = (int)(rb.size() * g / ng), r1 = (int)(rb.size() * (g + 1) / ng);
    ColsUnit& u = d.unit[d.nunit++];
    u.nb = r1 - r0;
    for (int q = 0; q < 5; ++q) {
      u.job[q] = rb[std::min(r0 + q, r1 - 1)].job;
      u.row[q] = rb[std::min(r0 + q, r1 - 1)].row;
      u.panel[q] = std::min(r0 + q, r1 - 1);
    }
    if (d.nunit == kMaxColsUnits) launch();
  }
  if (d.nunit > 0) launch();
  return launches;
}

int frag_gather(const FragJob* jobs, int njob, const cplx* B, int v, int vp, const int* bl, int nblk, int group,
                hipStream_t s) {
  if (nblk <= 0 || njob <= 0) return 0;
  RTCC3_CHECK(njob <= 2 && v >= 1 && vp >= v && group >= 1, "frag: bad gathered product");
  RTCC3_CHECK((int64_t)v * v * vp < (1LL << 27) && (int64_t)v * v < (1 << 22), "frag: product too large");
  FragGather d;
  d.B = B;
  d.bl = bl;
  d.v = v;
  d.vp = vp;
  d.nblk = nblk;
  d.ncol = (v * v + 63) / 64;
  d.nunit = 0;
  struct RowBlock {
    int job, row;
  };
  std::vector<RowBlock> rb;
  for (int j = 0; j < njob; ++j) {
    RTCC3_CHECK(jobs[j].M >= 1 && jobs[j].lA >= (int64_t)(jobs[j].M - 1) * jobs[j].sAm + v && jobs[j].lA + 4 < (1LL << 27),
                "frag: gathered operand too large");
    d.job[j] = jobs[j];
    for (int m = 0; m < jobs[j].M; m += 16) rb.push_back({j, m});
  }
  int launches = 0;
  auto launch = [&]() {
    // Chunks of whole groups (stretches with one output of a job: fewer flushes)
    // for at least eight rounds of the chip's 2048 waves; below one group a
    // chunk, shorter ones down to two rounds (Z_i and Y2 at o=10, v=38: chunks of
    // 1, 5 and 11 blocks took 1.5, 0.50 and 0.48 ms).
    const int64_t waves = (int64_t)nblk * d.ncol * d.nunit;
    const int64_t c = waves / (8 * 2048) / group;
    d.chunk = (int)(c >= 1 ? c * group : std::max<int64_t>(1, std::min<int64_t>(group, waves / (2 * 2048))));
    const int64_t nw = (int64_t)((nblk + d.chunk - 1) / d.chunk) * d.ncol * d.nunit;
    RTCC3_CHECK(nw < (1LL << 31), "frag: product too large");
    hipLaunchKernelGGL(frag_gather_kernel, dim3((unsigned)((nw + 3) / 4)), dim3(256), 0, s, d);
    RTCC3_HIP(hipGetLastError());
    ++launches;
    d.nunit = 0;
  };
  for (size_t q = 0; q < rb.size();) {
    const bool pair = q + 1 < rb.size();
    for (int h = 0; h < (pair ? 2 : 1); ++h) {
      FragUnit& u = d.unit[d.nunit++];
      u.job[0] = rb[q].job;
      u.row[0] = rb[q].row;
      u.job[1] = pair ? rb[q + 1].job : rb[q].job;
      u.row[1] = pair ? rb[q + 1].row : rb[q].row;
      u.single = !pair;
      u.half = h;
    }
    q += pair ? 2 : 1;
    if (d.nunit + 2 > kMaxUnits) launch();
  }
  if (d.nunit > 0) launch();
  return launches;
}

int frag_seg(const GemmDesc& g, const int* row_tiles, int nrt, hipStream_t s) {
  if (nrt <= 0) return 0;
  RTCC3_CHECK(g.nseg >= 1 && g.nseg <= 4 && g.bl && row_tiles && g.M0 == g.M && g.sCn0 == 1 && g.alpha.re == 1.0 &&
                  g.alpha.im == 0.0 && (g.store != 0) != (g.atomic != 0) && g.cC[0] == 0 && g.cC[1] == 0 &&
                  g.cC[2] == 0 && g.sCm0 == (int64_t)(g.N / g.N0) * g.sCn1 && g.N == g.M * g.N0 && g.N0 == g.M,
              "frag: bad segmented product");
  FragSeg d;
  d.nseg = g.nseg;
  for (int t = 0; t < g.nseg; ++t) {
    d.seg[t] = g.seg[t];
    RTCC3_CHECK(g.seg[t].sBn == 1 && g.seg[t].cA[3] == 0 && g.seg[t].cB[3] == 0 && g.seg[t].len >= 1 &&
                    (int64_t)g.seg[t].len * g.seg[t].sBk + g.N < (1LL << 27) &&
                    (int64_t)g.M * g.seg[t].sAm + (int64_t)g.seg[t].len * g.seg[t].sAk < (1LL << 27),
                "frag: bad segment");
  }
  d.v = g.M;
  d.N = g.N;
  d.vp = (int)g.sCn1;
  d.C = g.C;
  d.vb = g.cC[3];
  d.bl = g.bl;
  d.rt = reinterpret_cast<const int4*>(row_tiles);
  d.ncol = (g.N + 63) / 64;
  RTCC3_CHECK((int64_t)kFragRun * g.M < (1 << 22) && g.N < (1 << 22) && (int64_t)nrt * d.ncol < (1LL << 31),
              "frag: product too large");
  const dim3 grid((unsigned)(nrt * d.ncol));
  if (g.atomic)
    hipLaunchKernelGGL(frag_seg_kernel<true>, grid, dim3(256), 0, s, d);
  else
    hipLaunchKernelGGL(frag_seg_kernel<false>, grid, dim3(256), 0, s, d);
  RTCC3_HIP(hipGetLastError());
  return 1;
}

}  // namespace rtcc3
