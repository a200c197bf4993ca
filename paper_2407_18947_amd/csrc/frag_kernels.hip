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
  __device__ __forceinline__ void clear() {
#pragma unroll
    for (int i = 0; i < IB; ++i)
#pragma unroll
      for (int j = 0; j < JB; ++j) p1[i][j] = p2[i][j] = p3[i][j] = d4{0, 0, 0, 0};
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
// k = l/16) into ra, rb; sak, sbk bytes per k.  Two register sets alternate as
// the step in flight.  A last partial step of four reads its missing k at the
// last valid one and multiplies by a zero A.
template <int IB, int JB>
__device__ __forceinline__ void contract(Acc<IB, JB>& acc, __amdgpu_buffer_rsrc_t ra, const int* ao, int sak,
                                         __amdgpu_buffer_rsrc_t rb, const int* bo, int sbk, int len, int kl) {
  d2v a0[IB], b0[JB], a1[IB], b1[JB];
  int sa = 0, sb = 0;
  auto load = [&](d2v* a, d2v* b) {
#pragma unroll
    for (int i = 0; i < IB; ++i) a[i] = frag_load(ra, ao[i], sa);
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
      const d2v z = frag_load(ra, ao[i] + back * sak, sa);
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

// The builds of t3 and lambda3 (o=15, v=57: t3 7.7 -> 5.6 ms, lambda3 12.5 ->
// 9.8 ms a launch, alone; 0.77 -> 0.36 ms for t3 at o=10, v=38, where an
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
  __shared__ unsigned ebase[kFragRun];  // first element of the entry's block in C
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
    ebase[tid] = (unsigned)(e0[4 * tid + 3] * d.vb);
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
    const auto ra = rsrc(g.A + g.cA[0] * I0 + g.cA[1] * J0 + g.cA[2] * K0, (1 << 27) - 1);
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
        const unsigned el = ebase[e] + off;
#pragma unroll
        for (int j = 0; j < JB; ++j)
          if (cok[j]) {
            const d2v z = acc.value(i, j, r);
            cplx* p = d.C + (uint64_t)(el + co[j]);
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

}  // namespace

void frag_seg(const GemmDesc& g, const int* row_tiles, int nrt, hipStream_t s) {
  if (nrt <= 0) return;
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
}

}  // namespace rtcc3
