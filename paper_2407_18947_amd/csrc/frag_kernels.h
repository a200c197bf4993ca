// FP64 products whose MFMA fragments are loaded straight from memory
// (frag_kernels.hip).
#pragma once

#include "common.h"

namespace rtcc3 {

// Row tiles of a segmented product over a block table sorted so that the
// entries of a run share their B operands (4 ints per tile: the run's first
// entry, its entries, the index of its first tile, its tiles).  The rows of a
// run's entries are numbered through, kFragRows of them per tile.
constexpr int kFragRows = 64;
constexpr int kFragRun = 64;  // most entries of a run

// The products over blocks below return the number of kernels they launched.

// The FP64 form of a segmented product (GemmDesc::seg, alpha = 1), plain store
// or atomic accumulation, with C contiguous rows of N0 elements at stride sCn1.
int frag_seg(const GemmDesc& g, const int* row_tiles, int nrt, hipStream_t s);

// Products that read the blocks of a window as rows c of v^2 columns and sum
// over c and over blocks,
//   C_j[m][n] += alpha_j * sum_blocks sum_c A_j[m][c] B[block][c][n],   n = (p, q) < v^2,
// A_j at A + cA.(I,J,K) + m*sAm + c, B at B + slot*vb + c*v*vp + p*vp + q and
// C_j at C + cC.(I,J,K) + m*sCm + n.  Every job reads the same blocks once.
struct FragJob {
  const cplx* A;
  int64_t cA[3], sAm;
  int64_t lA;  // elements of one block's A operand, (M - 1)*sAm + v
  int M;
  cplx* C;
  int64_t cC[3], sCm;
  double alpha;
};
// bl: nblk block table entries (I, J, K, slot), in an order that keeps each
// job's output in place over long stretches; group: the usual length of the
// shortest such stretches.
int frag_gather(const FragJob* jobs, int njob, const cplx* B, int v, int vp, const int* bl, int nblk, int group,
                hipStream_t s);

// Products that read the blocks of a window as rows k < v^2 of v columns b, and
// whose other operand depends on the block table's K only,
//   C_j[I][J][m][b] += sum_K sum_k A_j[K][m][k] Z[IJK][k][b],
// Z one block, or 2 X0 - X1 - X2 of three (nstream = 3), the blocks at slots
// part[6 n + perm[w]] of entry n's orderings.  A_j at A + K*cAK + m*sAm + k, C_j
// at C + cC.(I,J) + m*sCm + b*sCb (atomic adds).  The columns of all entries of a
// K are numbered through and cut into fragments of up to 16 (4 ints each: the
// first column's entry in bl and its b, the number of columns, 0) whose
// entries share K and whose blocks lie within 2^31 bytes of each other.
struct ColsJob {
  const cplx* A;
  int64_t cAK, sAm;
  int M;
  cplx* C;
  int64_t cC[2], sCm, sCb;
};
// pack: space for frag_cols_pack() elements, used on s only until the product is
// done; o: the extent of K.
int frag_cols(const ColsJob* jobs, int njob, const cplx* B, const int* perm, int nstream, int v, int vp,
               const int* part, const int* bl, const int* frags, int nfrag, int o, cplx* pack, hipStream_t s);
int64_t frag_cols_pack(const int* rows, int njob, int o, int v);

// Products of one block each, X[b][k] read as rows k < v^2 of v columns b (the
// block at slot part[6 n + perm] of entry n), with the n columns of several
// groups,
//   C_g[b][x] += alpha_g * sum_k X[k][b] B_g[x][k],   x < n,
// B_g at B + (I, J or K, by key)*sKey + x*sB + k, C_g at C + cC.(I,J,K) + b*sCm +
// x*sCx (atomic adds).  A trace takes the column x = (I, J or K, by col) of a
// group once more, times its own alpha, into C + (I, J or K, by row)*sC + b.
struct BlockCols {
  const cplx* B;
  int key;
  int64_t sKey, sB;
  cplx* C;
  int64_t cC[3], sCm, sCx;
  double alpha;
};
struct BlockTrace {
  int group, col, row;
  cplx* C;
  int64_t sC;
  double alpha;
};
constexpr int kMaxBlockCols = 4;
// pack: space for frag_block_pack() elements, used on s only until the product
// is done; o: the extent of I, J and K; reach: the most bytes from the first to
// past the last panel of the groups that one launch takes (32-bit offsets).
int frag_block(const BlockCols* groups, int ng, int n, const BlockTrace* tr, int ntr, const cplx* X, int perm, int o,
               int v, int vp, const int* part, const int* bl, int nblk, cplx* pack, hipStream_t s,
               int64_t reach = (int64_t)1 << 32);
int64_t frag_block_pack(const BlockCols* groups, int ng, int n, int o, int v);

// A plain FP64 product (no segments, gathered K or combined operands) with its
// k split over ksplit workgroups (atomic adds if more than one);
// frag_gemm_fits: whether the kernel takes it (32-bit operand spans),
// frag_gemm_split: the split to use where none was measured.
bool frag_gemm_fits(const GemmDesc& g);
int frag_gemm_split(const GemmDesc& g);
void frag_gemm(const GemmDesc& g, int ksplit, hipStream_t s);
// Products of one 16 x 16 block a workgroup (frag_gemm_small), k not split over
// workgroups, that do not depend on each other, in launches of up to eight.
bool frag_gemm_small(const GemmDesc& g);
void frag_gemm_group(const GemmDesc* g, int n, hipStream_t s);

}  // namespace rtcc3
