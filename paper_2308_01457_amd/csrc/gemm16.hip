// Complex64 products on the fp16 matrix cores:  C = beta C + alpha A B.
//
// Every FP32 operand x, scaled by powers of two, is the sum of two fp16 numbers:
// h = fp16(x), l = fp16(x - h).  h and l carry 11 bits each, so h + l differs
// from x by at most 2^-22 |x| (entries 2^-13 below their row's largest and
// smaller: by 2^-25 in scaled units, 2^-35 of that largest entry).  Exact
// scalings keep the entries in the short range of fp16: A's column k is
// multiplied by 2^e_k, which brings its largest entry to [1, 2), and B's row k by
// 2^-e_k, so that an entry of B weighs as the largest term it enters (a matrix
// whose unknowns have different units is graded along k); then each row of A and
// column of B is brought to a largest entry in [2^10, 2^11).  The scaling along k
// comes from A alone: one from B too would let a large column of B take the
// bits of the others.  In L D L^T both operands are scaled by the half exponent of
// d_k instead.  A real product is then the sum of three fp16 products, l h, h l
// and h h, accumulated in FP32 by v_mfma_f32_32x32x16_f16; the complex product
// takes three real ones (3M, as in gemm.hip), whose operand sums re + im are
// formed in FP32 before they are split.  (Splitting into two half-precision parts:
// Markidis et al., IPDPSW 2018; Ootomo and Yokota, IJHPCA 36, 2022.)
//
// The error of an entry of column j is thus below about K 2^-22 times the
// largest term |a_ik b_kj| of that column over all rows i: normwise by column,
// not entry by entry as with FP32 products, where a row of A with small entries
// against large ones of other rows keeps its own relative accuracy.
//
// Error: one rounding per 16 of K replaces one per entry of K, which more than
// makes up for the two missing bits of the operands.  Against 64 bits on normal
// random operands the Frobenius error is 0.67 (K = 256), 0.63 (768) and 0.61
// (4096) of the FP32 matrix instruction's (4.0e-7, 7.0e-7, 1.6e-6).
//
// Operands are packed once per product into the order in which the kernel reads
// them: [32-row block][16-deep k block][plane][lane][8 fp16], planes h and l of
// re, im and re + im, 1 KB per plane, rows and k padded with zeros.  A wavefront
// copies 1 KB straight into LDS per instruction, reads fragments without bank
// conflicts, and no load needs an edge check.
#include <algorithm>

#include "common.h"

namespace fosb {

typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef float f16v __attribute__((ext_vector_type(16)));
typedef __attribute__((address_space(3))) void* lds_ptr;
typedef const __attribute__((address_space(1))) void* glb_ptr;

constexpr int kPlanes = 6;               // h, l of re, im, re + im
constexpr int kChunk = 64;               // h8 values per plane of a block (one per lane)
constexpr int kTileM = 256, kTileN = 128;
constexpr int kTargetExp = 10;           // scaled row and column maxima lie in [2^10, 2^11)

// An operand in memory: element (r, k) at p[r * rs + k * ks], conjugated if conj.
struct SplitSrc {
  const c64* p;
  int64_t rs, ks;
  int conj;
};

// Exponents of magnitudes: floor(log2 max(|re|, |im|)), denormals included; below
// kLowExp for zero, above kHighExp for infinities and NaN, also after a scaling.
constexpr int kZeroExp = -(1 << 23), kLowExp = -(1 << 19);
constexpr int kInfExp = 1 << 23, kHighExp = 1 << 19;
// Scaling along K of a term that adds nothing (A's column is all zero): B's
// entries there count nothing (a large one would take the bits of its column's
// others) and are scaled to zero, unless they are not finite.
constexpr int kNoTerm = 1 << 21;

__device__ __forceinline__ int mag_exp(c64 v) {
  const unsigned m = max(__float_as_uint(v.re) & 0x7fffffffu, __float_as_uint(v.im) & 0x7fffffffu);
  const int e = __builtin_amdgcn_frexp_expf(__uint_as_float(m)) - 1;
  return m == 0u ? kZeroExp : m >= 0x7f800000u ? kInfExp : e;
}

// ke or, with flip = -1, -ke
__device__ __forceinline__ int turned(int ke, int flip) { return (ke ^ flip) - flip; }

__device__ __forceinline__ int wave_max_i32(int m) {
  for (int o = 32; o > 0; o >>= 1) m = max(m, __shfl_xor(m, o, 64));
  return m;
}

// Largest exponent along r for each k: workgroup (x, y) takes 64 k and 512 r;
// the maximum is independent of order.
__global__ __launch_bounds__(256) void k_split_kmax(SplitSrc s, int64_t R, int64_t K, int* __restrict__ mx) {
  __shared__ int red[4][64];
  const int64_t k0 = (int64_t)blockIdx.x * 64, r0 = (int64_t)blockIdx.y * 512, r1 = min(R, r0 + 512);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (s.ks == 1) {   // neighbouring lanes along k
    int m = kZeroExp;
    if (k0 + lane < K)
      for (int64_t r = r0 + wave; r < r1; r += 4) m = max(m, mag_exp(s.p[r * s.rs + k0 + lane]));
    red[wave][lane] = m;
    __syncthreads();
    if (wave == 0 && k0 + lane < K)
      atomicMax(mx + k0 + lane, max(max(m, red[1][lane]), max(red[2][lane], red[3][lane])));
    return;
  }
  for (int q = wave; q < 64; q += 4) {   // neighbouring lanes along r
    const int64_t k = k0 + q;
    if (k >= K) break;
    int m = kZeroExp;
    for (int64_t r = r0 + lane; r < r1; r += 64) m = max(m, mag_exp(s.p[r * s.rs + k * s.ks]));
    m = wave_max_i32(m);
    if (lane == 0) atomicMax(mx + k, m);
  }
}

// e_k from the largest exponent of A's column k: brings it to 0; 0 where the
// column is not finite.
__global__ void k_split_kexp(const int* __restrict__ ma, int64_t K, int* __restrict__ ke) {
  const int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (k >= K) return;
  ke[k] = ma[k] < kLowExp ? kNoTerm : ma[k] > kHighExp ? 0 : -ma[k];
}

// e_k for L times D L^T, D on a matrix's diagonal: half the exponent of d_k.
__global__ void k_split_kexp_diag(const c64* __restrict__ A, int64_t lda, int64_t K, int* __restrict__ ke) {
  const int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (k >= K) return;
  const int e = mag_exp(A[k * lda + k]);
  ke[k] = (e < kLowExp || e > kHighExp) ? 0 : e >> 1;
}

// Largest exponent of each row, scaled along K by 2^e_k (2^-e_k with flip = -1):
// workgroup (x, y) takes 32 rows and 512 of K.
__global__ __launch_bounds__(256) void k_split_max(SplitSrc s, int64_t R, int64_t K, const int* __restrict__ ke,
                                                   int flip, int* __restrict__ mx) {
  __shared__ int red[8][32];
  const int64_t r0 = (int64_t)blockIdx.x * 32, k0 = (int64_t)blockIdx.y * 512;
  if (s.ks == 1) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int q = wave; q < 32; q += 4) {
      const int64_t r = r0 + q;
      int m = kZeroExp;
      if (r < R)
        for (int64_t k = k0 + lane; k < min(K, k0 + 512); k += 64)
          m = max(m, mag_exp(s.p[r * s.rs + k]) + turned(ke[k], flip));
      m = wave_max_i32(m);
      if (lane == 0 && r < R) atomicMax(mx + r, m);
    }
    return;
  }
  const int c = threadIdx.x & 31, g = threadIdx.x >> 5;
  const int64_t r = r0 + c;
  int m = kZeroExp;
  if (r < R)
    for (int64_t k = k0 + g; k < min(K, k0 + 512); k += 8)
      m = max(m, mag_exp(s.p[r * s.rs + k * s.ks]) + turned(ke[k], flip));
  red[g][c] = m;
  __syncthreads();
  if (g == 0 && r < R) {
    int b = red[0][c];
    for (int q = 1; q < 8; ++q) b = max(b, red[q][c]);
    atomicMax(mx + r, b);
  }
}

// Power of two that scales a row with the largest exponent m; the entries of a
// zero or a not finite row stay as they are.
__device__ __forceinline__ int split_exp(int m) {
  return (m < kLowExp || m > kHighExp) ? 0 : kTargetExp - m;
}

__device__ __forceinline__ void split2(float x, _Float16& h, _Float16& l) {
  h = (_Float16)x;
  l = (_Float16)(x - (float)h);
}

// Packs rows [32 blk, 32 blk + 32) of the k blocks of this workgroup.  Lane l
// holds row l % 32 and k = 8 (l / 32) .. + 7 of a block (the operand layout of
// the 32x32x16 instruction, the same for A's rows and B's columns).  Rows that
// are contiguous along k are read 64 B per lane; columns of a row-major matrix
// 256 B per k.
__global__ __launch_bounds__(256) void k_split_pack(SplitSrc s, int64_t R, int64_t K, int64_t nkb,
                                                    const int* __restrict__ ke, int flip,
                                                    const int* __restrict__ mx, h8* __restrict__ P) {
  const int64_t blk = blockIdx.y, kb = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (kb >= nkb) return;
  const int lane = threadIdx.x & 63;
  const int64_t row = blk * 32 + (lane & 31), k0 = kb * 16 + (lane >> 5) * 8;
  const int e = row < R ? split_exp(mx[row]) : 0;
  h8 o[kPlanes];
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    c64 v{0.f, 0.f};
    int eq = e;
    if (row < R && k0 + q < K) {
      v = s.p[row * s.rs + (k0 + q) * s.ks];
      eq += turned(ke[k0 + q], flip);
    }
    const float re = ldexpf(v.re, eq), im = ldexpf(s.conj ? -v.im : v.im, eq);
    _Float16 h, l;
    split2(re, h, l);
    o[0][q] = h;
    o[1][q] = l;
    split2(im, h, l);
    o[2][q] = h;
    o[3][q] = l;
    split2(re + im, h, l);
    o[4][q] = h;
    o[5][q] = l;
  }
  h8* d = P + ((blk * nkb + kb) * kPlanes) * kChunk + lane;
#pragma unroll
  for (int p = 0; p < kPlanes; ++p) d[p * kChunk] = o[p];
}

__global__ void k_split_zero(int* p, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) p[i] = kZeroExp;
}

// One K block (16 deep) of a tile into LDS: 8 blocks of A, 4 of B, 6 planes
// each; 8 wavefronts move 9 chunks of 1 KB apiece.
__device__ __forceinline__ void stage_block(const h8* __restrict__ Ap, const h8* __restrict__ Bp, int64_t nkb,
                                            int64_t kb, h8* __restrict__ dst, int wave, int lane) {
#pragma unroll
  for (int q = 0; q < 12 * kPlanes / 8; ++q) {
    const int ch = q * 8 + wave, blk = ch / kPlanes, p = ch % kPlanes;
    const h8* src = blk < 8 ? Ap + ((int64_t)blk * nkb + kb) * (kPlanes * kChunk)
                            : Bp + ((int64_t)(blk - 8) * nkb + kb) * (kPlanes * kChunk);
    __builtin_amdgcn_global_load_lds((glb_ptr)(src + p * kChunk + lane), (lds_ptr)(dst + ch * kChunk), 16, 0, 0);
  }
}

// The wavefront's 64 x 64 part of a K block: per component (re, im, re + im)
// l h, then h l, then h h.
__device__ __forceinline__ void multiply_block(const h8* __restrict__ s, int wr, int wc, int lane,
                                               f16v (&t)[3][2][2]) {
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    h8 a[2][2], b[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int p = 0; p < 2; ++p) {
        a[i][p] = s[((wr * 2 + i) * kPlanes + c * 2 + p) * kChunk + lane];
        b[i][p] = s[((8 + wc * 2 + i) * kPlanes + c * 2 + p) * kChunk + lane];
      }
#pragma unroll
    for (int q = 0; q < 3; ++q)
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          t[c][i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[i][q == 0], b[j][q == 1], t[c][i][j], 0, 0, 0);
  }
}

// 256 x 128 tiles, 8 wavefronts of 64 x 64 (192 accumulator registers, two
// wavefronts per SIMD), two 72 KB buffers: the copies of K block b + 1 run
// during the products of block b.  One workgroup per compute unit walks its
// share of its XCD's tiles, in groups of four tile rows, so that the
// workgroups of one XCD share panels in its L2; the next tile's first K block
// is copied during the stores of the last one.  Each 32 x 32 part of C is
// loaded 16 rows at once (an element at a time, the tile's 64 dependent round
// trips cost as much as 24 K blocks: the factorisation at N = 30720 took 228
// instead of 197 ms without overlap).
// What bounds long products is the matrix rate the chip sustains: 8192 x 8192 x
// 4096 at 470 TFLOP/s counted as 8 MNK (18 MNK executed: 1.06 PFLOP/s), against
// 170 of the FP32 instruction; a 128 x 128 tile, whose panels are read twice as
// often, reached 320.  At K = 768 the round trip of C adds a quarter: 28672 x
// 2304 x 768 at 365 against 143.
// With diag_nb > 0 the tiles entirely above the diag_nb-wide diagonal blocks
// (rows and columns counted from the same origin) are left out.
__global__ __launch_bounds__(512, 2) void k_gemm_split(int64_t M, int64_t N, int64_t nkb, float alpha,
                                                       const h8* __restrict__ A, const int* __restrict__ ma,
                                                       const h8* __restrict__ B, const int* __restrict__ mb,
                                                       float beta, c64* __restrict__ C, int64_t ldc, int nM, int nN,
                                                       int diag_nb) {
  __shared__ __align__(16) h8 s0[12 * kPlanes * kChunk];
  __shared__ __align__(16) h8 s1[12 * kPlanes * kChunk];
  __shared__ int ex[kTileM + kTileN];   // exponents of the tile's rows and columns
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wr = wave >> 1, wc = wave & 1;
  const int ntile = nM * nN;
  const int x = blockIdx.x % 8, per = ntile / 8, count = per + (x < ntile % 8 ? 1 : 0);
  const int start = x * per + min(x, ntile % 8);
  int slot = blockIdx.x / 8, tm = 0, tn = 0;
  auto find = [&]() {   // the workgroup's next tile, from slot on; false when there is none
    for (; slot < count; slot += gridDim.x / 8) {
      const int tile = start + slot;
      const int group = tile / (4 * nN), fm = group * 4, gs = min(nM - fm, 4), in = tile - group * 4 * nN;
      tm = fm + in % gs;
      tn = in / gs;
      if (diag_nb <= 0 || (tm + 1) * kTileM > tn * kTileN / diag_nb * diag_nb) return true;
    }
    return false;
  };
  const h8 *Ap = A, *Bp = B;
  auto first = [&]() {   // start copying the tile's first K block
    Ap = A + (int64_t)tm * 8 * nkb * (kPlanes * kChunk);
    Bp = B + (int64_t)tn * 4 * nkb * (kPlanes * kChunk);
    stage_block(Ap, Bp, nkb, 0, s0, wave, lane);
  };
  bool more = find();
  if (more) first();
  while (more) {
    const int64_t m0 = (int64_t)tm * kTileM, n0 = (int64_t)tn * kTileN;
    if (threadIdx.x < kTileM)
      ex[threadIdx.x] = m0 + threadIdx.x < M ? split_exp(ma[m0 + threadIdx.x]) : 0;
    else if (threadIdx.x < kTileM + kTileN)
      ex[threadIdx.x] = n0 + threadIdx.x - kTileM < N ? split_exp(mb[n0 + threadIdx.x - kTileM]) : 0;
    f16v t[3][2][2] = {};
    __syncthreads();
    for (int64_t kb = 0; kb < nkb; kb += 2) {
      if (kb + 1 < nkb) stage_block(Ap, Bp, nkb, kb + 1, s1, wave, lane);
      multiply_block(s0, wr, wc, lane, t);
      __syncthreads();
      if (kb + 1 < nkb) {
        if (kb + 2 < nkb) stage_block(Ap, Bp, nkb, kb + 2, s0, wave, lane);
        multiply_block(s1, wr, wc, lane, t);
        __syncthreads();
      }
    }
    const bool interior = m0 + kTileM <= M && n0 + kTileN <= N;
    slot += gridDim.x / 8;
    more = find();
    if (more) first();   // in flight during the stores below
    const int lr = wr * 64 + (lane >> 5) * 4, lc = wc * 64 + (lane & 31);
    c64* Ct = C + (m0 + lr) * ldc + n0 + lc;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        // 16 rows at once: their loads are issued together
        c64 o[16];
        const int ec = ex[kTileM + lc + 32 * j];
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int dr = i * 32 + (v / 4) * 8 + v % 4;
          o[v] = c64{0.f, 0.f};
          if (beta != 0.f && (interior || (m0 + lr + dr < M && n0 + lc + 32 * j < N)))
            o[v] = Ct[(int64_t)dr * ldc + 32 * j];
        }
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int dr = i * 32 + (v / 4) * 8 + v % 4;
          const int e = -(ec + ex[lr + dr]);
          const float cr = ldexpf(t[0][i][j][v] - t[1][i][j][v], e);
          const float ci = ldexpf(t[2][i][j][v] - t[0][i][j][v] - t[1][i][j][v], e);
          if (interior || (m0 + lr + dr < M && n0 + lc + 32 * j < N))
            Ct[(int64_t)dr * ldc + 32 * j] = beta == 0.f ? c64{alpha * cr, alpha * ci}
                                                         : c64{beta * o[v].re + alpha * cr, beta * o[v].im + alpha * ci};
        }
      }
    __syncthreads();   // ex is read
  }
}

static SplitSrc source_a(const c64* A, int64_t lda, bool conj_trans) {
  return conj_trans ? SplitSrc{A, 1, lda, 1} : SplitSrc{A, lda, 1, 0};
}

static void zero_max(hipStream_t st, int* p, int64_t n) {
  hipLaunchKernelGGL(k_split_zero, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, p, n);
  FOSB_LAUNCH_CHECK();
}

// 32-row blocks of a packed A, one tile more than M needs (a product may start at
// any multiple of 32 rows), and of a packed B.
static int64_t blocks_a(int64_t M) { return ((M + kTileM - 1) / kTileM + 1) * (kTileM / 32); }
static int64_t blocks_b(int64_t N) { return (N + kTileN - 1) / kTileN * (kTileN / 32); }
static int64_t pack_bytes(int64_t nblk, int64_t K) {
  return nblk * ((K + 15) / 16) * kPlanes * kChunk * (int64_t)sizeof(h8);
}

PackBytes split_pack_bytes(int64_t M, int64_t N, int64_t K) {
  return PackBytes{pack_bytes(blocks_a(M), K), pack_bytes(blocks_b(N), K)};
}

bool split_reserve(Context& ctx, const PackBytes& p) {
  if (ctx.pack_a.try_reserve((size_t)p.a) && ctx.pack_b.try_reserve((size_t)p.b)) return true;
  ctx.pack_a.release();   // the room is needed elsewhere
  ctx.pack_b.release();
  return false;
}

bool split_reserve(Context& ctx, int64_t M, int64_t N, int64_t K) {
  return split_reserve(ctx, split_pack_bytes(M, N, K)) && ctx.pack_ma.try_reserve((size_t)M * sizeof(int)) &&
         ctx.pack_mb.try_reserve((size_t)N * sizeof(int)) && ctx.pack_ke.try_reserve((size_t)K * 2 * sizeof(int));
}

void split_scale(Context& ctx, const c64* A, int64_t lda, bool conj_trans, int64_t M, int64_t K) {
  hipStream_t st = ctx.stream;
  int* ke = ctx.pack_ke.as<int>();
  int* ma = ke + K;
  zero_max(st, ma, K);
  hipLaunchKernelGGL(k_split_kmax, dim3((unsigned)((K + 63) / 64), (unsigned)((M + 511) / 512)), dim3(256), 0, st,
                     source_a(A, lda, conj_trans), M, K, ma);
  FOSB_LAUNCH_CHECK();
  hipLaunchKernelGGL(k_split_kexp, dim3((unsigned)((K + 255) / 256)), dim3(256), 0, st, ma, K, ke);
  FOSB_LAUNCH_CHECK();
}

void split_scale_diag(Context& ctx, const c64* A, int64_t lda, int64_t K) {
  hipLaunchKernelGGL(k_split_kexp_diag, dim3((unsigned)((K + 255) / 256)), dim3(256), 0, ctx.stream, A, lda, K,
                     ctx.pack_ke.as<int>());
  FOSB_LAUNCH_CHECK();
}

// nblk: 32-row blocks written, those past R with zeros
static void pack(Context& ctx, const SplitSrc& s, int64_t R, int64_t K, int flip, int64_t nblk, DevBuf& buf,
                 DevBuf& mx) {
  const int64_t nkb = (K + 15) / 16;
  if (buf.cap < (size_t)pack_bytes(nblk, K) || mx.cap < (size_t)R * sizeof(int))
    fail(FOSB_E_DEVICE, "internal: packed operand without room");
  hipStream_t st = ctx.stream;
  const int* ke = ctx.pack_ke.as<int>();
  zero_max(st, mx.as<int>(), R);
  hipLaunchKernelGGL(k_split_max, dim3((unsigned)((R + 31) / 32), (unsigned)((K + 511) / 512)), dim3(256), 0, st, s, R,
                     K, ke, flip, mx.as<int>());
  FOSB_LAUNCH_CHECK();
  hipLaunchKernelGGL(k_split_pack, dim3((unsigned)((nkb + 3) / 4), (unsigned)nblk), dim3(256), 0, st, s, R, K, nkb, ke,
                     flip, mx.as<int>(), buf.as<h8>());
  FOSB_LAUNCH_CHECK();
}

void split_pack_a(Context& ctx, const c64* A, int64_t lda, bool conj_trans, int64_t M, int64_t K) {
  pack(ctx, source_a(A, lda, conj_trans), M, K, 0, blocks_a(M), ctx.pack_a, ctx.pack_ma);
}
void split_pack_b(Context& ctx, const c64* B, int64_t ldb, int64_t N, int64_t K) {
  pack(ctx, SplitSrc{B, 1, ldb, 0}, N, K, -1, blocks_b(N), ctx.pack_b, ctx.pack_mb);
}

void split_gemm(Context& ctx, int64_t row0, int64_t M, int64_t N, int64_t K, double alpha, double beta, c64* C,
                int64_t ldc, int diag_nb) {
  if (M <= 0 || N <= 0) return;
  if (row0 % 32 != 0) fail(FOSB_E_DEVICE, "internal: packed rows start at a multiple of 32");
  const int64_t nkb = (K + 15) / 16;
  const int64_t nM = (M + kTileM - 1) / kTileM, nN = (N + kTileN - 1) / kTileN;
  if (nM * nN > INT32_MAX / 2) fail(FOSB_E_UNSUPPORTED, "product of %lld x %lld", (long long)M, (long long)N);
  const int64_t grid = std::min<int64_t>((nM * nN + 7) / 8 * 8, std::max<int64_t>(8, ctx.n_cu / 8 * 8));
  hipLaunchKernelGGL(k_gemm_split, dim3((unsigned)grid), dim3(512), 0, ctx.stream, M, N, nkb, (float)alpha,
                     ctx.pack_a.as<h8>() + row0 / 32 * nkb * (kPlanes * kChunk), ctx.pack_ma.as<int>() + row0,
                     ctx.pack_b.as<h8>(), ctx.pack_mb.as<int>(), (float)beta, C, ldc, (int)nM, (int)nN, diag_nb);
  FOSB_LAUNCH_CHECK();
}

}  // namespace fosb
