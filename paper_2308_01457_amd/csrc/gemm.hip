// Complex GEMM on CDNA matrix cores:  C = beta*C + alpha*op(A)*B  (row-major,
// interleaved complex, real alpha/beta; op(A) = A or its conjugate transpose).  FP64 uses v_mfma_f64_16x16x4f64,
// FP32 uses v_mfma_f32_16x16x4f32.  The complex product is formed with three
// real products (Higham's 3M form):
//   T1 = Ar Br,  T2 = Ai Bi,  T3 = (Ar + Ai)(Br + Bi),
//   Re C = T1 - T2,  Im C = T3 - T1 - T2,
// the operand sums being formed in registers from the staged tiles.
//
// Tiling: 256 threads (4 wave64) per workgroup, 2 x 2 waves of WM x WN MFMA 16x16
// blocks each; K is staged in slices through double-buffered LDS (planar for
// FP32, interleaved for FP64), A stored k-major so that a fragment load is 16
// consecutive rows.  Operand fragments (16x16x4): lane l holds
// A[l%16][k0 + l/16] and B[k0 + l/16][l%16]; accumulator element v (0..3) of
// lane l is D[row][l%16] with row = 4*(l/16) + v for the FP32 instruction and
// row = l/16 + 4*v for the FP64 one.
#include <algorithm>
#include <functional>
#include <map>
#include <type_traits>

#include "common.h"

namespace fosb {

template <typename T>
struct Mfma;

template <>
struct Mfma<double> {
  typedef double v4 __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ v4 op(double a, double b, v4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int q, int v) { return q + 4 * v; }
};

template <>
struct Mfma<float> {
  typedef float v4 __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ v4 op(float a, float b, v4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int q, int v) { return 4 * q + v; }
};

constexpr int NXCD = 8;  // accelerator complex dies; workgroups are dealt to them round-robin
constexpr int GM = 8;    // tile rows per group of the tile order
constexpr int PADA = 4, PADB = 4;
// K slice staged per LDS buffer: 16 (FP32) / 8 (FP64), two buffers, so one
// barrier per slice and the next slice's global loads overlap the MFMAs.
template <typename T> struct Slice { static constexpr int BK = 16; };
template <> struct Slice<double> { static constexpr int BK = 8; };

// XCD-aware tile order: workgroup L runs on XCD L % 8, so XCD x is given the
// contiguous tile range [start(x), start(x) + count(x)), walked in groups of
// GM tile rows, column by column: the ~64 workgroups resident on one XCD then
// cover an 8 x 8 block of tiles and share their A rows and B columns in that
// XCD's L2.
__device__ __forceinline__ void tile_of_block(int64_t& tm, int64_t& tn) {
  const int64_t nN = gridDim.x, nM = gridDim.y, ntile = nN * nM;
  const int64_t L = (int64_t)blockIdx.y * nN + blockIdx.x;
  const int64_t x = L % NXCD, slot = L / NXCD;
  const int64_t t = x * (ntile / NXCD) + min(x, ntile % NXCD) + slot;
  const int64_t group = t / (GM * nN);
  const int64_t fm = group * GM;
  const int64_t gs = min<int64_t>(nM - fm, GM);
  const int64_t in = t - group * GM * nN;
  tm = fm + in % gs;
  tn = in / gs;
}

// One entry of C, or (P given) of a split-K partial product, from the three real products.
template <typename T>
__device__ __forceinline__ void store_entry(int64_t M, int64_t N, int64_t row, int64_t col, T t1, T t2, T t3, T alpha,
                                            T beta, cplx<T>* __restrict__ C, int64_t ldc, cplx<T>* __restrict__ P) {
  if (row >= M || col >= N) return;
  const T cr = t1 - t2;
  const T ci = t3 - t1 - t2;
  if (P) {
    P[row * N + col] = cplx<T>{cr, ci};
    return;
  }
  cplx<T>* p = C + row * ldc + col;
  if (beta == T(0)) {
    *p = cplx<T>{alpha * cr, alpha * ci};
  } else {
    const cplx<T> o = *p;
    *p = cplx<T>{beta * o.re + alpha * cr, beta * o.im + alpha * ci};
  }
}

// Split K: workgroup z of gridDim.z covers K range [kb, ke) = [z*kc, min(K, (z+1)*kc));
// with gridDim.z > 1 it writes its raw partial product to P + z*M*N (row stride N)
// and k_gemm_splitk_sum forms C = beta*C + alpha*sum_z P_z in fixed z order.
// Tile: 2 x 2 waves, each owning WM x WN blocks of 16 x 16, so the workgroup
// covers BM = 32 WM rows and BN = 32 WN columns.  Every variant accumulates an
// output element over K in the same order (same slices, same MFMA steps), so
// the tile choice does not change results.
template <typename T, bool CONJ_A, int WM, int WN>
__device__ __forceinline__ void gemm_tile(int64_t M, int64_t N, int64_t K, T alpha, const cplx<T>* __restrict__ A,
                                          int64_t lda, const cplx<T>* __restrict__ B, int64_t ldb, T beta,
                                          cplx<T>* __restrict__ C, int64_t ldc, int64_t kb, int64_t ke,
                                          cplx<T>* __restrict__ P) {
  using V4 = typename Mfma<T>::v4;
  constexpr int BK = Slice<T>::BK;
  constexpr int BM = 32 * WM, BN = 32 * WN;
  constexpr int AE = BM * BK / 256;  // A elements staged per thread
  constexpr int BE = BN * BK / 256;  // B elements staged per thread
  __shared__ T AsR[2][BK][BM + PADA];
  __shared__ T AsI[2][BK][BM + PADA];
  __shared__ T BsR[2][BK][BN + PADB];
  __shared__ T BsI[2][BK][BN + PADB];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int wr = wave >> 1;  // wave row (0..1): rows wr*16*WM ..
  const int wc = wave & 1;   // wave col (0..1): cols wc*16*WN ..
  int64_t tm, tn;
  tile_of_block(tm, tn);
  const int64_t m0 = tm * BM;
  const int64_t n0 = tn * BN;

  // global -> register staging assignment (op(A) = A^H: threads run along the
  // rows of op(A), which are contiguous in memory)
  const int a_row = CONJ_A ? tid % BM : tid / (BK / AE);
  const int a_k = CONJ_A ? (tid / BM) * AE : (tid % (BK / AE)) * AE;
  const int b_k = tid / (BN / BE);
  const int b_col = (tid % (BN / BE)) * BE;

  cplx<T> ra[AE], rb[BE];
  const bool interior = m0 + BM <= M && n0 + BN <= N;  // no tile edge in M or N
  auto load_tiles = [&](int64_t k0) {
    const int64_t gr = m0 + a_row;
    if (interior && k0 + BK <= ke) {  // the whole slice is inside the operands: no edge checks
      // B's loads first: issued last, they would equal the checked path's
      // closing loads, and the compiler would merge the two tails and wait for
      // A's loads before issuing them.
      const cplx<T>* brow = B + (k0 + b_k) * ldb + n0 + b_col;
#pragma unroll
      for (int e = 0; e < BE; ++e) rb[e] = brow[e];
#pragma unroll
      for (int e = 0; e < AE; ++e) {
        const int64_t gk = k0 + a_k + e;
        if (CONJ_A) {
          const cplx<T> v = A[gk * lda + gr];
          ra[e] = cplx<T>{v.re, -v.im};
        } else {
          ra[e] = A[gr * lda + gk];
        }
      }
      return;
    }
#pragma unroll
    for (int e = 0; e < AE; ++e) {
      const int64_t gk = k0 + a_k + e;
      if (CONJ_A) {
        const cplx<T> v = (gr < M && gk < ke) ? A[gk * lda + gr] : cplx<T>{T(0), T(0)};
        ra[e] = cplx<T>{v.re, -v.im};
      } else {
        ra[e] = (gr < M && gk < ke) ? A[gr * lda + gk] : cplx<T>{T(0), T(0)};
      }
    }
    const int64_t gk = k0 + b_k;
#pragma unroll
    for (int e = 0; e < BE; ++e) {
      const int64_t gc = n0 + b_col + e;
      rb[e] = (gk < ke && gc < N) ? B[gk * ldb + gc] : cplx<T>{T(0), T(0)};
    }
  };
  auto store_tiles = [&](int buf) {
#pragma unroll
    for (int e = 0; e < AE; ++e) {
      AsR[buf][a_k + e][a_row] = ra[e].re;
      AsI[buf][a_k + e][a_row] = ra[e].im;
    }
#pragma unroll
    for (int e = 0; e < BE; ++e) {
      BsR[buf][b_k][b_col + e] = rb[e].re;
      BsI[buf][b_k][b_col + e] = rb[e].im;
    }
  };

  V4 t1[WM][WN], t2[WM][WN], t3[WM][WN];
#pragma unroll
  for (int i = 0; i < WM; ++i)
#pragma unroll
    for (int j = 0; j < WN; ++j) {
      t1[i][j] = V4{0, 0, 0, 0};
      t2[i][j] = V4{0, 0, 0, 0};
      t3[i][j] = V4{0, 0, 0, 0};
    }

  const int r16 = lane & 15;
  const int kq = lane >> 4;
  auto compute = [&](int buf) {
#pragma unroll
    for (int kk = 0; kk < BK; kk += 4) {
      T ar[WM], ai[WM], as[WM], br[WN], bi[WN], bs[WN];
#pragma unroll
      for (int i = 0; i < WM; ++i) {
        ar[i] = AsR[buf][kk + kq][wr * 16 * WM + i * 16 + r16];
        ai[i] = AsI[buf][kk + kq][wr * 16 * WM + i * 16 + r16];
        as[i] = ar[i] + ai[i];
      }
#pragma unroll
      for (int j = 0; j < WN; ++j) {
        br[j] = BsR[buf][kk + kq][wc * 16 * WN + j * 16 + r16];
        bi[j] = BsI[buf][kk + kq][wc * 16 * WN + j * 16 + r16];
        bs[j] = br[j] + bi[j];
      }
#pragma unroll
      for (int i = 0; i < WM; ++i)
#pragma unroll
        for (int j = 0; j < WN; ++j) {
          t1[i][j] = Mfma<T>::op(ar[i], br[j], t1[i][j]);
          t2[i][j] = Mfma<T>::op(ai[i], bi[j], t2[i][j]);
          t3[i][j] = Mfma<T>::op(as[i], bs[j], t3[i][j]);
        }
    }
  };

  if (ke > kb) {
    load_tiles(kb);
    store_tiles(0);
    __syncthreads();
    int buf = 0;
    for (int64_t k0 = kb; k0 < ke; k0 += BK) {
      const bool more = k0 + BK < ke;
      if (more) load_tiles(k0 + BK);  // next slice in flight during the MFMAs
      compute(buf);
      if (more) store_tiles(buf ^ 1);  // the other buffer was last read before the previous barrier
      __syncthreads();
      buf ^= 1;
    }
  }

  // epilogue
#pragma unroll
  for (int i = 0; i < WM; ++i)
#pragma unroll
    for (int j = 0; j < WN; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int64_t row = m0 + wr * 16 * WM + i * 16 + Mfma<T>::row(kq, v);
        const int64_t col = n0 + wc * 16 * WN + j * 16 + r16;
        store_entry<T>(M, N, row, col, t1[i][j][v], t2[i][j][v], t3[i][j][v], alpha, beta, C, ldc, P);
      }
}

#define FOSB_GEMM_ARGS(T)                                                                                     \
  int64_t M, int64_t N, int64_t K, T alpha, const cplx<T>* __restrict__ A, int64_t lda,                       \
      const cplx<T>* __restrict__ B, int64_t ldb, T beta, cplx<T>* __restrict__ C, int64_t ldc, int64_t kc,    \
      cplx<T>* __restrict__ P

template <typename T, bool CONJ_A, int WM, int WN>
__global__ __launch_bounds__(256) void k_gemm(FOSB_GEMM_ARGS(T)) {
  const int64_t kb = (int64_t)blockIdx.z * kc;
  gemm_tile<T, CONJ_A, WM, WN>(M, N, K, alpha, A, lda, B, ldb, beta, C, ldc, kb, min(K, kb + kc),
                               gridDim.z > 1 ? P + (int64_t)blockIdx.z * M * N : nullptr);
}

// FP64 products.  A 3M block of 16 x 16 x 4 is three MFMAs of 32 cycles, so what
// bounds this kernel is everything else a wave issues between them and waits for:
//  - the tiles stay interleaved in LDS and a fragment is one 16-byte read; rows are
//    padded by one entry, so neither the k-major store of A nor the reads conflict;
//  - a slice's global loads are issued two slices ahead;
//  - the loop over whole slices has no edge checks: rows and columns outside the
//    operands read the last one inside (their results are not stored), and the
//    last slices (K's tail) take the checked loads of the second loop;
//  - at most 256 registers, so that the accumulators are VGPRs: with more, the
//    compiler keeps them in AGPRs and copies them in and out on every step;
//  - 64 x 32 and 64 x 64 tiles run at four and three waves per SIMD, which cover
//    each other's waits; 64 x 96, the least LDS reading per MFMA, leaves room for two and
//    reads the next step's fragments while this step's MFMAs run (PIPE).
// Accumulation over K is in steps of 4 from the lowest, as in gemm_tile, so that
// tiles give identical results. TFLOP/s (8 per complex multiply-add) of the best
// tile, planar LDS tiles with checked loads before -> this kernel: 30720 x 480 x
// 30720 71 -> 84, 7680^3 76 -> 88, 7680 x 7680 x 256 66 -> 76, 7680 x 273 x 7680 51
// -> 59, 7680 x 480 x 7680 61 -> 73 (A^H B 56 -> 73), 3840 x 96 x 3840 35 -> 40.
// The MFMAs alone would allow 105.
template <bool CONJ_A, int WM, int WN>
__device__ __forceinline__ void gemm64_tile(int64_t M, int64_t N, int64_t K, double alpha,
                                            const c128* __restrict__ A, int64_t lda, const c128* __restrict__ B,
                                            int64_t ldb, double beta, c128* __restrict__ C, int64_t ldc, int64_t kb,
                                            int64_t ke, c128* __restrict__ P) {
  using V4 = Mfma<double>::v4;
  constexpr bool PIPE = WN > 2;
  constexpr int BK = Slice<double>::BK;
  constexpr int BM = 32 * WM, BN = 32 * WN;
  constexpr int AE = BM * BK / 256, BE = BN * BK / 256;   // entries staged per thread
  __shared__ __align__(16) c128 As[2][BK][BM + 1];
  __shared__ __align__(16) c128 Bs[2][BK][BN + 1];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, wr = wave >> 1, wc = wave & 1;
  int64_t tm, tn;
  tile_of_block(tm, tn);
  const int64_t m0 = tm * BM, n0 = tn * BN;

  int ak[AE], ar[AE], bk[BE], bc[BE];
  const c128 *pa[AE], *pb[BE];
#pragma unroll
  for (int e = 0; e < AE; ++e) {
    const int x = e * 256 + tid;
    ak[e] = CONJ_A ? x / BM : x % BK;   // op(A) = A^H: its rows are contiguous in memory
    ar[e] = CONJ_A ? x % BM : x / BK;
    const int64_t r = min(m0 + ar[e], M - 1);
    pa[e] = CONJ_A ? A + (kb + ak[e]) * lda + r : A + r * lda + kb + ak[e];
  }
#pragma unroll
  for (int e = 0; e < BE; ++e) {
    const int x = e * 256 + tid;
    bk[e] = x / BN;
    bc[e] = x % BN;
    pb[e] = B + (kb + bk[e]) * ldb + min(n0 + bc[e], N - 1);
  }
  const int64_t da = CONJ_A ? BK * lda : BK, db = BK * ldb;
  c128 ra[AE], rb[BE];
  auto load = [&](auto whole, int64_t k0) {
#pragma unroll
    for (int e = 0; e < BE; ++e) {
      rb[e] = whole || k0 + bk[e] < ke ? *pb[e] : c128{0.0, 0.0};
      pb[e] += db;
    }
#pragma unroll
    for (int e = 0; e < AE; ++e) {
      ra[e] = whole || k0 + ak[e] < ke ? *pa[e] : c128{0.0, 0.0};
      pa[e] += da;
    }
  };
  auto store = [&](int buf) {
#pragma unroll
    for (int e = 0; e < BE; ++e) Bs[buf][bk[e]][bc[e]] = rb[e];
#pragma unroll
    for (int e = 0; e < AE; ++e) As[buf][ak[e]][ar[e]] = c128{ra[e].re, CONJ_A ? -ra[e].im : ra[e].im};
  };
  V4 t1[WM][WN], t2[WM][WN], t3[WM][WN];
#pragma unroll
  for (int i = 0; i < WM; ++i)
#pragma unroll
    for (int j = 0; j < WN; ++j) t1[i][j] = t2[i][j] = t3[i][j] = V4{0, 0, 0, 0};
  const int r16 = lane & 15, kq = lane >> 4;
  struct Frag {
    c128 a[WM], b[WN];
  } f[2];
  auto read = [&](Frag& x, int buf, int kk) {
#pragma unroll
    for (int i = 0; i < WM; ++i) x.a[i] = As[buf][4 * kk + kq][wr * 16 * WM + i * 16 + r16];
#pragma unroll
    for (int j = 0; j < WN; ++j) x.b[j] = Bs[buf][4 * kk + kq][wc * 16 * WN + j * 16 + r16];
  };
  auto mul = [&](const Frag& x) {
    double as[WM], bs[WN];
#pragma unroll
    for (int i = 0; i < WM; ++i) as[i] = x.a[i].re + x.a[i].im;
#pragma unroll
    for (int j = 0; j < WN; ++j) bs[j] = x.b[j].re + x.b[j].im;
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
      for (int j = 0; j < WN; ++j) {
        t1[i][j] = Mfma<double>::op(x.a[i].re, x.b[j].re, t1[i][j]);
        t2[i][j] = Mfma<double>::op(x.a[i].im, x.b[j].im, t2[i][j]);
        t3[i][j] = Mfma<double>::op(as[i], bs[j], t3[i][j]);
      }
  };
  constexpr std::true_type whole{};
  constexpr std::false_type checked{};
  // one slice; ra and rb hold the next one, with PIPE f[0] the fragments of its first step
  auto slice = [&](auto w, int64_t k0, int buf) {
    static_assert(BK == 8, "two steps of 4 a slice");
    if constexpr (PIPE) {
      read(f[1], buf, 1);
      store(buf ^ 1);
      load(w, k0 + 2 * BK);
      mul(f[0]);
      // the reads, stores and loads between the MFMAs, not before them
#pragma unroll
      for (int q = 0; q < 3 * WM * WN; ++q) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // MFMA
        __builtin_amdgcn_sched_group_barrier(0x002, 2, 0);   // VALU
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);   // LDS read
        __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);   // LDS write
        __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);   // global load
      }
      __syncthreads();
      read(f[0], buf ^ 1, 0);
      mul(f[1]);
    } else {
      read(f[0], buf, 0);
      mul(f[0]);
      read(f[0], buf, 1);
      mul(f[0]);
      store(buf ^ 1);
      load(w, k0 + 2 * BK);
      __syncthreads();
    }
  };
  if (ke > kb) {
    int64_t k0 = kb;
    int buf = 0;
    load(checked, k0);
    store(0);
    load(checked, k0 + BK);
    __syncthreads();
    if constexpr (PIPE) read(f[0], 0, 0);
    for (; k0 + 3 * BK <= ke; k0 += BK, buf ^= 1) slice(whole, k0, buf);
    for (; k0 < ke; k0 += BK, buf ^= 1) slice(checked, k0, buf);
  }
#pragma unroll
  for (int i = 0; i < WM; ++i)
#pragma unroll
    for (int j = 0; j < WN; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int64_t row = m0 + wr * 16 * WM + i * 16 + Mfma<double>::row(kq, v);
        const int64_t col = n0 + wc * 16 * WN + j * 16 + r16;
        store_entry<double>(M, N, row, col, t1[i][j][v], t2[i][j][v], t3[i][j][v], alpha, beta, C, ldc, P);
      }
}

template <bool CONJ_A, int WM, int WN>
__global__ __launch_bounds__(256, WN == 1 ? 4 : WN == 2 ? 3 : 2) void k_gemm64(FOSB_GEMM_ARGS(double)) {
  const int64_t kb = (int64_t)blockIdx.z * kc;
  gemm64_tile<CONJ_A, WM, WN>(M, N, K, alpha, A, lda, B, ldb, beta, C, ldc, kb, min(K, kb + kc),
                              gridDim.z > 1 ? P + (int64_t)blockIdx.z * M * N : nullptr);
}
#undef FOSB_GEMM_ARGS

// Inverse of a triangular 2h x 2h diagonal block from those of its h x h halves:
// lower, X21 = -(A22^-1) (A21 A11^-1); upper, X12 = -(A11^-1) (A12 A22^-1).  STEP 0 forms the
// product in parentheses in T (h x h a pair), STEP 1 the other.  Pair z is at
// row 2hz of the factor; W holds the inverses in blocks of ib rows.  The last
// pair's second half may be short (m rows) or missing.
template <bool LOWER, int STEP>
__global__ __launch_bounds__(256) void k_inverse_merge(int64_t n, const c64* __restrict__ A, int64_t lda,
                                                       c64* __restrict__ W, int64_t ib, int64_t h,
                                                       c64* __restrict__ T) {
  const int64_t r = 2 * h * blockIdx.z, m = min(h, n - r - h);
  if (m <= 0) return;
  c64* w11 = W + r / ib * ib * ib + r % ib * (ib + 1);
  c64* w22 = w11 + h * (ib + 1);
  T += h * h * blockIdx.z;
  const int64_t rows = LOWER ? m : h, cols = LOWER ? h : m;
  if (STEP == 0)
    gemm_tile<float, false, 2, 2>(rows, cols, cols, 1.f, LOWER ? A + (r + h) * lda + r : A + r * lda + r + h, lda,
                                  LOWER ? w11 : w22, ib, 0.f, T, h, 0, cols, nullptr);
  else
    gemm_tile<float, false, 2, 2>(rows, cols, rows, -1.f, LOWER ? w22 : w11, ib, T, h, 0.f,
                                  LOWER ? w11 + h * ib : w11 + h, ib, 0, rows, nullptr);
}

void inverse_merge(hipStream_t s, bool lower, int64_t n, const c64* A, int64_t lda, c64* W, int64_t ib, int64_t h,
                   c64* T) {
  const int64_t pairs = (n - h + 2 * h - 1) / (2 * h);   // pairs with a second half
  if (n <= h) return;
  const dim3 g((unsigned)((h + 63) / 64), (unsigned)((h + 63) / 64), (unsigned)pairs), b(256);
  if (lower) {
    hipLaunchKernelGGL((k_inverse_merge<true, 0>), g, b, 0, s, n, A, lda, W, ib, h, T);
    hipLaunchKernelGGL((k_inverse_merge<true, 1>), g, b, 0, s, n, A, lda, W, ib, h, T);
  } else {
    hipLaunchKernelGGL((k_inverse_merge<false, 0>), g, b, 0, s, n, A, lda, W, ib, h, T);
    hipLaunchKernelGGL((k_inverse_merge<false, 1>), g, b, 0, s, n, A, lda, W, ib, h, T);
  }
  FOSB_LAUNCH_CHECK();
}

template <typename T>
__global__ __launch_bounds__(256) void k_gemm_splitk_sum(int64_t M, int64_t N, int nz, T alpha,
                                                         const cplx<T>* __restrict__ P, T beta,
                                                         cplx<T>* __restrict__ C, int64_t ldc) {
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= M * N) return;
  const int64_t row = idx / N, col = idx % N;
  T sr = 0, si = 0;
  for (int z = 0; z < nz; ++z) {
    const cplx<T> v = P[(int64_t)z * M * N + idx];
    sr += v.re;
    si += v.im;
  }
  cplx<T>* p = C + row * ldc + col;
  if (beta == T(0)) {
    *p = cplx<T>{alpha * sr, alpha * si};
  } else {
    const cplx<T> o = *p;
    *p = cplx<T>{beta * o.re + alpha * sr, beta * o.im + alpha * si};
  }
}

// Narrow right-hand sides (N <= 4, e.g. one incidence): a bandwidth-bound
// product, one wave per row of A streaming it once with 16-byte loads; the N
// columns of B are read through the cache.  Row sums are reduced in the wave.
constexpr int GEMV_MAXN = 4;

template <typename T, int NC>
__global__ __launch_bounds__(256) void k_gemv(int64_t M, int64_t K, T alpha, const cplx<T>* __restrict__ A,
                                              int64_t lda, const cplx<T>* __restrict__ B, int64_t ldb, T beta,
                                              cplx<T>* __restrict__ C, int64_t ldc) {
  const int lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= M) return;
  const cplx<T>* a = A + row * lda;
  T ar[NC], ai[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) ar[c] = ai[c] = T(0);
  int64_t k = lane;
  for (; k + 192 < K; k += 256) {
    cplx<T> v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = a[k + 64 * u];
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const cplx<T> b = B[(k + 64 * u) * ldb + c];
        ar[c] += v[u].re * b.re - v[u].im * b.im;
        ai[c] += v[u].re * b.im + v[u].im * b.re;
      }
  }
  for (; k < K; k += 64) {
    const cplx<T> v = a[k];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const cplx<T> b = B[k * ldb + c];
      ar[c] += v.re * b.re - v.im * b.im;
      ai[c] += v.re * b.im + v.im * b.re;
    }
  }
#pragma unroll
  for (int c = 0; c < NC; ++c) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      ar[c] += __shfl_xor(ar[c], o);
      ai[c] += __shfl_xor(ai[c], o);
    }
  }
  if (lane < NC) {
    T sr = ar[0], si = ai[0];
#pragma unroll
    for (int c = 1; c < NC; ++c)
      if (lane == c) sr = ar[c], si = ai[c];
    cplx<T>* p = C + row * ldc + lane;
    if (beta == T(0)) {
      *p = cplx<T>{alpha * sr, alpha * si};
    } else {
      const cplx<T> o = *p;
      *p = cplx<T>{beta * o.re + alpha * sr, beta * o.im + alpha * si};
    }
  }
}

template <typename T, int NC>
static void gemv_launch(Context& ctx, int64_t M, int64_t K, double alpha, const cplx<T>* A, int64_t lda,
                        const cplx<T>* B, int64_t ldb, double beta, cplx<T>* C, int64_t ldc) {
  hipLaunchKernelGGL((k_gemv<T, NC>), dim3((unsigned)((M + 3) / 4)), dim3(256), 0, ctx.stream, M, K, (T)alpha, A,
                     lda, B, ldb, (T)beta, C, ldc);
  FOSB_LAUNCH_CHECK();
}

// Tile variants (WM, WN) offered to the autotuner, fastest-first by measurement
// on gfx950 (the first entry is the built-in choice when tuning is off).
template <typename T> struct Tiles;
// `lean` is the variant with the smallest register and LDS footprint.
template <> struct Tiles<float> {
  static constexpr int n = 4;
  static constexpr int wm[4] = {2, 2, 2, 4}, wn[4] = {2, 1, 4, 2};
  static constexpr int lean = 1;  // 64 x 32
};
template <> struct Tiles<double> {
  static constexpr int n = 3;
  static constexpr int wm[3] = {2, 2, 2}, wn[3] = {1, 2, 3};
  static constexpr int lean = 0;  // 64 x 32
};

template <typename T, bool CONJ_A, int WM, int WN>
static void launch_tile(hipStream_t s, int64_t M, int64_t N, int64_t K, T alpha, const cplx<T>* A, int64_t lda,
                        const cplx<T>* B, int64_t ldb, T beta, cplx<T>* C, int64_t ldc, int64_t kc, cplx<T>* P,
                        int64_t nz) {
  dim3 grid((unsigned)((N + 32 * WN - 1) / (32 * WN)), (unsigned)((M + 32 * WM - 1) / (32 * WM)), (unsigned)nz);
  if constexpr (sizeof(T) == 8)
    hipLaunchKernelGGL((k_gemm64<CONJ_A, WM, WN>), grid, dim3(256), 0, s, M, N, K, alpha, A, lda, B, ldb, beta, C, ldc,
                       kc, P);
  else
    hipLaunchKernelGGL((k_gemm<T, CONJ_A, WM, WN>), grid, dim3(256), 0, s, M, N, K, alpha, A, lda, B, ldb, beta, C,
                       ldc, kc, P);
  FOSB_LAUNCH_CHECK();
}

template <typename T, bool CONJ_A>
static void launch_variant(int var, hipStream_t s, int64_t M, int64_t N, int64_t K, T alpha, const cplx<T>* A,
                           int64_t lda, const cplx<T>* B, int64_t ldb, T beta, cplx<T>* C, int64_t ldc, int64_t kc,
                           cplx<T>* P, int64_t nz) {
  if constexpr (sizeof(T) == 4) {
    switch (var) {
      case 1: return launch_tile<T, CONJ_A, 2, 1>(s, M, N, K, alpha, A, lda, B, ldb, beta, C, ldc, kc, P, nz);
      case 2: return launch_tile<T, CONJ_A, 2, 4>(s, M, N, K, alpha, A, lda, B, ldb, beta, C, ldc, kc, P, nz);
      case 3: return launch_tile<T, CONJ_A, 4, 2>(s, M, N, K, alpha, A, lda, B, ldb, beta, C, ldc, kc, P, nz);
      default: return launch_tile<T, CONJ_A, 2, 2>(s, M, N, K, alpha, A, lda, B, ldb, beta, C, ldc, kc, P, nz);
    }
  } else {
    switch (var) {
      case 1: return launch_tile<T, CONJ_A, 2, 2>(s, M, N, K, alpha, A, lda, B, ldb, beta, C, ldc, kc, P, nz);
      case 2: return launch_tile<T, CONJ_A, 2, 3>(s, M, N, K, alpha, A, lda, B, ldb, beta, C, ldc, kc, P, nz);
      default: return launch_tile<T, CONJ_A, 2, 1>(s, M, N, K, alpha, A, lda, B, ldb, beta, C, ldc, kc, P, nz);
    }
  }
}

static inline int log2_bucket(int64_t x) {
  int b = 0;
  while (x > 1) {
    x >>= 1;
    ++b;
  }
  return b;
}

// Tile variant for this product: the tuned choice of its size bucket (precision,
// A operand form, floor(log2) of M, N and K).  A bucket met for the first time
// with tuning on is settled by timing every variant on the real operands into
// scratch output (three interleaved rounds, each variant's fastest run counts);
// the choice is kept by the root context.  The variants give identical
// results, so tuning only affects speed.
template <typename T, bool CONJ_A>
static int pick_variant(Context& ctx, int64_t M, int64_t N, int64_t K, const cplx<T>* A, int64_t lda,
                        const cplx<T>* B, int64_t ldb) {
  Context& root = ctx.prof_root ? *ctx.prof_root : ctx;
  if (!root.autotune) return 0;
  const int64_t key = ((int64_t)(sizeof(T) == 8) << 40) | ((int64_t)CONJ_A << 39) | ((int64_t)log2_bucket(M) << 26) |
                      ((int64_t)log2_bucket(N) << 13) | (int64_t)log2_bucket(K);
  {
    std::lock_guard<std::mutex> lock(root.tune_mu);
    auto it = root.tune.find(key);
    if (it != root.tune.end()) return it->second;
  }
  if (ctx.no_alloc) return 0;  // no scratch output to time into
  ctx.tune_out.reserve((size_t)M * N * sizeof(cplx<T>));
  if (!ctx.tune_ev[0]) {
    FOSB_HIP(hipEventCreate(&ctx.tune_ev[0]));
    FOSB_HIP(hipEventCreate(&ctx.tune_ev[1]));
  }
  // three rounds over the variants, each variant keeping its fastest run: the
  // chip may be shared with other streams' work, which only ever adds time
  float t[Tiles<T>::n];
  for (int v = 0; v < Tiles<T>::n; ++v) t[v] = 1e30f;
  for (int rep = 0; rep < 3; ++rep)
    for (int v = 0; v < Tiles<T>::n; ++v) {
      FOSB_HIP(hipEventRecord(ctx.tune_ev[0], ctx.stream));
      launch_variant<T, CONJ_A>(v, ctx.stream, M, N, K, T(1), A, lda, B, ldb, T(0),
                                static_cast<cplx<T>*>(ctx.tune_out.p), N, K, nullptr, 1);
      FOSB_HIP(hipEventRecord(ctx.tune_ev[1], ctx.stream));
      FOSB_HIP(hipEventSynchronize(ctx.tune_ev[1]));
      float ms = 0.f;
      FOSB_HIP(hipEventElapsedTime(&ms, ctx.tune_ev[0], ctx.tune_ev[1]));
      t[v] = std::min(t[v], ms);
    }
  int best = 0;
  for (int v = 1; v < Tiles<T>::n; ++v)
    if (t[v] < t[best]) best = v;
  std::lock_guard<std::mutex> lock(root.tune_mu);
  root.tune[key] = best;
  return best;
}

// A packed operand of a split product takes 12 bytes an entry.  1 GiB: solves with
// 480 columns at N = 30720 took 196 ms; bounds of 384, 192 and 96 MiB, whose
// shorter K chunks add more passes over C, 199, 213 and 231 ms.
constexpr int64_t kSplitPackBytes = (int64_t)1 << 30;

// Complex64 products worth packing for the fp16 matrix cores (gemm16.hip): at least
// 256 columns and 256 of K, so that reading and packing A (28 bytes an entry) stays
// below the products saved, and tiles for half the compute units.
static bool split_size(int n_cu, int64_t M, int64_t N, int64_t K) {
  return N >= 256 && K >= 256 && ((M + 255) / 256) * ((N + 127) / 128) >= n_cu / 2;
}
static bool split_pays(const Context& ctx, int64_t M, int64_t N, int64_t K) {
  if (ctx.no_alloc || ctx.lean_tiles > 0) return false;
  return split_size(ctx.n_cu, M, N, K);
}
// K in chunks, so that a packed operand stays within kSplitPackBytes
static int64_t split_chunk(int64_t M, int64_t N) {
  return std::max<int64_t>(256, kSplitPackBytes / (12 * std::max(M, N)) / 256 * 256);
}

PackBytes solve_pack_bytes(int n_cu, int64_t n, int64_t nrhs, int64_t ib) {
  PackBytes p;
  auto product = [&](int64_t M, int64_t K) {
    if (!split_size(n_cu, M, nrhs, K)) return;
    const PackBytes q = split_pack_bytes(M, nrhs, std::min(split_chunk(M, nrhs), K));
    p.a = std::max(p.a, q.a);
    p.b = std::max(p.b, q.b);
  };
  std::function<void(int64_t)> solve = [&](int64_t m) {   // the splits of the triangular solves
    if (m <= ib) return product(m, m);
    const int64_t m1 = ib * (((m + ib - 1) / ib + 1) / 2);
    product(m - m1, m1);
    product(m1, m - m1);
    solve(m1);
    solve(m - m1);
  };
  if (nrhs >= 256) solve(n);
  return p;
}

template <typename T, bool CONJ_A>
static void gemm_launch(Context& ctx, int64_t M, int64_t N, int64_t K, double alpha, const cplx<T>* A, int64_t lda,
                        const cplx<T>* B, int64_t ldb, double beta, cplx<T>* C, int64_t ldc) {
  if (M <= 0 || N <= 0) return;
  if (K <= 0) {
    if (beta == 1.0) return;
  }
  // algorithmic work: 8 flop per complex multiply-add; A, B read and C read+written once
  const double flops = 8.0 * (double)M * (double)N * (double)std::max<int64_t>(K, 0);
  const double bytes = (double)sizeof(cplx<T>) * ((double)M * K + (double)K * N + (beta != 0.0 ? 2.0 : 1.0) * M * N);
  if (!CONJ_A && N <= GEMV_MAXN && K > 0 && (M + 3) / 4 <= INT32_MAX) {
    ProfScope prof(ctx, FOSB_K_GEMV, flops, bytes);
    switch (N) {
      case 1: return gemv_launch<T, 1>(ctx, M, K, alpha, A, lda, B, ldb, beta, C, ldc);
      case 2: return gemv_launch<T, 2>(ctx, M, K, alpha, A, lda, B, ldb, beta, C, ldc);
      case 3: return gemv_launch<T, 3>(ctx, M, K, alpha, A, lda, B, ldb, beta, C, ldc);
      default: return gemv_launch<T, 4>(ctx, M, K, alpha, A, lda, B, ldb, beta, C, ldc);
    }
  }
  const int64_t Kp = std::max<int64_t>(K, 0);
  if constexpr (sizeof(T) == 4) {
    const int64_t kc = split_chunk(M, N);   // the later chunks add to C
    if (split_pays(ctx, M, N, Kp) && split_reserve(ctx, M, N, std::min(kc, Kp))) {
      ProfScope prof(ctx, FOSB_K_GEMM_F32, flops, bytes);
      for (int64_t k0 = 0; k0 < Kp; k0 += kc) {
        const int64_t kn = std::min(kc, Kp - k0);
        const cplx<T>* Ak = CONJ_A ? A + k0 * lda : A + k0;
        const cplx<T>* Bk = B + k0 * ldb;
        split_scale(ctx, Ak, lda, CONJ_A, M, kn);
        split_pack_a(ctx, Ak, lda, CONJ_A, M, kn);
        split_pack_b(ctx, Bk, ldb, N, kn);
        split_gemm(ctx, 0, M, N, kn, alpha, k0 == 0 ? beta : 1.0, C, ldc, 0);
      }
      return;
    }
  }
  // split K when the output has too few tiles to fill the chip: about two
  // workgroups per CU, each still streaming at least 64 of K.  (With 256 instead,
  // from K = 512 on, the solves' leaf and coupling products ran on a few dozen
  // workgroups.  N = 7680: FP64, 480 columns 5.3 -> 4.6 ms, 16 columns 2.9 ->
  // 1.6; mixed, 17 columns 4.4 -> 2.9; adjoint gradient 15.2 -> 12.7.)  The
  // decision uses a fixed 64 x 64 reference tile, so it (and the summation order)
  // does not depend on the tile variant chosen below.
  const int64_t tiles = ((N + 63) / 64) * ((M + 63) / 64);
  int64_t nz = 1;
  const int64_t want = 2LL * ctx.n_cu;
  if (tiles < want && Kp >= 256 && !ctx.no_alloc) nz = std::min<int64_t>({(want + tiles - 1) / tiles, Kp / 64, 64});
  int64_t kc = Kp;
  cplx<T>* P = nullptr;
  if (nz > 1) {
    kc = ((Kp + nz - 1) / nz + Slice<T>::BK - 1) / Slice<T>::BK * Slice<T>::BK;
    nz = (Kp + kc - 1) / kc;
    ctx.splitk.reserve((size_t)nz * M * N * sizeof(cplx<T>), true);
    P = static_cast<cplx<T>*>(ctx.splitk.p);
  }
  // The trailing update's large complex64 products (at least four 128 x 64
  // tiles per CU) take the 64 x 64 tile.  Timed beside the panel stream, the
  // tuner often prefers the 64 x 32 tile for them, whose five workgroups per
  // CU leave the panel stream's kernels no room: the step is then ~4% slower.
  const bool update_big =
      sizeof(T) == 4 && ctx.trailing_update > 0 && ((M + 127) / 128) * ((N + 63) / 64) >= 4LL * ctx.n_cu;
  const int var = (nz != 1 || Kp <= 0) ? 0
                  : ctx.lean_tiles > 0 ? Tiles<T>::lean
                  : update_big         ? 0
                                       : pick_variant<T, CONJ_A>(ctx, M, N, Kp, A, lda, B, ldb);
  {
    ProfScope prof(ctx, sizeof(T) == 8 ? FOSB_K_GEMM_F64 : FOSB_K_GEMM_F32, flops, bytes);
    launch_variant<T, CONJ_A>(var, ctx.stream, M, N, Kp, (T)alpha, A, lda, B, ldb, (T)beta, C, ldc, kc, P, nz);
  }
  if (nz > 1) {
    ProfScope prof(ctx, FOSB_K_SPLITK_SUM, 2.0 * (double)nz * M * N,
                   (double)sizeof(cplx<T>) * ((double)nz + 2.0) * M * N);
    hipLaunchKernelGGL((k_gemm_splitk_sum<T>), dim3((unsigned)((M * N + 255) / 256)), dim3(256), 0, ctx.stream, M, N,
                       (int)nz, (T)alpha, P, (T)beta, C, ldc);
    FOSB_LAUNCH_CHECK();
  }
}

template <typename T>
void gemm(Context& ctx, int64_t M, int64_t N, int64_t K, double alpha, const cplx<T>* A, int64_t lda,
          const cplx<T>* B, int64_t ldb, double beta, cplx<T>* C, int64_t ldc) {
  gemm_launch<T, false>(ctx, M, N, K, alpha, A, lda, B, ldb, beta, C, ldc);
}

template <typename T>
void gemm_ch(Context& ctx, int64_t M, int64_t N, int64_t K, double alpha, const cplx<T>* A, int64_t lda,
             const cplx<T>* B, int64_t ldb, double beta, cplx<T>* C, int64_t ldc) {
  gemm_launch<T, true>(ctx, M, N, K, alpha, A, lda, B, ldb, beta, C, ldc);
}

template void gemm<double>(Context&, int64_t, int64_t, int64_t, double, const c128*, int64_t, const c128*, int64_t,
                           double, c128*, int64_t);
template void gemm<float>(Context&, int64_t, int64_t, int64_t, double, const c64*, int64_t, const c64*, int64_t,
                          double, c64*, int64_t);
template void gemm_ch<double>(Context&, int64_t, int64_t, int64_t, double, const c128*, int64_t, const c128*, int64_t,
                              double, c128*, int64_t);
template void gemm_ch<float>(Context&, int64_t, int64_t, int64_t, double, const c64*, int64_t, const c64*, int64_t,
                             double, c64*, int64_t);

}  // namespace fosb
