// Batched (grouped) dense GEMM on the CDNA4 matrix cores, FP64 and FP32:
//   C_p = alpha A_p B_p + beta C_p    for every problem p of the batch,
// row-major operands with per-problem sizes and leading dimensions.
//
// It forms X_e = A_ii(e)^-1 A_ib(e) and the element blocks T_e = F_e - A_bi(e) X_e
// of the condensed matrix (eq. SC_step1; F_e the A_bb node blocks folded into
// the element, added from a per-element map in the epilogue, so T_e is written
// once), and the trailing updates of the dense LU of S.
//
// Tiling: a workgroup computes a BM x BN tile of one problem; its waves form a
// WM x WN grid, each owning (BM/WM) x (BN/WN) as a block of 16x16x4 MFMAs.  K
// advances in steps of 16: the next A and B slabs are loaded into registers
// (coalesced: consecutive lanes read consecutive addresses) while the current
// slabs, double-buffered in LDS, feed the matrix cores.  A is stored k-major in
// LDS so the 16 lanes of one MFMA operand column read
// consecutive words.  The tile list orders tiles so that one problem's tiles
// share an XCD (workgroups are dealt to the 8 XCDs round-robin), keeping an
// element's operands in that XCD's L2.
//
// Bound by the matrix cores: an FP64 MFMA keeps a SIMD's vector unit for 64 cycles,
// so every vector instruction of the loop is time it does not multiply.  The slab
// loads therefore carry no guard and no address arithmetic (a lane's offset is
// fixed, the slab's address advances in scalar registers), and the last slab of a
// K that is no multiple of 16 is a step of its own; guards inside the loop also
// made the compiler wait for the loads before the products they should overlap.
// 512 elements of order 5 (K = 320): X 2.39 -> 2.12 ms, T 9.19 -> 8.02 ms in FP64
// (58.8 TFLOP/s), 1.31 -> 1.13 and 5.26 -> 4.24 ms in FP32; 216 of order 7 (K =
// 1080): X 21.4 -> 18.6 ms, T 50.0 -> 44.4 ms in FP64 (66.8 TFLOP/s), 11.9 -> 9.3 and
// 27.7 -> 22.5 ms in FP32 (132 TFLOP/s).
#include <algorithm>
#include <type_traits>

#include "internal.hpp"
#include "mfma.hpp"

namespace scdg {

namespace {

constexpr int BK = 16;

// one element at a 32-bit byte offset from a wave-uniform address (both inside an
// operand): the address lives in scalar registers, so a slab's advance costs the
// vector unit nothing
template <typename T>
struct Slab {
  __amdgpu_buffer_rsrc_t r;
  __device__ __forceinline__ explicit Slab(const T *p)
      : r(__builtin_amdgcn_make_buffer_rsrc(const_cast<T *>(p), 0, 0xffffffffu, 0x00027000)) {}
  __device__ __forceinline__ T at(uint32_t off) const {
    if constexpr (sizeof(T) == 8)
      return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0));
    else
      return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));
  }
};

// One tile of C; tile: its place in the tile list (without a list: the tile of the
// only problem).
template <typename T, int BM, int BN, int WM, int WN, bool PRE>
__device__ __forceinline__ void gemm_tile(const GemmDesc *__restrict__ desc, const int32_t *__restrict__ tiles, int tile,
                                          const T *__restrict__ A, const T *__restrict__ B, T *__restrict__ C, T alpha,
                                          T beta, const int32_t *__restrict__ fmap, const double *__restrict__ fval) {
  using M = Mfma<T>;
  constexpr int kThreads = 64 * WM * WN;
  constexpr int PA = BM + 4;             // LDS row strides (padding against bank conflicts)
  constexpr int PB = BN + 4;
  constexpr int WTM = BM / WM, WTN = BN / WN;          // wave tile
  constexpr int TM = WTM / 16, TN = WTN / 16;          // MFMA blocks per wave
  static_assert(WTM % 16 == 0 && WTN % 16 == 0, "wave tile must be a multiple of 16");
  static_assert((BM * BK) % kThreads == 0 && kThreads % BK == 0, "A slab split");
  static_assert((BN * BK) % kThreads == 0 && kThreads % BN == 0, "B slab split");
  constexpr int A_ELEMS = BM * BK / kThreads;          // per-thread slab loads
  constexpr int B_ELEMS = BN * BK / kThreads;
  constexpr int A_ROWS_PER_STEP = kThreads / BK;       // rows of A covered per load step
  constexpr int B_ROWS_PER_STEP = kThreads / BN;       // k rows of B covered per load step
  __shared__ T as[2][BK][PA];
  __shared__ T bs[2][BK][PB];

  int prob, tm, tn;
  if (tiles != nullptr) {
    prob = tiles[3 * tile];
    tm = tiles[3 * tile + 1];
    tn = tiles[3 * tile + 2];
    if (prob < 0) return;
  } else {
    prob = 0;
    const int tiles_m = (desc[0].m + BM - 1) / BM;
    tm = tile % tiles_m;
    tn = tile / tiles_m;
  }
  const GemmDesc d = desc[prob];
  const T *__restrict__ a = A + d.a_off;
  const T *__restrict__ b = B + d.b_off;
  T *__restrict__ c = C + d.c_off;
  const int m0 = tm * BM, n0 = tn * BN;
  if (m0 >= d.m || n0 >= d.n || d.k < 1) return;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wid / WN, wn = wid % WN;

  // A slab: lane t reads k = t % 16 of rows t / 16 + step * 16
  const int a_k = tid % BK, a_r = tid / BK;
  // B slab: lane t reads column t % BN of k rows t / BN + step * (threads / BN)
  const int b_c = tid % BN, b_k = tid / BN;

  // A lane's 32-bit byte offsets from the slab's first element stay the same for
  // every slab; the slab's address advances in scalar registers.  Rows past m and
  // columns past n read the last one's values, which only reach entries that are
  // never stored; only the last slab of a K that is no multiple of 16 is guarded.
  uint32_t oa[A_ELEMS], ob[B_ELEMS];
#pragma unroll
  for (int u = 0; u < A_ELEMS; ++u)
    oa[u] = (uint32_t)(min(a_r + u * A_ROWS_PER_STEP, d.m - 1 - m0) * d.lda + a_k) * (uint32_t)sizeof(T);
#pragma unroll
  for (int u = 0; u < B_ELEMS; ++u)
    ob[u] = (uint32_t)((b_k + u * B_ROWS_PER_STEP) * d.ldb + min(b_c, d.n - 1 - n0)) * (uint32_t)sizeof(T);
  const T *__restrict__ a0 = a + (int64_t)m0 * d.lda;
  const T *__restrict__ b0 = b + n0;
  T ra[A_ELEMS], rb[B_ELEMS];
  auto load = [&](int k0) {
    const Slab<T> pa(a0 + k0), pb(b0 + (int64_t)k0 * d.ldb);
#pragma unroll
    for (int u = 0; u < A_ELEMS; ++u) ra[u] = pa.at(oa[u]);
#pragma unroll
    for (int u = 0; u < B_ELEMS; ++u) rb[u] = pb.at(ob[u]);
  };
  auto load_tail = [&](int k0) {               // the last slab, k0 < k < k0 + 16
    const Slab<T> pa(a0 + k0), pb(b0 + (int64_t)k0 * d.ldb);
    const bool ka = k0 + a_k < d.k;
#pragma unroll
    for (int u = 0; u < A_ELEMS; ++u) {
      const T v = pa.at(ka ? oa[u] : 0);
      ra[u] = ka ? v : T(0);
    }
#pragma unroll
    for (int u = 0; u < B_ELEMS; ++u) {
      const bool kb = k0 + b_k + u * B_ROWS_PER_STEP < d.k;
      const T v = pb.at(kb ? ob[u] : 0);
      rb[u] = kb ? v : T(0);
    }
  };
  auto store = [&](int buf) {
#pragma unroll
    for (int u = 0; u < A_ELEMS; ++u) as[buf][a_k][a_r + u * A_ROWS_PER_STEP] = ra[u];
#pragma unroll
    for (int u = 0; u < B_ELEMS; ++u) bs[buf][b_k + u * B_ROWS_PER_STEP][b_c] = rb[u];
  };

  typename M::acc_t acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = M::zero();

  // 16x16 blocks of this wave's tile that hold real rows / columns: blocks lying
  // wholly in the zero padding of a ragged tile skip their MFMAs (wave-uniform)
  const int tm_valid = min(TM, max(0, (d.m - (m0 + wm * WTM) + 15) / 16));
  const int tn_valid = min(TN, max(0, (d.n - (n0 + wn * WTN) + 15) / 16));
  const int n_full = d.k / BK, nk = (d.k + BK - 1) / BK;
  if (n_full > 0) load(0);
  else load_tail(0);
  // C += +-A B: C's loads run beside the last slab's products, not after them.  (The
  // sums could start from C instead, but then every product is rounded at C's size:
  // the inverse of 1080 rows was a third further off.)
  T old[PRE ? TM : 1][PRE ? TN : 1][4];
  store(0);
  __syncthreads();
  // the K loop is compiled twice: without per-block guards for a wave whose
  // blocks all hold real rows and columns (every wave but those on the ragged
  // edge), so the matrix-core instructions issue back to back with the LDS
  // reads scheduled around them, and with the guards for the others
  auto kloop = [&](auto full_c) {
    constexpr bool FULL = decltype(full_c)::value;
    auto products = [&](int buf) {
#pragma unroll
      for (int kk = 0; kk < BK; kk += 4) {
        T af[TM], bf[TN];
#pragma unroll
        for (int i = 0; i < TM; ++i)
          af[i] = as[buf][kk + (lane >> 4)][wm * WTM + i * 16 + (lane & 15)];
#pragma unroll
        for (int j = 0; j < TN; ++j)
          bf[j] = bs[buf][kk + (lane >> 4)][wn * WTN + j * 16 + (lane & 15)];
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j)
            if (FULL || (i < tm_valid && j < tn_valid)) acc[i][j] = M::mma(af[i], bf[j], acc[i][j]);
      }
    };
    int kt = 0;
    for (; kt + 1 < n_full; ++kt) {
      load((kt + 1) * BK);
      products(kt & 1);
      store((kt + 1) & 1);
      __syncthreads();
    }
    if (kt + 1 < nk) {
      load_tail((kt + 1) * BK);
      products(kt & 1);
      store((kt + 1) & 1);
      __syncthreads();
      ++kt;
    }
    if constexpr (PRE) {
      const T *__restrict__ c0 = c + (int64_t)m0 * d.ldc + n0;
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          const int col = min(wn * WTN + j * 16 + (lane & 15), d.n - 1 - n0);
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int row = min(wm * WTM + i * 16 + M::row(lane, r), d.m - 1 - m0);
            old[i][j][r] = c0[(uint32_t)(row * d.ldc + col)];
          }
        }
    }
    products(kt & 1);
    __syncthreads();                           // the epilogue stages in the slabs' memory
  };
  if (tm_valid == TM && tn_valid == TN)
    kloop(std::true_type{});
  else
    kloop(std::false_type{});

  // the folded A_bb node blocks of this problem's C (Schur GEMM only): the
  // tile's part of the fold map is staged in LDS (free after the K loop), and
  // for each row group of 16 the epilogue first issues every fold-value load
  // of its entries (entries without a fold read block 0, which exists when the
  // tile has any fold, and discard it), then adds and stores, so the loads are
  // in flight together
  const bool fold = fmap != nullptr && d.f_off >= 0;
  int *fm_s = reinterpret_cast<int *>(&as[0][0][0]);
  const int rb0 = m0 / 5, cb0 = n0 / 5;
  const int frw = (min(m0 + BM, d.m) - 1) / 5 - rb0 + 1, fcw = (min(n0 + BN, d.n) - 1) / 5 - cb0 + 1;
  static_assert((BM / 5 + 2) * (BN / 5 + 2) * sizeof(int) <= sizeof(as), "fold map tile fits in LDS");
  bool tile_fold = false;
  if (fold) {
    const int32_t *__restrict__ fm = fmap + d.f_off;
    const int fbn = d.n / 5;
    int any = 0;
    for (int q = threadIdx.x; q < frw * fcw; q += kThreads) {
      const int a = q / fcw, b = q - a * fcw;
      const int32_t f = fm[(int64_t)(rb0 + a) * fbn + cb0 + b];
      fm_s[q] = f;
      any |= f >= 0;
    }
    tile_fold = __syncthreads_or(any) != 0;
  }
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    double fv[TN][4];
    int fok = 0;   // bit 4 j + r: entry (j, r) has a folded value
    if (tile_fold) {
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const int col = n0 + wn * WTN + j * 16 + (lane & 15);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = m0 + wm * WTM + i * 16 + M::row(lane, r);
          int f = -1, off = 0;
          if (col < d.n && row < d.m) {
            const int rb = row / 5, cb = col / 5;
            f = fm_s[(rb - rb0) * fcw + cb - cb0];
            off = (row - 5 * rb) * 5 + (col - 5 * cb);
          }
          fok |= (f >= 0 ? 1 : 0) << (4 * j + r);
          fv[j][r] = fval[(int64_t)(f >= 0 ? f : 0) * 25 + (f >= 0 ? off : 0)];
        }
      }
    }
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int col = n0 + wn * WTN + j * 16 + (lane & 15);
      if (col >= d.n) continue;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = m0 + wm * WTM + i * 16 + M::row(lane, r);
        if (row < d.m) {
          T *dst = c + (int64_t)row * d.ldc + col;
          T v = alpha * acc[i][j][r];
          if (PRE) v += old[PRE ? i : 0][PRE ? j : 0][r];
          else if (beta != T(0)) v += beta * (*dst);
          if ((fok >> (4 * j + r)) & 1) v = (T)((double)v + fv[j][r]);
          *dst = v;
        }
      }
    }
  }
}

template <typename T, int BM, int BN, int WM, int WN>
__global__ __launch_bounds__(64 * WM * WN) void gemm_batched_kernel(const GemmDesc *__restrict__ desc,
                                                                    const int32_t *__restrict__ tiles,
                                                                    const T *__restrict__ A, const T *__restrict__ B,
                                                                    T *__restrict__ C, T alpha, T beta,
                                                                    const int32_t *__restrict__ fmap,
                                                                    const double *__restrict__ fval) {
  gemm_tile<T, BM, BN, WM, WN, false>(desc, tiles, blockIdx.x, A, B, C, alpha, beta, fmap, fval);
}

template <int BM, int BN, int WM, int WN>
hipError_t launch_cfg(const GemmDesc *d_desc, const int32_t *d_tiles, int32_t n_tiles,
                      const void *a, const void *b, void *c, double alpha, double beta, bool fp32,
                      hipStream_t s, const int32_t *fmap, const double *fval) {
  const dim3 block(64 * WM * WN);
  if (fp32) {
    hipLaunchKernelGGL((gemm_batched_kernel<float, BM, BN, WM, WN>), dim3(n_tiles), block, 0, s,
                       d_desc, d_tiles, static_cast<const float *>(a), static_cast<const float *>(b),
                       static_cast<float *>(c), (float)alpha, (float)beta, fmap, fval);
  } else {
    hipLaunchKernelGGL((gemm_batched_kernel<double, BM, BN, WM, WN>), dim3(n_tiles), block, 0, s,
                       d_desc, d_tiles, static_cast<const double *>(a), static_cast<const double *>(b),
                       static_cast<double *>(c), alpha, beta, fmap, fval);
  }
  return hipGetLastError();
}

// C += alpha A B, a tile a workgroup; skip: not for problems with skip[desc.gate] set
template <typename T>
__global__ __launch_bounds__(256) void gemm_update_kernel(const GemmDesc *__restrict__ desc,
                                                          const int32_t *__restrict__ tiles, const T *__restrict__ A,
                                                          const T *__restrict__ B, T *__restrict__ C, T alpha,
                                                          const int32_t *__restrict__ skip) {
  if (skip != nullptr) {
    const int prob = tiles[3 * blockIdx.x];
    if (prob < 0 || skip[desc[prob].gate]) return;
  }
  gemm_tile<T, 64, 64, 2, 2, true>(desc, tiles, blockIdx.x, A, B, C, alpha, T(1), nullptr, nullptr);
}

// The same for the problems with only[desc.gate] set, mostly none (*any zero): a
// workgroup goes through every gridDim.x-th tile, so that a launch with nothing to do
// is small (62 000 workgroups that return at once take about 50 us).
template <typename T>
__global__ __launch_bounds__(256) void gemm_update_few_kernel(const GemmDesc *__restrict__ desc,
                                                              const int32_t *__restrict__ tiles, int n_tiles,
                                                              const T *__restrict__ A, const T *__restrict__ B,
                                                              T *__restrict__ C, T alpha,
                                                              const int32_t *__restrict__ only,
                                                              const int32_t *__restrict__ any) {
  if (!*any) return;
  for (int t = blockIdx.x; t < n_tiles; t += gridDim.x) {
    const int prob = tiles[3 * t];
    if (prob < 0 || !only[desc[prob].gate]) continue;
    gemm_tile<T, 64, 64, 2, 2, true>(desc, tiles, t, A, B, C, alpha, T(1), nullptr, nullptr);
    __syncthreads();                           // the next tile's slabs
  }
}

}  // namespace

// Tile configurations: C tile rows x columns and the wave grid.
//   0: 64x64 (2x2 waves)    1: 64x128 (2x2)    2: 128x128 (2x2)
//   3: 128x128 (2x4 waves)  4: 128x64 (2x2)    5: 240x80 (5x1; divides 1200 = n_c at N = 5)
//   6: 80x80 (5x1 waves)   7: 256x128 (4x2 waves)   8: 128x256 (2x4 waves)
void gemm_tile_shape(int cfg, int *bm, int *bn) {
  static const int shapes[kGemmConfigs][2] = {{64, 64}, {64, 128}, {128, 128}, {128, 128}, {128, 64},
                                              {240, 80}, {80, 80},          {256, 128}, {128, 256}};
  if (cfg < 0 || cfg >= kGemmConfigs) cfg = 0;
  *bm = shapes[cfg][0];
  *bn = shapes[cfg][1];
}

hipError_t launch_gemm_batched(int cfg, const GemmDesc *d_desc, const int32_t *d_tiles,
                               int32_t n_tiles, const void *a, const void *b, void *c, double alpha,
                               double beta, bool fp32, hipStream_t s, const int32_t *fold_map,
                               const double *fold_val) {
  if (n_tiles <= 0) return hipSuccess;
  switch (cfg) {
    case 1: return launch_cfg<64, 128, 2, 2>(d_desc, d_tiles, n_tiles, a, b, c, alpha, beta, fp32, s, fold_map, fold_val);
    case 2: return launch_cfg<128, 128, 2, 2>(d_desc, d_tiles, n_tiles, a, b, c, alpha, beta, fp32, s, fold_map, fold_val);
    case 3: return launch_cfg<128, 128, 2, 4>(d_desc, d_tiles, n_tiles, a, b, c, alpha, beta, fp32, s, fold_map, fold_val);
    case 4: return launch_cfg<128, 64, 2, 2>(d_desc, d_tiles, n_tiles, a, b, c, alpha, beta, fp32, s, fold_map, fold_val);
    case 5: return launch_cfg<240, 80, 5, 1>(d_desc, d_tiles, n_tiles, a, b, c, alpha, beta, fp32, s, fold_map, fold_val);
    case 6: return launch_cfg<80, 80, 5, 1>(d_desc, d_tiles, n_tiles, a, b, c, alpha, beta, fp32, s, fold_map, fold_val);
    case 7: return launch_cfg<256, 128, 4, 2>(d_desc, d_tiles, n_tiles, a, b, c, alpha, beta, fp32, s, fold_map, fold_val);
    case 8: return launch_cfg<128, 256, 2, 4>(d_desc, d_tiles, n_tiles, a, b, c, alpha, beta, fp32, s, fold_map, fold_val);
    default: return launch_cfg<64, 64, 2, 2>(d_desc, d_tiles, n_tiles, a, b, c, alpha, beta, fp32, s, fold_map, fold_val);
  }
}

// the updates of a factorisation, C += alpha A B with alpha = +-1: few slabs, so C's
// loads count and run beside the last slab's products (216 blocks of 1080 with K = 128:
// 1.51 -> 1.33 ms; on 128x128 tiles the values cost the second workgroup of a CU)
hipError_t launch_gemm_updates(const GemmDesc *d_desc, const int32_t *d_tiles, int32_t n_tiles, const void *a,
                               const void *b, void *c, double alpha, bool fp32, hipStream_t s, const int32_t *skip) {
  if (n_tiles <= 0) return hipSuccess;
  if (fp32)
    hipLaunchKernelGGL(gemm_update_kernel<float>, dim3(n_tiles), dim3(256), 0, s, d_desc, d_tiles,
                       static_cast<const float *>(a), static_cast<const float *>(b), static_cast<float *>(c),
                       (float)alpha, skip);
  else
    hipLaunchKernelGGL(gemm_update_kernel<double>, dim3(n_tiles), dim3(256), 0, s, d_desc, d_tiles,
                       static_cast<const double *>(a), static_cast<const double *>(b), static_cast<double *>(c), alpha,
                       skip);
  return hipGetLastError();
}

hipError_t launch_gemm_updates_few(const GemmDesc *d_desc, const int32_t *d_tiles, int32_t n_tiles, const void *a,
                                   const void *b, void *c, double alpha, bool fp32, hipStream_t s, const int32_t *only,
                                   const int32_t *any) {
  if (n_tiles <= 0) return hipSuccess;
  const dim3 grid(std::min(n_tiles, 2048));    // a multiple of the 8 XCDs: tiles stay on their XCD
  if (fp32)
    hipLaunchKernelGGL(gemm_update_few_kernel<float>, grid, dim3(256), 0, s, d_desc, d_tiles, n_tiles,
                       static_cast<const float *>(a), static_cast<const float *>(b), static_cast<float *>(c),
                       (float)alpha, only, any);
  else
    hipLaunchKernelGGL(gemm_update_few_kernel<double>, grid, dim3(256), 0, s, d_desc, d_tiles, n_tiles,
                       static_cast<const double *>(a), static_cast<const double *>(b), static_cast<double *>(c), alpha,
                       only, any);
  return hipGetLastError();
}

}  // namespace scdg
