// Dense direct solve of the condensed system S Q_b = b_S (the paper solves the
// condensed system with a direct LU solver; Section 4, Tables 'Advantages').
//
// S is assembled densely from A_bb and the element Schur blocks, its rows scaled
// by powers of two, and factored by right-looking blocked LU with row exchanges,
// 64 columns a panel.  Partial pivoting over a whole column is a search through
// n rows per column, one after another.  Here the pivots of a panel are first
// sought in its diagonal block alone (one workgroup, in registers), and the
// rows below then form their multipliers at once; the panel is accepted when
// every multiplier is at most kMaxMultiplier, and otherwise refactored with
// partial pivoting over all its rows:
//   diagonal block -> L21 and the test -> (whole-panel pivoting if rejected)
//   -> row exchanges, U12 = L11^-1 A12 -> A22 -= L21 U12 on the matrix cores.
// Bounded multipliers alone do not bound the entries, which can still grow by
// their product from panel to panel, so the rows of U of an accepted panel are
// measured too; above kMaxGrowth S is factored again, from the start, with partial
// pivoting in every panel (the host reads that flag with the zero-pivot one).
// The row-scaled S of flow systems has multipliers up to 2.3 and entries of U up
// to 1.04 at time steps to 1e-2, 4.5 and 1.3 at 0.1.
// The triangular solves take one launch per 64 x 64 diagonal block.
// Factor and solve with the steps around them: 75.0 -> 3.3 ms at n = 2240 and
// 681 -> 16.6 ms at n = 7560, against whole-column pivoting in one workgroup on
// 32-column panels and two barriers a column in the triangular solves; with
// every panel rejected 52 and 617 ms.
#include "internal.hpp"
#include "mfma.hpp"

namespace scdg {

namespace {

constexpr int kThreads = 256;
constexpr int kPanel = kDensePanel;
// largest multiplier accepted from pivots chosen inside a panel's diagonal block
// (2 is the bound of exact scaled pivoting up to the power-of-two scales), and
// largest entry of U beside them, on rows with largest entries in [1/2, 1)
constexpr double kMaxMultiplier = 4.0;
constexpr double kMaxGrowth = 4.0;

// remainder blocks of A_bb (those not folded into an element block)
__global__ void dense_fill_bb_kernel(int64_t n_bnodes, const int64_t *__restrict__ rowptr,
                                     const int32_t *__restrict__ col,
                                     const int32_t *__restrict__ src,
                                     const double *__restrict__ val, double *__restrict__ s,
                                     int64_t ld) {
  const int64_t g = blockIdx.x;
  if (g >= n_bnodes) return;
  for (int64_t b = rowptr[g]; b < rowptr[g + 1]; ++b) {
    const int64_t h = col[b];
    for (int q = threadIdx.x; q < 25; q += blockDim.x) {
      const int r = q / 5, w = q % 5;
      s[(5 * g + r) * ld + 5 * h + w] += val[(int64_t)src[b] * 25 + q];
    }
  }
}

// S[C_e, C_e] += T_e for one element (launched element after element so that
// overlapping entries are summed in a fixed order)
template <typename TM>
__global__ void dense_sub_elem_kernel(const TM *__restrict__ sloc, int nc,
                                      const int32_t *__restrict__ cmap, double *__restrict__ s,
                                      int64_t ld) {
  const int64_t n2 = (int64_t)nc * nc;
  for (int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; q < n2;
       q += (int64_t)gridDim.x * blockDim.x) {
    const int r = (int)(q / nc), c = (int)(q % nc);
    s[(int64_t)cmap[r] * ld + cmap[c]] += (double)sloc[q];
  }
}

__global__ void zero_kernel(double *__restrict__ x, int64_t n) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    x[i] = 0.0;
}

// S <- D S with D diagonal, powers of two that bring every row's largest entry
// to [1/2, 1): no rounding, and pivots are chosen on rows of one scale (scaled
// partial pivoting; the energy rows of S are about 1/((gamma - 1) Ma^2) larger
// than the others).  A zero or non-finite row keeps its scale.
__global__ __launch_bounds__(kThreads) void dense_scale_rows_kernel(double *__restrict__ a, int n,
                                                                    double *__restrict__ scale,
                                                                    int32_t *__restrict__ perm,
                                                                    int32_t *__restrict__ info) {
  __shared__ double red[kThreads / 64];
  double *row = a + (int64_t)blockIdx.x * n;
  double m = 0.0;
  for (int j = threadIdx.x; j < n; j += kThreads) m = fmax(m, fabs(row[j]));
  m = wave_max_dpp(m);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
  __syncthreads();
  m = fmax(fmax(red[0], red[1]), fmax(red[2], red[3]));
  const double f = (m > 0.0 && isfinite(m)) ? ldexp(1.0, max(-1000, min(1000, -ilogb(m) - 1))) : 1.0;
  for (int j = threadIdx.x; j < n; j += kThreads) row[j] *= f;
  if (threadIdx.x == 0) {
    scale[blockIdx.x] = f;
    perm[blockIdx.x] = blockIdx.x;
    if (blockIdx.x == 0) info[0] = info[1] = 0;
  }
}

// Inverses of the four 16 x 16 diagonal blocks of L (unit lower) and of U^T from
// an LU in LDS (pad: identity), into dinv[which][block][row][col], row-major:
// lane 16 q + c of wave `which` solves T y = e_c for block q; rd: reciprocals of
// the diagonal of U.
__device__ __forceinline__ void diagonal_inverses(const double (*__restrict__ lu)[kPanel + 2],
                                                  const double *__restrict__ rd, int which, int lane,
                                                  double *__restrict__ dinv) {
  const int q = lane >> 4, c = lane & 15, o = 16 * q;
  double y[16];
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    double v = r == c ? 1.0 : 0.0;
#pragma unroll
    for (int k = 0; k < r; ++k) v -= (which == 0 ? lu[o + r][o + k] : lu[o + k][o + r]) * y[k];
    y[r] = which == 0 ? v : v * rd[o + r];
    dinv[((which * 4 + q) * 16 + r) * 16 + c] = y[r];
  }
}

// Step 1 of a panel: LU of its diagonal block with partial pivoting among the
// block's own rows.  Lane r of every wave holds row r, wave q the columns
// 16 q .. 16 q + 15, all in registers.  The wave that holds column c finds the
// pivot by cross-lane reductions, leaves the multipliers and the pivot's lane in
// LDS and goes on with its own columns; the waves to its right follow one
// barrier behind, each taking the pivot row's entries from the pivot's lane.
// Rows do not move; blk gets them in pivot order, with the inverses of its 16 x 16
// diagonal blocks behind.
//   Bound by the chain of nbw column steps in one workgroup: 30 us for 64 columns
// (35 us with the search on FP64 keys and an IEEE division; 40 us with the
// column loop rolled, the owner's columns moving down one register per step).
__global__ __launch_bounds__(256) void dense_block_lu_kernel(const double *__restrict__ a, int n, int kb, int nbw,
                                                             double *__restrict__ blk,
                                                             int32_t *__restrict__ state) {
  __shared__ double l_s[2][kPanel];
  __shared__ int p_s[2];
  __shared__ double lu[kPanel][kPanel + 2];
  __shared__ double rd[kPanel];
  const int lane = threadIdx.x & 63, q = threadIdx.x >> 6;
  double x[16];
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    const int col = 16 * q + j;
    x[j] = (lane < nbw && col < nbw) ? a[(int64_t)(kb + lane) * n + kb + col] : (lane == col ? 1.0 : 0.0);
  }
  bool used = lane >= nbw, bad = false;
  int pos = lane;
#pragma unroll 1
  for (int owner = 0; owner < 4; ++owner) {
#pragma unroll
    for (int jj = 0; jj < 16; ++jj) {
      const int c = 16 * owner + jj, par = jj & 1;
      if (c < nbw) {
        int p = 0;
        if (q == owner) {
          // searched by sign-free high words (20 fraction bits: a pivot within 1e-6
          // of the largest, lowest row on ties; NaN and infinities win and are
          // rejected)
          const unsigned key = used ? 0u : (unsigned)__double2hiint(x[jj]) & 0x7fffffffu;
          p = __ffsll((long long)__ballot(key == wave_max_u32(key) && !used)) - 1;
          // taken with every lane active: the pivot's lane is not among `below`
          const double d = read_lane(x[jj], p);
          const double ad = fabs(d);
          const bool ok = ad > 1e-280 && ad < 1e280;
          const double inv = ok ? fast_reciprocal(d) : 1.0;
          const bool below = !used && lane != p;
          const double l = below ? x[jj] * inv : 0.0;
          if (below) x[jj] = l;
          bad = bad || !ok || !(fabs(l) <= kMaxMultiplier);
          l_s[par][lane] = l;
          if (lane == 0) {
            p_s[par] = p;
            rd[c] = inv;
          }
#pragma unroll
          for (int j = jj + 1; j < 16; ++j) x[j] -= l * read_lane(x[j], p);
        }
        __syncthreads();
        if (q != owner) p = __builtin_amdgcn_readfirstlane(p_s[par]);
        if (q > owner) {
          const double l = l_s[par][lane];
#pragma unroll
          for (int j = 0; j < 16; ++j) x[j] -= l * read_lane(x[j], p);
        }
        if (lane == p) {
          used = true;
          pos = c;
        }
      }
    }
  }
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    lu[pos][16 * q + j] = x[j];
    blk[pos * kPanel + 16 * q + j] = x[j];
  }
  if (q == 0) {
    state[pos] = lane;
    if (lane >= nbw) rd[lane] = 1.0;
  }
  const int any = __syncthreads_or(bad);
  if (threadIdx.x == 0) state[kPanel] = any ? 1 : 0;
  if (q < 2) diagonal_inverses(lu, rd, q, lane, blk + kPanel * kPanel);
}

// Steps 2 and 4: triangular solves with the panel's diagonal block on the matrix
// cores, 16 x 16 blocks, X_i = T_ii^-1 (B_i - sum_{j<i} T_ij X_j).  Each of the
// four waves holds 16 columns of B (64 x 16) as four accumulators; the rows a
// lane holds of an accumulator are the ones it supplies as the next product's
// operand, so X_j never leaves its registers.
//   A wave's 40 products take under 2 us; what is left is the launch and the
// latency of the loads.  One row or column per lane with T from LDS took 64 us a
// launch for U12 and, spilling, 91 us for L21 at n = 7560.
__device__ __forceinline__ void solve_lower_16(const double (*__restrict__ t)[kPanel + 2], f64x4 (&x)[4], int lane) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
#pragma unroll
    for (int j = 0; j < i; ++j)
#pragma unroll
      for (int s = 0; s < 4; ++s)
        x[i] = Mfma<double>::mma(-t[16 * i + (lane & 15)][16 * j + 4 * s + (lane >> 4)], x[j][s], x[i]);
    f64x4 y = Mfma<double>::zero();
#pragma unroll
    for (int s = 0; s < 4; ++s)
      y = Mfma<double>::mma(t[16 * i + (lane & 15)][16 * i + 4 * s + (lane >> 4)], x[i][s], y);
    x[i] = y;
  }
}

// T = L11 (which = 0) or U11^T (1) into LDS, its diagonal blocks inverted; the
// loads are all in flight together
__device__ __forceinline__ void load_triangle(const double *__restrict__ blk, int which, double (*__restrict__ t)[kPanel + 2]) {
  double v[kPanel * kPanel / 256];
#pragma unroll
  for (int u = 0; u < kPanel * kPanel / 256; ++u) {
    const int q = threadIdx.x + 256 * u, r = q / kPanel, c = q % kPanel;
    v[u] = r / 16 == c / 16 ? blk[kPanel * kPanel + (which * 4 + r / 16) * 256 + (r % 16) * 16 + c % 16] : blk[q];
  }
#pragma unroll
  for (int u = 0; u < kPanel * kPanel / 256; ++u) {
    const int q = threadIdx.x + 256 * u, r = q / kPanel, c = q % kPanel;
    if (which == 0 || r / 16 == c / 16) t[r][c] = v[u];
    else t[c][r] = v[u];
  }
}

// Step 2: L21 = A21 U11^-1 for the rows below the diagonal block (as U11^T
// L21^T = A21^T), 64 rows a workgroup, into lbuf; raises state[kPanel] when a
// multiplier exceeds kMaxMultiplier or is not a number.
__global__ __launch_bounds__(256) void dense_l21_kernel(const double *__restrict__ a, int n, int kb,
                                                        const double *__restrict__ blk, double *__restrict__ lbuf,
                                                        int32_t *__restrict__ state) {
  __shared__ double t[kPanel][kPanel + 2];
  const int lane = threadIdx.x & 63, row = kb + kPanel + blockIdx.x * 64 + 16 * (threadIdx.x >> 6) + (lane & 15);
  f64x4 x[4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r)
      x[i][r] = row < n ? a[(int64_t)row * n + kb + 16 * i + Mfma<double>::row(lane, r)] : 0.0;
  load_triangle(blk, 1, t);
  __syncthreads();
  solve_lower_16(t, x, lane);
  if (row >= n) return;
  bool ok = true;
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      ok = ok && fabs(x[i][r]) <= kMaxMultiplier;
      lbuf[(int64_t)row * kPanel + 16 * i + Mfma<double>::row(lane, r)] = x[i][r];
    }
  if (!ok) state[kPanel] = 1;                        // every writer stores 1
}

// Step 3, when the diagonal block's own pivots were rejected (otherwise it
// returns at once) or are not to be tried (whole): the panel a[kb:n, kb:kb+nbw] with partial pivoting over all
// its rows, in place, in one workgroup, 32 columns at a time and then their update
// of the others (every column step reads and writes the columns it updates, a row a
// thread: 64 columns at once cost twice the memory traffic); the swaps go to state,
// the results to blk and lbuf, and the rows of prev (the pair's first panel's
// lbuf, or null) move with them.
__global__ __launch_bounds__(1024) void dense_panel_lu_kernel(double *__restrict__ a, int n, int kb, int nbw,
                                                              double *__restrict__ blk, double *__restrict__ lbuf,
                                                              double *__restrict__ prev, int32_t *__restrict__ state,
                                                              int32_t *__restrict__ perm,
                                                              int32_t *__restrict__ info, bool whole) {
  constexpr int NT = 1024, kSub = kPanel / 2;
  // info[1]: S is factored again anyway (the row indexes left in state stay below n)
  if (!whole && (state[kPanel] == 0 || info[1] != 0)) return;
  __shared__ double red_v[NT / 64];
  __shared__ int red_i[NT / 64];
  __shared__ double pivot_row[kPanel];
  __shared__ double lu[kPanel][kPanel + 2];
  __shared__ double rd[kPanel];
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  for (int c = 0; c < nbw; ++c) {
    const int k = kb + c, end = c < kSub ? min(nbw, kSub) : nbw;
    double best = -1.0;
    int bi = n;
    for (int i = k + tid; i < n; i += NT) {
      const double v = fabs(a[(int64_t)i * n + k]);
      if (v > best) {
        best = v;
        bi = i;
      }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
      const double ov = __shfl_xor(best, off);
      const int oi = __shfl_xor(bi, off);
      if (ov > best || (ov == best && oi < bi)) {
        best = ov;
        bi = oi;
      }
    }
    if (lane == 0) {
      red_v[wid] = best;
      red_i[wid] = bi;
    }
    __syncthreads();
    best = red_v[0];
    bi = red_i[0];
    for (int w = 1; w < NT / 64; ++w)
      if (red_v[w] > best || (red_v[w] == best && red_i[w] < bi)) {
        best = red_v[w];
        bi = red_i[w];
      }
    const int pr = (bi < n) ? bi : k;
    if (tid < nbw && pr != k) {
      const int j = kb + tid;
      const double t = a[(int64_t)k * n + j];
      a[(int64_t)k * n + j] = a[(int64_t)pr * n + j];
      a[(int64_t)pr * n + j] = t;
    }
    if (prev != nullptr && tid >= 64 && tid < 64 + kPanel && pr != k) {
      const int j = tid - 64;
      const double t = prev[(int64_t)k * kPanel + j];
      prev[(int64_t)k * kPanel + j] = prev[(int64_t)pr * kPanel + j];
      prev[(int64_t)pr * kPanel + j] = t;
    }
    if (tid == 0) {
      state[c] = pr;
      const int32_t t = perm[k];
      perm[k] = perm[pr];
      perm[pr] = t;
    }
    __syncthreads();
    if (tid < nbw) pivot_row[tid] = a[(int64_t)k * n + kb + tid];
    __syncthreads();
    double d = pivot_row[c];
    if (!(d != 0.0) || !isfinite(d)) {
      if (tid == 0 && info[0] == 0) info[0] = k + 1;
      d = 1.0;
    }
    const double inv_d = 1.0 / d;
    for (int i = k + 1 + tid; i < n; i += NT) {
      double *row = a + (int64_t)i * n;
      const double l = row[k] * inv_d;
      row[k] = l;
      for (int j = c + 1; j < end; ++j) row[kb + j] -= l * pivot_row[j];
    }
    __syncthreads();
    if (c != kSub - 1 || nbw <= kSub) continue;
    // the second half's columns: U12 (into the second half of lu) from L11, then the rows below
    for (int q = tid; q < kSub * kSub; q += NT) lu[q / kSub][q % kSub] = a[(int64_t)(kb + q / kSub) * n + kb + q % kSub];
    __syncthreads();
    if (tid < nbw - kSub) {
      double x[kSub];
#pragma unroll
      for (int r = 0; r < kSub; ++r) {
        double *at = a + (int64_t)(kb + r) * n + kb + kSub + tid;
        double v = *at;
#pragma unroll
        for (int q = 0; q < r; ++q) v -= lu[r][q] * x[q];
        x[r] = v;
        *at = v;
        lu[kSub + r][tid] = v;
      }
    }
    __syncthreads();
    for (int i = kb + kSub + tid; i < n; i += NT) {
      double *row = a + (int64_t)i * n + kb;
      double l[kSub];
#pragma unroll
      for (int q = 0; q < kSub; ++q) l[q] = row[q];
      for (int j = kSub; j < nbw; ++j) {
        double v = row[j];
#pragma unroll
        for (int q = 0; q < kSub; ++q) v -= l[q] * lu[kSub + q][j - kSub];
        row[j] = v;
      }
    }
    __syncthreads();
  }
  for (int q = tid; q < kPanel * kPanel; q += NT) {
    const int r = q / kPanel, cc = q % kPanel;
    const double v = (r < nbw && cc < nbw) ? a[(int64_t)(kb + r) * n + kb + cc] : (r == cc ? 1.0 : 0.0);
    lu[r][cc] = v;
    blk[q] = v;
    if (r == cc) rd[r] = 1.0 / v;
  }
  for (int64_t q = tid; q < (int64_t)(n - kb - nbw) * nbw; q += NT) {
    const int64_t i = kb + nbw + q / nbw;
    lbuf[i * kPanel + q % nbw] = a[i * n + kb + q % nbw];
  }
  if (tid == 0) state[kPanel] = 1;             // read by every thread before the first barrier
  __syncthreads();
  if (wid < 2) diagonal_inverses(lu, rd, wid, lane, blk + kPanel * kPanel);
}

// Step 4: the row exchanges on the columns outside the panel, U12 = L11^-1 A12
// on those right of it, 64 columns a workgroup, and the panel's own columns from
// blk and lbuf.  The second panel of a pair first takes the first one's update
// from its rows (prev: the first panel's lbuf, whose rows are in the order of
// before this panel's exchanges unless those are swaps; its U12 is in the 64 rows
// above): until then rows inside and outside the panel have the same updates, so
// that they can be exchanged.  Grid: ceil(n / 64) workgroups; the one at the panel writes its
// diagonal block, one right of it also the rows of L21 that its index names.
// After step 3 the exchanges are a list of swaps and the panel is in place, else
// they are a permutation of the panel's rows and entries of U above kMaxGrowth
// raise info[1].
__global__ __launch_bounds__(256) void dense_u12_kernel(double *__restrict__ a, int n, int kb, int nbw,
                                                        const double *__restrict__ blk,
                                                        const double *__restrict__ lbuf,
                                                        const double *__restrict__ prev,
                                                        const int32_t *__restrict__ state,
                                                        int32_t *__restrict__ perm, int32_t *__restrict__ info) {
  __shared__ double t[kPanel][kPanel + 2];
  const int tid = threadIdx.x, lane = tid & 63;
  const int j0 = blockIdx.x * 64, j = j0 + 16 * (tid >> 6) + (lane & 15);
  const bool swaps = state[kPanel] != 0;
  if (j0 == kb) {
    if (swaps) return;
    const int src = tid < nbw ? perm[kb + state[tid]] : 0;
    __syncthreads();
    if (tid < nbw) perm[kb + tid] = src;
    bool ok = true;
    for (int q = tid; q < nbw * nbw; q += 256) {
      const double v = blk[(q / nbw) * kPanel + q % nbw];
      ok = ok && (q % nbw < q / nbw || fabs(v) <= kMaxGrowth);
      a[(int64_t)(kb + q / nbw) * n + kb + q % nbw] = v;
    }
    if (!ok) info[1] = 1;                            // every writer stores 1
    return;
  }
  if (j0 > kb && !swaps) {
    const int rows = min(64, n - j0);
    double v[kPanel / 4];
#pragma unroll
    for (int u = 0; u < kPanel / 4; ++u)
      v[u] = tid + 256 * u < rows * kPanel ? lbuf[(int64_t)j0 * kPanel + tid + 256 * u] : 0.0;
#pragma unroll
    for (int u = 0; u < kPanel / 4; ++u)
      if (tid + 256 * u < rows * kPanel)
        a[(int64_t)(j0 + (tid + 256 * u) / kPanel) * n + kb + tid % kPanel] = v[u];
  }
  if (swaps) {
    if (tid < 64 && j0 + tid < n)
      for (int c = 0; c < nbw; ++c) {
        const int64_t k = (int64_t)(kb + c) * n + j0 + tid, pr = (int64_t)state[c] * n + j0 + tid;
        if (pr != k) {
          const double v = a[k];
          a[k] = a[pr];
          a[pr] = v;
        }
      }
    __syncthreads();
  }
  f64x4 x[4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int m = 16 * i + Mfma<double>::row(lane, r);
      const int src = swaps ? m : state[m];
      x[i][r] = (m < nbw && j < n) ? a[(int64_t)(kb + src) * n + j] : 0.0;
    }
  if (j0 > kb) {                                     // nbw = kPanel: columns remain right of the panel
    if (prev != nullptr) {
      double v[kPanel / 4], u[kPanel / 4];
#pragma unroll
      for (int s = 0; s < kPanel / 4; ++s) {
        const int m = 4 * s + (tid >> 6);
        v[s] = prev[(int64_t)(kb + (swaps ? m : state[m])) * kPanel + lane];
      }
#pragma unroll
      for (int s = 0; s < kPanel / 4; ++s)
        u[s] = j < n ? a[(int64_t)(kb - kPanel + 4 * s + (lane >> 4)) * n + j] : 0.0;
#pragma unroll
      for (int s = 0; s < kPanel / 4; ++s) t[4 * s + (tid >> 6)][lane] = v[s];
      __syncthreads();
#pragma unroll
      for (int s = 0; s < kPanel / 4; ++s)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          x[i] = Mfma<double>::mma(-t[16 * i + (lane & 15)][4 * s + (lane >> 4)], u[s], x[i]);
      __syncthreads();
    }
    load_triangle(blk, 0, t);
    __syncthreads();
    solve_lower_16(t, x, lane);
  }
  bool ok = true;
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int m = 16 * i + Mfma<double>::row(lane, r);
      if (m < nbw && j < n) {
        a[(int64_t)(kb + m) * n + j] = x[i][r];
        ok = ok && fabs(x[i][r]) <= kMaxGrowth;
      }
    }
  if (!ok && !swaps && j0 > kb) info[1] = 1;
}

__global__ void dense_permute_kernel(const double *__restrict__ b, const double *__restrict__ scale,
                                     const int32_t *__restrict__ perm, double *__restrict__ w, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) w[i] = scale[perm[i]] * b[perm[i]];
}

// One step of a triangular solve with LU: every workgroup solves the 64 x 64
// diagonal block for itself (lane r holds row r; the chain of 64 steps is the
// bound), then subtracts its product with the block column (UPPER: block rows
// above, else below) from 64 entries of w.  The first workgroup keeps the
// solution.  One launch per block in place of two barriers per column.
template <bool UPPER>
__global__ __launch_bounds__(256) void dense_tri_step_kernel(const double *__restrict__ lu, int n, int kb, int nbw,
                                                             double *__restrict__ w, double *__restrict__ out) {
  __shared__ double xs[kPanel];
  const int tid = threadIdx.x, lane = tid & 63;
  const int r_end = UPPER ? kb : n;
  const int row = (UPPER ? 0 : kb + nbw) + blockIdx.x * 64 + (tid >> 2);
  const int c0 = (tid & 3) * (kPanel / 4);
  double m[kPanel / 4];
#pragma unroll
  for (int c = 0; c < kPanel / 4; ++c)
    m[c] = (row < r_end && c0 + c < nbw) ? lu[(int64_t)row * n + kb + c0 + c] : 0.0;
  if (tid < 64) {
    double v = lane < nbw ? w[kb + lane] : 0.0;
    const double *t = lu + (int64_t)(kb + min(lane, nbw - 1)) * n + kb;
    double tr[kPanel];
#pragma unroll
    for (int c = 0; c < kPanel; ++c) tr[c] = c < nbw ? t[c] : 0.0;
    if (UPPER) {
      const double inv = 1.0 / t[min(lane, nbw - 1)];
#pragma unroll
      for (int c = kPanel - 1; c >= 0; --c) {
        if (c < nbw) {
          if (lane == c) v *= inv;
          const double xc = read_lane(v, c);
          if (lane < c) v -= tr[c] * xc;
        }
      }
    } else {
#pragma unroll
      for (int c = 0; c < kPanel; ++c) {
        const double xc = read_lane(v, c);
        if (lane > c) v -= tr[c] * xc;
      }
    }
    if (lane >= nbw) v = 0.0;
    xs[lane] = v;
    if (blockIdx.x == 0 && lane < nbw) out[kb + lane] = v;
  }
  __syncthreads();
  double s = 0.0;
#pragma unroll
  for (int c = 0; c < kPanel / 4; ++c) s += m[c] * xs[c0 + c];
  s += dpp_mov<0xB1>(s);
  s += dpp_mov<0x4E>(s);
  if ((tid & 3) == 0 && row < r_end) w[row] -= s;
}

}  // namespace

hipError_t launch_dense_assemble(const Plan &p, double *s) {
  const int64_t n = p.n1;
  hipLaunchKernelGGL(zero_kernel, dim3(2048), dim3(kThreads), 0, p.stream, s, n * n);
  hipLaunchKernelGGL(dense_fill_bb_kernel, dim3((unsigned)p.n_bnodes), dim3(32), 0, p.stream,
                     p.n_bnodes, p.d_rem_rowptr, p.d_rem_col, p.d_rem_src, p.bb_val, s, n);
  const bool fp32 = p.prec == SCDG_FP32;
  const size_t esz = fp32 ? sizeof(float) : sizeof(double);
  for (int e = 0; e < p.n_elem; ++e) {
    const int nc = p.nc[e];
    const char *base = static_cast<const char *>(p.sloc) + esz * p.off_cc[e];
    const int grid = (int)std::min<int64_t>(1024, ((int64_t)nc * nc + kThreads - 1) / kThreads);
    if (fp32)
      hipLaunchKernelGGL(dense_sub_elem_kernel<float>, dim3(grid), dim3(kThreads), 0, p.stream,
                         reinterpret_cast<const float *>(base), nc, p.d_cmap + p.off_c[e], s, n);
    else
      hipLaunchKernelGGL(dense_sub_elem_kernel<double>, dim3(grid), dim3(kThreads), 0, p.stream,
                         reinterpret_cast<const double *>(base), nc, p.d_cmap + p.off_c[e], s, n);
  }
  return hipGetLastError();
}

// work arrays of the dense path, kept with the plan (S has one size per plan)
static hipError_t dense_work(Plan &p) {
  if (p.d_dense_desc) return hipSuccess;
  const int32_t n = (int32_t)p.n1;
  auto get = [](auto **ptr, size_t count) {
    return *ptr ? hipSuccess : hipMalloc(reinterpret_cast<void **>(ptr), sizeof(**ptr) * count);
  };
  hipError_t err = get(&p.s_dense, (size_t)n * n);
  if (err == hipSuccess) err = get(&p.dl_scale, (size_t)n);
  if (err == hipSuccess) err = get(&p.dl_lbuf, (size_t)2 * n * kPanel);
  if (err == hipSuccess) err = get(&p.dl_blk, (size_t)kPanel * kPanel + 2 * 4 * 16 * 16);
  if (err == hipSuccess) err = get(&p.dl_x, (size_t)2 * n);
  if (err == hipSuccess) err = get(&p.dl_perm, (size_t)n);
  if (err == hipSuccess) err = get(&p.dl_state, (size_t)kPanel + 1);
  if (err == hipSuccess) err = get(&p.d_dense_info, (size_t)2);
  if (err != hipSuccess) return err;
  // per pair of panels: the first panel's update of the second's columns, and the
  // pair's update of the rest
  std::vector<GemmDesc> descs;
  for (int kb = 0; kb < n; kb += 2 * kPanel) {
    const int k1 = std::min(n, kb + kPanel), k2 = std::min(n, kb + 2 * kPanel);
    auto at = [n](int64_t r, int64_t c) { return r * n + c; };
    descs.push_back(GemmDesc{at(k1, kb), at(kb, k1), at(k1, k1), n - k1, k2 - k1, k1 - kb, n, n, n});
    descs.push_back(GemmDesc{at(k2, kb), at(kb, k2), at(k2, k2), n - k2, n - k2, k2 - kb, n, n, n});
  }
  GemmDesc *d = nullptr;
  err = hipMalloc(&d, sizeof(GemmDesc) * descs.size());
  if (err != hipSuccess) return err;
  err = hipMemcpy(d, descs.data(), sizeof(GemmDesc) * descs.size(), hipMemcpyHostToDevice);
  if (err != hipSuccess) {
    (void)hipFree(d);
    return err;
  }
  p.d_dense_desc = d;
  return hipSuccess;
}

// whole: partial pivoting over all rows in every panel
hipError_t launch_dense_lu(Plan &p, bool whole) {
  hipError_t err = dense_work(p);
  if (err != hipSuccess) return err;
  err = launch_dense_assemble(p, p.s_dense);
  if (err != hipSuccess) return err;
  const int32_t n = (int32_t)p.n1;
  double *a = p.s_dense;
  hipLaunchKernelGGL(dense_scale_rows_kernel, dim3(n), dim3(kThreads), 0, p.stream, a, n, p.dl_scale, p.dl_perm,
                     p.d_dense_info);
  // Panels in pairs: the first's update goes at once only to the second's columns
  // (and with the second's exchanges to its rows), so the rest of S is read and
  // written once per pair.
  auto update = [&](int which, int kb, int m, int nn) {
    if (m <= 0 || nn <= 0 || err != hipSuccess) return;
    // 64x64 tiles: n = 7560 takes 16.6 ms for the solve, 18.7 with 128x128 from 512 rows on
    err = launch_gemm_updates(p.d_dense_desc + 2 * (kb / (2 * kPanel)) + which, nullptr,
                              ((m + 63) / 64) * ((nn + 63) / 64), a, a, a, -1.0, false, p.stream);
  };
  auto panel = [&](int kb, double *lbuf, double *prev) {
    const int nbw = std::min(kPanel, n - kb), rest = n - kb - nbw;
    if (nbw <= 0 || err != hipSuccess) return;
    if (!whole)
      hipLaunchKernelGGL(dense_block_lu_kernel, dim3(1), dim3(256), 0, p.stream, a, n, kb, nbw, p.dl_blk, p.dl_state);
    if (!whole && rest > 0)
      hipLaunchKernelGGL(dense_l21_kernel, dim3((rest + 63) / 64), dim3(256), 0, p.stream, a, n, kb, p.dl_blk,
                         lbuf, p.dl_state);
    hipLaunchKernelGGL(dense_panel_lu_kernel, dim3(1), dim3(1024), 0, p.stream, a, n, kb, nbw, p.dl_blk, lbuf, prev,
                       p.dl_state, p.dl_perm, p.d_dense_info, whole);
    hipLaunchKernelGGL(dense_u12_kernel, dim3((n + 63) / 64), dim3(256), 0, p.stream, a, n, kb, nbw, p.dl_blk,
                       lbuf, prev, p.dl_state, p.dl_perm, p.d_dense_info);
    err = hipGetLastError();
  };
  for (int kb = 0; kb < n && err == hipSuccess; kb += 2 * kPanel) {
    const int k1 = std::min(n, kb + kPanel), k2 = std::min(n, kb + 2 * kPanel);
    panel(kb, p.dl_lbuf, nullptr);
    update(0, kb, n - k1, k2 - k1);
    panel(k1, p.dl_lbuf + (int64_t)n * kPanel, p.dl_lbuf);
    update(1, kb, n - k2, n - k2);
  }
  return err;
}

hipError_t launch_dense_solve(Plan &p, const double *b, double *x) {
  const int32_t n = (int32_t)p.n1;
  const int last = (n - 1) / kPanel * kPanel;
  double *w = p.dl_x, *y = p.dl_x + n;
  hipLaunchKernelGGL(dense_permute_kernel, dim3((n + kThreads - 1) / kThreads), dim3(kThreads), 0, p.stream, b,
                     p.dl_scale, p.dl_perm, w, n);
  for (int kb = 0; kb < n; kb += kPanel) {
    const int nbw = std::min(kPanel, n - kb), rest = n - kb - nbw;
    hipLaunchKernelGGL(dense_tri_step_kernel<false>, dim3(std::max(1, (rest + 63) / 64)), dim3(256), 0, p.stream,
                       p.s_dense, n, kb, nbw, w, y);
  }
  for (int kb = last; kb >= 0; kb -= kPanel) {
    const int nbw = std::min(kPanel, n - kb);
    hipLaunchKernelGGL(dense_tri_step_kernel<true>, dim3(std::max(1, kb / 64)), dim3(256), 0, p.stream, p.s_dense, n,
                       kb, nbw, y, x);
  }
  return hipGetLastError();
}

}  // namespace scdg
