// Centre hop by Cholesky factorisation of the Gram matrix (LDS-resident, FP64).
//
// Left-to-right hop of the orthogonality centre from site j to j+1: C_j (rows (a,s), n = chi_R
// columns) = Q R with E = C^dag C = R^dag R (upper-triangular R); R is written out for
// C_{j+1} = R B_{j+1}, inverted in place in LDS, and Q = C R^{-1} replaces C_j in place.
// Right-to-left hop from j to j-1: C_j (n = chi_L rows, 2 chi_R columns) = R^dag Q with
// E = C C^dag = R^dag R; R is written out for C_{j-1} = A_{j-1} R^dag and Q = R^{-dag} C
// replaces C_j.  The products with R^{-1} run on f64 MFMA over its nonzero triangle (a
// triangular solve per vector spent most of its time moving broadcasts, not computing).
// Pivots below tol * max(diag E) are dropped (the row of R and the row and column of R^{-1}
// become zero): such directions carry no weight of the state.
#include "common.h"
#include "kernels.h"

namespace mpsb {

typedef double v4d_t __attribute__((ext_vector_type(4)));
__device__ inline v4d_t mfma64(double a, double b, v4d_t c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }

__device__ inline int pk(int i, int k, int n) { return i * n - (i * (i - 1)) / 2 + (k - i); }   // packed upper

__device__ inline double lane_f64(double x, int l) {   // the value of lane l (uniform) in every lane
  const long long b = __double_as_longlong(x);
  const int lo = __builtin_amdgcn_readlane((int)b, l), hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// LDS written by a wave is read by the same wave: no workgroup barrier
__device__ inline void wave_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// lane L of each row of 16 lanes, in every lane of the row (DPP row_newbcast)
template <int L>
__device__ inline double row_bcast(double x) {
  const long long b = __double_as_longlong(x);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)b, 0x150 + L, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), 0x150 + L, 0xf, 0xf, false);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// column JJ of the inverse of a 16 x 16 upper triangle, row ii in the lane's x[], from the
// columns before it: x[JJ] = -dj sum_l x[l] R[l][JJ], R[l][JJ] still in lane l's x[JJ]
template <int JJ, int L>
__device__ inline void inv_sum(const c64d (&x)[16], double (&re)[2], double (&im)[2]) {
  if constexpr (L < JJ) {
    const c64d t{row_bcast<L>(x[JJ].re), row_bcast<L>(x[JJ].im)};
    re[L & 1] = fma(x[L].re, t.re, re[L & 1]);
    re[L & 1] = fma(-x[L].im, t.im, re[L & 1]);
    im[L & 1] = fma(x[L].re, t.im, im[L & 1]);
    im[L & 1] = fma(x[L].im, t.re, im[L & 1]);
    inv_sum<JJ, L + 1>(x, re, im);
  }
}
template <int JJ>
__device__ inline void inv_cols(c64d (&x)[16], int ii, int nc, const double* ipiv) {   // columns JJ .. nc - 1
  if constexpr (JJ < 16) {
    if (JJ >= nc) return;
    const double dj = ipiv[JJ];
    double re[2] = {0, 0}, im[2] = {0, 0};
    inv_sum<JJ, 0>(x, re, im);
    if (ii < JJ) x[JJ] = c64d{-dj * (re[0] + re[1]), -dj * (im[0] + im[1])};
    if (ii == JJ) x[JJ] = c64d{dj, 0.0};
    inv_cols<JJ + 1>(x, ii, nc, ipiv);
  }
}

// What bounds it: chains of dependent steps (pivot, square root, divisions, row updates) at one
// workgroup per CU for n > 96, where the packed triangle fills the LDS.  A panel of 8 rows of the
// Cholesky factor is therefore held in the registers of one wave (a lane owns one or two columns,
// pivots and multipliers by readlane: no barrier and no LDS between its columns) while the other
// waves apply the previous panel's update to the rows past it; the instances for smaller n leave
// room for several workgroups per CU.  Every element's operations and their order are those of
// the column-by-column form (two barriers per column, one instance for all n), bit for bit.
// Per launch (FP64, 2 n rows), that form -> this one: 15 trajectories of n = 1 7.1 -> 5.2 us, n = 4
// 9.8 -> 6.4 (the ends of every chain; 11.4 and 11.8 with every column of a panel and of a diagonal
// block worked through), n = 32 58 -> 37, n = 64 116 -> 79, n = 128 333 -> 252; 512 of n = 64
// 231 -> 117, n = 100 529 -> 419; 2048 of n = 16 234 -> 51, n = 32 435 -> 116, n = 128 2905 -> 2230.
// At n = 128 a workgroup spends a third of that in the product with R^-1 (two thirds of its
// matrix-core time), a quarter in the panels and a fifth in the inverse's block columns.
// Registers: 128 up to 64 columns, for four workgroups per CU (160 without the spills: 15 of
// n = 64 84 -> 79 us, but 1024 of n = 40 97 -> 116); 224 at 96, whose eight waves then fill a CU
// alone although its LDS would admit two workgroups (at 128 registers and 0.5 KB of scratch -> 224,
// FP32 / FP64: 15 of n = 96 258 / 237 -> 158 / 153 us, 2048 1754 / 1798 -> 1361 / 1405; only FP32 of
// 65 to 80 columns gains by the second workgroup, 512 of n = 72 223 against 233).
template <typename T, int NMAX, int HT>
__global__ __launch_bounds__(HT, NMAX > 64 ? 2 : 4) void k_hop_chol(int n, int left_to_right, int other, const c64d* __restrict__ Eg,
                                                 long long sE, cplx<T>* __restrict__ C, long long sC,
                                                 cplx<T>* __restrict__ Rout, long long sR, double tol) {
  __shared__ c64d R[NMAX * (NMAX + 1) / 2];
  __shared__ double piv[NMAX], ipiv[NMAX];   // pivots R[c][c] and their inverses (0 if dropped)
  __shared__ double red[HT / 64];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const c64d* E = Eg + blockIdx.x * sE;
  cplx<T>* Cj = C + blockIdx.x * sC;
  cplx<T>* Ro = Rout + blockIdx.x * sR;
  // load the upper triangle, find max diagonal
  double dm = 0;
  for (int i = wv; i < n; i += HT / 64)
    for (int k = i + lane; k < n; k += 64) {
      c64d v = E[(long long)i * n + k];
      R[pk(i, k, n)] = v;
      if (k == i) dm = fmax(dm, v.re);
    }
  for (int off = 32; off > 0; off >>= 1) dm = fmax(dm, __shfl_down(dm, off, 64));
  if (lane == 0) red[wv] = dm;
  __syncthreads();
  double dmax = 0;
  for (int w = 0; w < HT / 64; ++w) dmax = fmax(dmax, red[w]);
  const double cut = tol * dmax;
  // blocked right-looking Cholesky E = R^dag R in panels of CB rows: the first wave factors the
  // rows c0 .. c0+cb-1 (updated by every earlier panel) in registers, lane l owning columns l
  // and l + 64
  constexpr int CB = 8, KS = (NMAX + 63) / 64;
  auto factor = [&](int c0) {
    c64d v[CB][KS];   // rows past n are zero: no pivot
#pragma unroll
    for (int a = 0; a < CB; ++a)
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        const int i = c0 + a, k = lane + 64 * s;
        v[a][s] = (k >= i && k < n) ? R[pk(i, k, n)] : c64d{0, 0};
      }
    const int l0 = c0 & 63;
    const bool up = KS > 1 && c0 >= 64;    // the panel's own columns are in the second set
#pragma unroll
    for (int a = 0; a < CB; ++a) {
      if (NMAX <= 64 && c0 + a >= n) break;   // (n < 8 mostly: at 65 columns and more the test costs 2%)
      const c64d own = up ? v[a][KS - 1] : v[a][0];
      const double p = lane_f64(own.re, l0 + a);
      const bool keep = p > cut && p > 0.0;
      const double r = keep ? sqrt(p) : 0.0;
      if (lane == 0) piv[c0 + a] = r;
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        const c64d x = v[a][s];
        v[a][s] = keep ? c64d{x.re / r, x.im / r} : c64d{0, 0};
      }
      // rows c+1 .. of the panel: E[i][k] -= conj(R[c][i]) R[c][k] (nothing for a dropped pivot,
      // whose row is zero)
      const c64d row = up ? v[a][KS - 1] : v[a][0];
#pragma unroll
      for (int b = a + 1; b < CB; ++b) {
        const c64d f{lane_f64(row.re, l0 + b), lane_f64(row.im, l0 + b)};
#pragma unroll
        for (int s = 0; s < KS; ++s) v[b][s] = v[b][s] - cmulc(f, v[a][s]);
      }
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        const int i = c0 + a, k = lane + 64 * s;
        if (k >= i && k < n) R[pk(i, k, n)] = k == i ? c64d{r, 0.0} : v[a][s];
      }
    }
  };
  if (wv == 0) factor(0);
  __syncthreads();
  for (int c0 = 0; c0 + CB < n; c0 += CB) {
    // the panel's update of the rows t0 .. n-1: first the rows of the next panel by every
    // wave, a row at a time, then the rest in 4 x 4 register tiles while the first wave
    // factors that panel
    const int t0 = c0 + CB;
    for (int i = t0 + wv; i < min(t0 + CB, n); i += HT / 64)
      for (int k = i + lane; k < n; k += 64) {
        c64d acc{0, 0};
#pragma unroll
        for (int cc = 0; cc < CB; ++cc) {
          const int c = c0 + cc;
          const c64d* row = R + (pk(c, c, n) - c);   // row[k] = R[c][k], zero for a dropped pivot
          acc = acc + cmulc(row[i], row[k]);
        }
        R[pk(i, k, n)] = R[pk(i, k, n)] - acc;
      }
    __syncthreads();
    if (wv == 0) {
      factor(t0);
    } else {
      const int t1 = t0 + CB, m = max(0, n - t1);
      const int nt = (m + 3) / 4, ntiles = nt * (nt + 1) / 2;
      for (int t = tid - 64; t < ntiles; t += HT - 64) {
        // tile (ti, tk), tk >= ti, linear index t = tk (tk + 1) / 2 + ti
        int tk = (int)((sqrtf(8.0f * t + 1.0f) - 1.0f) * 0.5f);
        while (tk * (tk + 1) / 2 > t) --tk;
        while ((tk + 1) * (tk + 2) / 2 <= t) ++tk;
        const int ti = t - tk * (tk + 1) / 2;
        const int i0 = t1 + 4 * ti, k0 = t1 + 4 * tk;
        c64d acc[4][4];
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
          for (int b = 0; b < 4; ++b) acc[a][b] = c64d{0, 0};
#pragma unroll 2
        for (int c = c0; c < t0; ++c) {
          c64d ri[4], rk[4];
          const c64d* row = R + (pk(c, c, n) - c);
#pragma unroll
          for (int a = 0; a < 4; ++a) {   // past n: read but not used (min: inside the triangle)
            ri[a] = row[min(i0 + a, n - 1)];
            rk[a] = row[min(k0 + a, n - 1)];
          }
#pragma unroll
          for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int b = 0; b < 4; ++b) acc[a][b] = acc[a][b] + cmulc(ri[a], rk[b]);
        }
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
          for (int b = 0; b < 4; ++b) {
            const int i = i0 + a, k = k0 + b;
            if (i < n && k < n && k >= i) R[pk(i, k, n)] = R[pk(i, k, n)] - acc[a][b];
          }
      }
    }
    __syncthreads();
  }
  if (tid < n) ipiv[tid] = piv[tid] > 0.0 ? 1.0 / piv[tid] : 0.0;
  // R out (upper, zeros below), precision of the state
  for (int i = wv; i < n; i += HT / 64)
    for (int k = lane; k < n; k += 64) {
      c64d v = k >= i ? R[pk(i, k, n)] : c64d{0, 0};
      Ro[(long long)i * n + k] = cplx<T>{(T)v.re, (T)v.im};
    }
  // R^{-1} in place (upper triangle, packed), by 16 x 16 blocks.  For R = [[A, B], [0, C]] the
  // inverse is [[A^-1, -(A^-1 B) C^-1], [0, C^-1]]: the diagonal blocks are inverted together,
  // column by column (column jj of a block's inverse is -(1 / R[j][j]) X[., 0:jj] R[0:jj, jj]
  // within the block), then block column J above the diagonal becomes -(X[0:a, 0:a] R[0:a, J])
  // X_JJ with a = 16 J, for J = 1, 2, ... in turn.  A dropped pivot (1 / R[j][j] taken as 0)
  // gives a zero row and column, so the products below leave those directions out exactly as
  // the substitution would.
  __syncthreads();   // R has been written out
  const int nbk = (n + 15) / 16;
  const int i16 = lane & 15, kq = lane >> 4;
  constexpr int NT16 = NMAX / 16;
  static_assert(HT >= NMAX && HT / 64 >= NT16 - 1, "a thread per row of a diagonal block, a wave per row block");
  if (tid < NMAX) {
    // diagonal blocks: row ii of block b in the registers of thread 16 b + ii, the column of R
    // from the other rows' threads by DPP row broadcasts.  Zeros stand for the elements left of
    // the diagonal; the even and the odd terms are summed apart.
    const int b = tid >> 4, ii = i16, r0 = 16 * b;
    const int bs = b < nbk ? min(16, n - r0) : 0;
    c64d x[16];
#pragma unroll
    for (int l = 0; l < 16; ++l) x[l] = (l >= ii && l < bs) ? R[pk(r0 + ii, r0 + l, n)] : c64d{0, 0};
    inv_cols<0>(x, ii, NMAX <= 64 ? min(n, 16) : 16, ipiv + min(r0, NMAX - 16));
#pragma unroll
    for (int l = 0; l < 16; ++l)
      if (l >= ii && l < bs) R[pk(r0 + ii, r0 + l, n)] = x[l];
  }
  __syncthreads();
  // block columns J >= 1, rows 16 I .. of the block above the diagonal by wave I.  The chains of
  // four fmas that the f64 MFMA runs along K are those of a sum over l taken term by term (real
  // part: x.re r.re, then -x.im r.im), two rows l of the same parity per instruction.
  for (int J = 1; J < nbk; ++J) {
    const int a = 16 * J, cw = min(16, n - a), I = wv, cl = a + min(i16, cw - 1);
    v4d_t y[2][2];                       // [parity of l][re, im]
#pragma unroll
    for (int z = 0; z < 2; ++z) y[z][0] = y[z][1] = v4d_t{0, 0, 0, 0};
    const bool odd = kq & 1;
    if (I < J) {
      // Y[i][jj] = sum_{l >= i} X[i][l] R[l][a + jj], the operands loaded a step ahead
      const int i = 16 * I + i16;
      const c64d* xrow = R + (pk(i, i, n) - i);
      c64d xv[2], rv[2];
      auto load = [&](int l0) {
#pragma unroll
        for (int z = 0; z < 2; ++z) {   // (l < i: some other element of the triangle, not used)
          const int l = min(l0, a - 4) + z + (kq & 2);
          xv[z] = xrow[l];
          rv[z] = R[pk(l, cl, n)];
          if (l < i) xv[z] = c64d{0, 0};
        }
      };
      load(16 * I);
      for (int l0 = 16 * I; l0 < a; l0 += 4) {
        double p[2][2], r[2][2];
#pragma unroll
        for (int z = 0; z < 2; ++z) {
          p[z][0] = odd ? -xv[z].im : xv[z].re;
          r[z][0] = odd ? rv[z].im : rv[z].re;
          p[z][1] = odd ? xv[z].im : xv[z].re;
          r[z][1] = odd ? rv[z].re : rv[z].im;
        }
        load(l0 + 4);
#pragma unroll
        for (int z = 0; z < 2; ++z) {
          y[z][0] = mfma64(p[z][0], r[z][0], y[z][0]);
          y[z][1] = mfma64(p[z][1], r[z][1], y[z][1]);
        }
      }
    }
    __syncthreads();                     // block column J of R has been read
    if (I < J) {
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (i16 < cw) R[pk(16 * I + 4 * q + kq, a + i16, n)] = c64d{y[0][0][q] + y[1][0][q], y[0][1][q] + y[1][1][q]};
      wave_fence();
      // X[i][a + jj] = -sum_{m <= jj} Y[i][m] X_JJ[m][jj]
      v4d_t xr = {0, 0, 0, 0}, xi = {0, 0, 0, 0};
#pragma unroll
      for (int m0 = 0; m0 < 16; m0 += 2) {
        const int m = m0 + (kq >> 1);
        const int mc = min(m, cw - 1);
        c64d yv = R[pk(16 * I + i16, a + mc, n)], zv = R[pk(a + mc, cl, n)];
        if (m >= cw) yv = c64d{0, 0};
        if (m > i16) zv = c64d{0, 0};
        xr = mfma64(odd ? -yv.im : yv.re, odd ? zv.im : zv.re, xr);
        xi = mfma64(odd ? yv.im : yv.re, odd ? zv.re : zv.im, xi);
      }
      wave_fence();
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (i16 < cw) R[pk(16 * I + 4 * q + kq, a + i16, n)] = c64d{-xr[q], -xi[q]};
      wave_fence();                      // read by this wave alone until the last barrier
    }
  }
  __syncthreads();
  // Q = C R^{-1} (L->R, C: other x n, row-major) or Q = R^{-dag} C (R->L, C: n x other), in
  // place, on f64 MFMA over the nonzero triangle of R^{-1}.  A wave owns 16 rows (L->R) or
  // 16 columns (R->L) of C with all their output tiles in registers, so it reads those rows /
  // columns completely before it writes them.  Lane layout (f64 16x16x4): A[i][k] in lane
  // i + 16 k, B[k][j] in lane j + 16 k, D[i][j] in lane j + 16 (i % 4), register i / 4.
  const int nt = nbk;
  if (left_to_right) {
    const int nvt = (other + 15) / 16;
    for (int vt = wv; vt < nvt; vt += HT / 64) {
      v4d_t ar[NT16], ai[NT16];
#pragma unroll
      for (int t = 0; t < NT16; ++t) ar[t] = ai[t] = v4d_t{0, 0, 0, 0};
      const int v = 16 * vt + i16;
      // the step's operands are loaded before its products, the row of C a step ahead
      auto row = [&](int l) { return v < other && l < n ? Cj[(long long)v * n + l] : cplx<T>{0, 0}; };
      cplx<T> cn = row(kq);
      for (int l0 = 0; l0 < n; l0 += 4) {
        const int l = l0 + kq;
        const cplx<T> cv = cn;
        cn = row(l + 4);
        const double cr = (double)cv.re, ci = (double)cv.im;
        c64d b[NT16];
        const c64d* rl = R + pk(min(l, n - 1), 0, n);   // rl[c] = Rinv[l][c]
#pragma unroll
        for (int t = 0; t < NT16; ++t)
          if (t < nt && l0 <= 16 * t + 15) {   // Rinv[l][c] = 0 for l > c
            const int c = 16 * t + i16;
            b[t] = rl[min(c, n - 1)];          // (l > c: some other element, not used)
            if (t == (l0 >> 4) || t == nt - 1)
              if (!(l < n && c < n && l <= c)) b[t] = c64d{0, 0};
          }
#pragma unroll
        for (int t = 0; t < NT16; ++t)
          if (t < nt && l0 <= 16 * t + 15) {
            ar[t] = mfma64(cr, b[t].re, ar[t]);
            ai[t] = mfma64(cr, b[t].im, ai[t]);
            ar[t] = mfma64(-ci, b[t].im, ar[t]);
            ai[t] = mfma64(ci, b[t].re, ai[t]);
          }
      }
#pragma unroll
      for (int t = 0; t < NT16; ++t)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int row = 16 * vt + kq + 4 * q, c = 16 * t + i16;
          if (t < nt && row < other && c < n) Cj[(long long)row * n + c] = cplx<T>{(T)ar[t][q], (T)ai[t][q]};
        }
    }
  } else {
    const int nvt = (other + 15) / 16;
    for (int vt = wv; vt < nvt; vt += HT / 64) {
      v4d_t ar[NT16], ai[NT16];
#pragma unroll
      for (int t = 0; t < NT16; ++t) ar[t] = ai[t] = v4d_t{0, 0, 0, 0};
      const int v = 16 * vt + i16;
      auto col = [&](int l) { return v < other && l < n ? Cj[(long long)l * other + v] : cplx<T>{0, 0}; };
      cplx<T> cn = col(kq);
      for (int l0 = 0; l0 < n; l0 += 4) {
        const int l = l0 + kq;
        const cplx<T> cv = cn;
        cn = col(l + 4);
        const double br = (double)cv.re, bi = (double)cv.im;
        c64d a[NT16];
        const c64d* rl = R + pk(min(l, n - 1), 0, n);
#pragma unroll
        for (int t = 0; t < NT16; ++t)
          if (t < nt && l0 <= 16 * t + 15) {   // conj(Rinv[l][r]) = 0 for l > r
            const int r = 16 * t + i16;
            a[t] = rl[min(r, n - 1)];
            if (t == (l0 >> 4) || t == nt - 1)
              if (!(l < n && r < n && l <= r)) a[t] = c64d{0, 0};
          }
        // A[r][l] = conj(Rinv[l][r])
#pragma unroll
        for (int t = 0; t < NT16; ++t)
          if (t < nt && l0 <= 16 * t + 15) {
            ar[t] = mfma64(a[t].re, br, ar[t]);
            ai[t] = mfma64(a[t].re, bi, ai[t]);
            ar[t] = mfma64(a[t].im, bi, ar[t]);
            ai[t] = mfma64(-a[t].im, br, ai[t]);
          }
      }
#pragma unroll
      for (int t = 0; t < NT16; ++t)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int r = 16 * t + kq + 4 * q, col = 16 * vt + i16;
          if (t < nt && r < n && col < other) Cj[(long long)r * other + col] = cplx<T>{(T)ar[t][q], (T)ai[t][q]};
        }
    }
  }
}

namespace {
template <typename T, int NMAX, int HT>
void launch_chol(int n, int left_to_right, int other, const void* E, long long sE, void* C, long long sC, void* Rout,
                 long long sR, double tol, int n_traj, hipStream_t st) {
  hipLaunchKernelGGL((k_hop_chol<T, NMAX, HT>), dim3(n_traj), dim3(HT), 0, st, n, left_to_right, other, (const c64d*)E, sE,
                     (cplx<T>*)C, sC, (cplx<T>*)Rout, sR, tol);
}
template <typename T>
void launch_chol_n(int n, int left_to_right, int other, const void* E, long long sE, void* C, long long sC, void* Rout,
                   long long sR, double tol, int n_traj, hipStream_t st) {
  // the smallest triangle that holds the factor: 9 and 35 KB of LDS leave room for several workgroups
  // per CU (1000 of n = 32 and 512 of n = 64 with the last one: 222, 235 us against 62, 117); the
  // 78 KB instance runs one by its registers, the 136 KB one by its LDS
  if (n <= 32) launch_chol<T, 32, 256>(n, left_to_right, other, E, sE, C, sC, Rout, sR, tol, n_traj, st);
  else if (n <= 64) launch_chol<T, 64, 256>(n, left_to_right, other, E, sE, C, sC, Rout, sR, tol, n_traj, st);
  else if (n <= 96) launch_chol<T, 96, 512>(n, left_to_right, other, E, sE, C, sC, Rout, sR, tol, n_traj, st);
  else launch_chol<T, 128, 512>(n, left_to_right, other, E, sE, C, sC, Rout, sR, tol, n_traj, st);
}
}  // namespace

hipError_t hop_chol(int prec, int n, int left_to_right, int other, const void* E, long long sE, void* C, long long sC,
                    void* Rout, long long sR, double tol, int n_traj, hipStream_t st) {
  if (n > 128) return hipErrorInvalidValue;
  if (prec == 0) launch_chol_n<float>(n, left_to_right, other, E, sE, C, sC, Rout, sR, tol, n_traj, st);
  else launch_chol_n<double>(n, left_to_right, other, E, sE, C, sC, Rout, sR, tol, n_traj, st);
  return hipGetLastError();
}

}  // namespace mpsb
