// The batched optimal unravelling of given reduced states: unravel.hip's steps (formulas there),
// one lane per item, in the form that is fastest where the results stand alone.  The Takagi
// factorisation runs in complex form on 4 x 4 registers and the rotations by Newton steps.  A
// trajectory's events keep the other form: a sweep carries their branch operators through every
// later truncation, and discarded weights at rounding level follow their last place (up to 1e-3
// of such a weight over four layers, against 2 % of a chi-64 layer).
// The steps between stand in both files: shared as templates over the two arithmetics, the compiler's
// fused operations in the events, and with them every recorded run's last place, were others, and the
// events slower (2048 single-site events 7.9 -> 10.6 us without, 128 -> 134 with the eigensolver).
// So what is mended in one belongs into the other.
// Bound by the serial chain of the Jacobi sweeps (1000 items are 16 waves on the chip; 200000 are
// three waves per SIMD).  Against the real 8 x 8 embedding with library divisions and 576 bytes of
// per-lane scratch: 1000 items 137 -> 72 us, 200000 items 596 -> 292 us.
#include <float.h>

#include "common.h"
#include "kernels.h"
#include "unravel_small.h"

namespace mpsb {

namespace {

// 1 / x and 1 / sqrt(x) by the hardware estimate and Newton steps to the last place or two (normal
// range; a division or square root of the library costs several times the rotation's own work)
__device__ inline double frcp(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = fma(r, fma(-x, r, 1.0), r);
  return fma(r, fma(-x, r, 1.0), r);
}
__device__ inline double frsqrt(double x) {
  double y = __builtin_amdgcn_rsq(x);
  y = fma(0.5 * y, fma(-(x * y), y, 1.0), y);
  return fma(0.5 * y, fma(-(x * y), y, 1.0), y);
}

// Jacobi rotation that annihilates the off-diagonal entry off of a symmetric 2 x 2 block with
// diagonal entries dp, dq: t = sign(z) / (|z| + sqrt(1 + z^2)), z = (dq - dp) / (2 off), and
// c = 1 / sqrt(1 + t^2), s = c t
__device__ inline void rotation(double dp, double dq, double off, double& c, double& s) {
  // an entry near the end of the range has no reciprocal
  const double z = fabs(off) > 1e-290 ? (dq - dp) * frcp(2.0 * off) : (dq - dp) / (2.0 * off), az = fabs(z);
  const double w = fma(az, az, 1.0);
  // past 1e8 the sum is 2 |z| to working precision (and z^2 may overflow)
  const double den = az > 1e8 ? 2.0 * az : az + w * frsqrt(w);
  double t = den > 1e300 ? 0.0 : frcp(den);
  t = z >= 0 ? t : -t;
  c = frsqrt(fma(t, t, 1.0));
  s = c * t;
}

// cyclic Jacobi eigen-decomposition of a real symmetric n x n matrix (n <= NMAX), in place:
// on exit a holds the eigenvalues on its diagonal, v the eigenvectors (columns).  The sweeps run
// on local copies with every index fixed at compile time (pairs and rows unrolled over NMAX,
// n as a guard), so that the matrices stay in registers rather than in per-lane scratch.  A
// pair is rotated only while its off-diagonal entry is not negligible against its diagonal
// entries (|a_pq| > eps (|a_pp| + |a_qq|) / 2), and the iteration stops after a sweep without a
// rotation (a test on the summed off-diagonal mass alone can stall above its threshold at
// rounding level and run every sweep).
template <int NMAX>
__device__ void jacobi_sym(int n, double (&a_io)[NMAX][NMAX], double (&v_io)[NMAX][NMAX]) {
  double a[NMAX][NMAX], v[NMAX][NMAX];
#pragma unroll
  for (int i = 0; i < NMAX; ++i)
#pragma unroll
    for (int j = 0; j < NMAX; ++j) {
      a[i][j] = (i < n && j < n) ? a_io[i][j] : 0.0;
      v[i][j] = (i == j) ? 1.0 : 0.0;
    }
  for (int sweep = 0; sweep < 30; ++sweep) {
    double off = 0, tot = 0;
#pragma unroll
    for (int i = 0; i < NMAX; ++i)
#pragma unroll
      for (int j = 0; j < NMAX; ++j) {
        tot += a[i][j] * a[i][j];
        if (i != j) off += a[i][j] * a[i][j];
      }
    if (off <= 1e-34 * tot || off == 0.0) break;
    bool rotated = false;
#pragma unroll
    for (int p = 0; p < NMAX - 1; ++p)
#pragma unroll
      for (int q = p + 1; q < NMAX; ++q) {
        const double apq = a[p][q];
        if (q < n && fabs(apq) > DBL_EPSILON * 0.5 * (fabs(a[p][p]) + fabs(a[q][q])) && fabs(apq) > 1e-300) {
          rotated = true;
          double c, s;
          rotation(a[p][p], a[q][q], apq, c, s);
#pragma unroll
          for (int k = 0; k < NMAX; ++k) {
            double akp = a[k][p], akq = a[k][q];
            a[k][p] = c * akp - s * akq;
            a[k][q] = s * akp + c * akq;
          }
#pragma unroll
          for (int k = 0; k < NMAX; ++k) {
            double apk = a[p][k], aqk = a[q][k];
            a[p][k] = c * apk - s * aqk;
            a[q][k] = s * apk + c * aqk;
          }
#pragma unroll
          for (int k = 0; k < NMAX; ++k) {
            double vkp = v[k][p], vkq = v[k][q];
            v[k][p] = c * vkp - s * vkq;
            v[k][q] = s * vkp + c * vkq;
          }
        }
      }
    if (!rotated) break;
  }
#pragma unroll
  for (int i = 0; i < NMAX; ++i)
#pragma unroll
    for (int j = 0; j < NMAX; ++j)
      if (i < n && j < n) {
        a_io[i][j] = a[i][j];
        v_io[i][j] = v[i][j];
      }
}

// Takagi vectors of a complex symmetric 4 x 4 matrix tau = A + iB by the cyclic Jacobi iteration
// on its real embedding [[A, B], [B, -A]] (8 x 8, eigenvalues +- sigma), in complex form: the
// embedding's pairs (p, q) and (p+4, q+4) take the same angle, a real rotation of the columns p
// and q of U; (p, q+4) and (q, p+4) take the same angle, a rotation by -i s; (p, p+4) is a phase.
// So a sweep is 16 rotations of 4-vectors of complex numbers instead of 28 of 8-vectors, and the
// matrices are 128 registers instead of 256 (which left the embedding's sweeps moving values
// between register files).  On exit tau = U^dag tau U* is diagonal and real, A_pp = +- sigma.
// A pair is rotated only while its entry is not negligible against the diagonal, as in jacobi_sym.
__device__ void takagi_jacobi(cd (&t)[4][4], cd (&U)[4][4]) {
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) U[i][j] = i == j ? cd{1.0, 0.0} : cz();
  for (int sweep = 0; sweep < 30; ++sweep) {
    bool rotated = false;
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      // phase: B_pp
      {
        const double off = t[p][p].im, d = t[p][p].re;
        if (fabs(off) > DBL_EPSILON * fabs(d) && fabs(off) > 1e-300) {
          rotated = true;
          double c, s;
          rotation(d, -d, off, c, s);
          const cd m = {c, s}, mu = {c, -s};
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            t[k][p] = m * t[k][p];
            U[k][p] = mu * U[k][p];
          }
#pragma unroll
          for (int k = 0; k < 4; ++k) t[p][k] = m * t[p][k];
        }
      }
#pragma unroll
      for (int q = p + 1; q < 4; ++q) {
        // real rotation: A_pq
        const double ar = t[p][q].re;
        if (fabs(ar) > DBL_EPSILON * 0.5 * (fabs(t[p][p].re) + fabs(t[q][q].re)) && fabs(ar) > 1e-300) {
          rotated = true;
          double c, s;
          rotation(t[p][p].re, t[q][q].re, ar, c, s);
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const cd x = t[k][p], y = t[k][q], u = U[k][p], v = U[k][q];
            t[k][p] = c * x - s * y;
            t[k][q] = s * x + c * y;
            U[k][p] = c * u - s * v;
            U[k][q] = s * u + c * v;
          }
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const cd x = t[p][k], y = t[q][k];
            t[p][k] = c * x - s * y;
            t[q][k] = s * x + c * y;
          }
        }
        // imaginary rotation: B_pq, between the diagonal entries A_pp and -A_qq
        const double ai = t[p][q].im;
        if (fabs(ai) > DBL_EPSILON * 0.5 * (fabs(t[p][p].re) + fabs(t[q][q].re)) && fabs(ai) > 1e-300) {
          rotated = true;
          double c, s;
          rotation(t[p][p].re, -t[q][q].re, ai, c, s);
          // columns p, q of tau by [[c, i s], [i s, c]], of U by [[c, -i s], [-i s, c]]
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const cd x = t[k][p], y = t[k][q], u = U[k][p], v = U[k][q];
            t[k][p] = cd{c * x.re - s * y.im, c * x.im + s * y.re};
            t[k][q] = cd{c * y.re - s * x.im, c * y.im + s * x.re};
            U[k][p] = cd{c * u.re + s * v.im, c * u.im - s * v.re};
            U[k][q] = cd{c * v.re + s * u.im, c * v.im - s * u.re};
          }
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const cd x = t[p][k], y = t[q][k];
            t[p][k] = cd{c * x.re - s * y.im, c * x.im + s * y.re};
            t[q][k] = cd{c * y.re - s * x.im, c * y.im + s * x.re};
          }
        }
      }
    }
    if (!rotated) break;
  }
}

__device__ void optimal_mixing(const cd (&rho)[2][2], const cd (&K)[4][2][2], int r, UnravelOut& out) {
  // Psi_eff = sqrt(rho) for a 2x2 PSD matrix: (rho + sqrt(det) I) / sqrt(tr + 2 sqrt(det))
  double tr = rho[0][0].re + rho[1][1].re;
  double det = rho[0][0].re * rho[1][1].re - norm2(rho[0][1]);
  double sd = sqrt(fmax(det, 0.0));
  double den = sqrt(fmax(tr + 2.0 * sd, 0.0));
  cd psi[2][2];
  for (int a = 0; a < 2; ++a)
    for (int b = 0; b < 2; ++b) {
      cd v = rho[a][b];
      if (a == b) v.re += sd;
      psi[a][b] = den > 0 ? cd{v.re / den, v.im / den} : cz();
    }
  // phi columns
  cd ph[4][4];   // [component][i]
  for (int i = 0; i < 4; ++i)
    for (int s = 0; s < 2; ++s)
      for (int e = 0; e < 2; ++e) {
        cd acc = cz();
        if (i < r)
          for (int m = 0; m < 2; ++m) cfma(acc, K[i][s][m], psi[m][e]);
        ph[2 * s + e][i] = acc;
      }
  // one-sided Jacobi: columns of ph made orthogonal, V accumulated
  cd V[4][4];
  for (int i = 0; i < 4; ++i)
    for (int j = 0; j < 4; ++j) V[i][j] = (i == j) ? cd{1.0, 0.0} : cz();
  // (pairs unrolled with r as a guard, so that ph and V keep compile-time indices)
  for (int sweep = 0; sweep < 30; ++sweep) {
    bool rotated = false;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int j = i + 1; j < 4; ++j) {
        if (j >= r) continue;
        double al = 0, be = 0;
        cd ga = cz();
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          al += norm2(ph[c][i]);
          be += norm2(ph[c][j]);
          ga = ga + cmulc(ph[c][i], ph[c][j]);
        }
        // columns orthogonal to working precision: no rotation (a relative 1e-17 test below the
        // rounding level of the products would keep every sweep rotating)
        double c, s;
        cd eph;   // e^{-i phi}
        const double g2 = norm2(ga);
        double g;
        if (g2 > 1e-250) {
          if (g2 <= 4.0 * DBL_EPSILON * DBL_EPSILON * (al * be)) continue;
          const double ig = frsqrt(g2);
          g = g2 * ig;
          eph = cd{ga.re * ig, -ga.im * ig};
        } else {   // the squares may underflow: scaled, so that the phase keeps its modulus
          const double m = fmax(fabs(ga.re), fabs(ga.im));
          if (m == 0.0) continue;
          const cd u = {ga.re / m, ga.im / m};
          const double n2 = norm2(u);
          g = m * sqrt(n2);
          if (g <= 2.0 * DBL_EPSILON * sqrt(al) * sqrt(be)) continue;
          const double iu = frsqrt(n2);
          eph = cd{u.re * iu, -u.im * iu};
        }
        rotated = true;
        rotation(al, be, g, c, s);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          cd ai = ph[k][i], aj = eph * ph[k][j];
          ph[k][i] = c * ai - s * aj;
          ph[k][j] = s * ai + c * aj;
          cd vi = V[k][i], vj = eph * V[k][j];
          V[k][i] = c * vi - s * vj;
          V[k][j] = s * vi + c * vj;
        }
      }
    if (!rotated) break;
  }
  // singular values in descending order: the exchange sort of the indices, on register copies
  double sv[4];
  int ord[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    double s2 = 0;
#pragma unroll
    for (int c = 0; c < 4; ++c) s2 += norm2(ph[c][i]);
    sv[i] = (i < r) ? sqrt(s2) : -1.0;
    ord[i] = i;
  }
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = i + 1; j < 4; ++j)
      if (sv[j] > sv[i]) {
        const double tv = sv[i];
        sv[i] = sv[j];
        sv[j] = tv;
        const int ti = ord[i];
        ord[i] = ord[j];
        ord[j] = ti;
      }
  const double smax = sv[0];
  int rank = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i)
    if (i < r && sv[i] > 1e-12 * smax) rank++;
  cd v[4][4];    // [component][k], k < rank
  cd Vs[4][4];   // sorted V columns
#pragma unroll
  for (int k = 0; k < 4; ++k)
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      cd pv = cz(), vv = cz();
#pragma unroll
      for (int t = 0; t < 4; ++t)
        if (ord[k] == t) {
          pv = ph[c][t];
          vv = V[c][t];
        }
      v[c][k] = (k < rank) ? pv : cz();
      Vs[c][k] = vv;
    }
  // From here on every array index is fixed at compile time (loops over the padded size 4
  // or 8 with the rank as a guard, gathers by selects), so that the arrays stay in registers
  // instead of per-lane scratch memory.
  // tau = v^dag v~ (zero outside its rank x rank block)
  cd tau[4][4];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      cd vb[4] = {v[0][b], v[1][b], v[2][b], v[3][b]};
      cd acc = cz();
#pragma unroll
      for (int c = 0; c < 4; ++c) acc = acc + cmulc(v[c][a], yy_flip(vb, c));
      tau[a][b] = (a < rank && b < rank) ? acc : cz();
    }
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = a + 1; b < 4; ++b) {
      cd m = {0.5 * (tau[a][b].re + tau[b][a].re), 0.5 * (tau[a][b].im + tau[b][a].im)};
      tau[a][b] = m;
      tau[b][a] = m;
    }
  cd UT[4][4];   // Takagi vectors
  double lam[4] = {0, 0, 0, 0};
  int kpos = 0;
  // Takagi by Jacobi rotations of the real embedding [[A, B], [B, -A]] of tau = A + iB (see
  // takagi_jacobi; the rows and columns beyond the rank are zero and never rotated)
  cd Q[4][4];
  takagi_jacobi(tau, Q);
  // eigenvalue A_pp belongs to column p of Q, -A_pp to i times it
  double sg4[4];
  double emax = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const bool neg = tau[i][i].re < 0.0;
    sg4[i] = fabs(tau[i][i].re);
    emax = fmax(emax, sg4[i]);
#pragma unroll
    for (int a = 0; a < 4; ++a)
      if (neg) Q[a][i] = cd{-Q[a][i].im, Q[a][i].re};
  }
  // columns of U_T: the positive eigenvalues in descending order (ties: lower index), at most
  // rank of them
  unsigned taken = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    int idx = -1;
    double best = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (!((taken >> i) & 1u) && (idx < 0 || sg4[i] > best)) {
        idx = i;
        best = sg4[i];
      }
    const bool use = kpos == k && k < rank && best > 1e-12 * emax;
    cd qc[4];
#pragma unroll
    for (int a = 0; a < 4; ++a) qc[a] = cz();
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (i == idx) {
#pragma unroll
        for (int a = 0; a < 4; ++a) qc[a] = Q[a][i];
      }
    double nn = 0;
#pragma unroll
    for (int a = 0; a < 4; ++a)
      if (a < rank) nn += norm2(qc[a]);
    nn = nn > 0 ? 1.0 / sqrt(nn) : 0.0;
#pragma unroll
    for (int a = 0; a < 4; ++a) UT[a][k] = (use && a < rank) ? nn * qc[a] : cz();
    lam[k] = use ? best : 0.0;
    if (use) {
      kpos = k + 1;
      taken |= 1u << idx;
    }
  }
  // null directions (tau singular on the rank block): columns of ~0 eigenvalue, complex
  // Gram-Schmidt against the chosen columns, the largest residual taken
  bool nostop = true;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    if (!(nostop && k == kpos && k < rank)) continue;
    double best = -1;
    cd cand[4] = {cz(), cz(), cz(), cz()};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (sg4[i] > 1e-12 * emax) continue;
      cd u[4];
#pragma unroll
      for (int a = 0; a < 4; ++a) u[a] = a < rank ? Q[a][i] : cz();
#pragma unroll
      for (int kk = 0; kk < k; ++kk) {
        cd pr = cz();
#pragma unroll
        for (int a = 0; a < 4; ++a) pr = pr + cmulc(UT[a][kk], u[a]);
#pragma unroll
        for (int a = 0; a < 4; ++a) u[a] = u[a] - pr * UT[a][kk];
      }
      double nn = 0;
#pragma unroll
      for (int a = 0; a < 4; ++a) nn += norm2(u[a]);
      if (nn > best) {
        best = nn;
#pragma unroll
        for (int a = 0; a < 4; ++a) cand[a] = u[a];
      }
    }
    if (best <= 1e-20) {
      nostop = false;
      continue;
    }
    const double inv = 1.0 / sqrt(best);
#pragma unroll
    for (int a = 0; a < 4; ++a) UT[a][k] = inv * cand[a];
    lam[k] = 0.0;
    kpos = k + 1;
  }
  // x = v U_T with the sign / phase pins: the first entry of largest modulus of column k made
  // real positive (sigma > 0: sign only; sigma = 0: its phase)
  cd x[4][4];
#pragma unroll
  for (int k = 0; k < 4; ++k)
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      cd acc = cz();
#pragma unroll
      for (int a = 0; a < 4; ++a)
        if (a < rank) cfma(acc, v[c][a], UT[a][k]);
      x[c][k] = k < kpos ? acc : cz();
    }
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    if (k >= kpos) continue;
    double mx = 0;
#pragma unroll
    for (int c = 0; c < 4; ++c) mx = fmax(mx, cabs_(x[c][k]));
    int i = -1;
#pragma unroll
    for (int c = 0; c < 4; ++c)
      if (i < 0 && cabs_(x[c][k]) >= mx * (1.0 - 1e-12)) i = c;
    cd e = x[0][k];
#pragma unroll
    for (int c = 1; c < 4; ++c)
      if (c == i) e = x[c][k];
    const double ae = cabs_(e);
    if (ae == 0.0) continue;
    cd f;
    if (lam[k] > 0.0) f = (e.re < 0.0 || (e.re == 0.0 && e.im < 0.0)) ? cd{-1.0, 0.0} : cd{1.0, 0.0};
    else f = cd{e.re / ae, -e.im / ae};
#pragma unroll
    for (int a = 0; a < 4; ++a) UT[a][k] = UT[a][k] * f;
#pragma unroll
    for (int c = 0; c < 4; ++c) x[c][k] = x[c][k] * f;
  }
  const double cdiff = lam[0] - lam[1] - lam[2] - lam[3];
  const double conc = fmax(0.0, cdiff);
  cd Em[4][4];   // E[a][col]
  const double h = 0.5;
  const double H4[4][4] = {{h, h, h, h}, {h, h, -h, -h}, {h, -h, h, -h}, {h, -h, -h, h}};
  if (cdiff > 0.0) {
    const cd u2[4] = {{1, 0}, {0, -1}, {0, -1}, {0, -1}};
    cd y[4][4];
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int k = 0; k < 4; ++k) y[c][k] = x[c][k] * u2[k];
    double MR[4][4], QR[4][4];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        cd yb[4] = {y[0][b], y[1][b], y[2][b], y[3][b]};
        cd s1 = cz(), s2 = cz();
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          s1 = s1 + cmulc(y[c][a], yy_flip(yb, c));
          s2 = s2 + cmulc(y[c][a], y[c][b]);
        }
        MR[a][b] = s1.re - conc * s2.re;
      }
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int b = a + 1; b < 4; ++b) {
        double m = 0.5 * (MR[a][b] + MR[b][a]);
        MR[a][b] = MR[b][a] = m;
      }
    jacobi_sym<4>(4, MR, QR);
    // eigenvalues ascending: the exchange sort of the indices, on register copies
    double qv[4];
    int qo[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      qv[i] = MR[i][i];
      qo[i] = i;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = i + 1; j < 4; ++j)
        if (qv[j] < qv[i]) {
          const double tv = qv[i];
          qv[i] = qv[j];
          qv[j] = tv;
          const int ti = qo[i];
          qo[i] = qo[j];
          qo[j] = ti;
        }
    double Qs[4][4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      double col[4] = {0, 0, 0, 0};
#pragma unroll
      for (int t = 0; t < 4; ++t)
        if (qo[k] == t) {
#pragma unroll
          for (int a = 0; a < 4; ++a) col[a] = QR[a][t];
        }
      double mx = 0;
#pragma unroll
      for (int a = 0; a < 4; ++a) mx = fmax(mx, fabs(col[a]));
      double lead = col[0];
      bool found = false;
#pragma unroll
      for (int a = 0; a < 4; ++a)
        if (!found && fabs(col[a]) >= mx * (1.0 - 1e-12)) {
          lead = col[a];
          found = true;
        }
      const double sg = lead < 0 ? -1.0 : 1.0;
#pragma unroll
      for (int a = 0; a < 4; ++a) Qs[a][k] = sg * col[a];
    }
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int cc = 0; cc < 4; ++cc) {
        double sum = 0;
#pragma unroll
        for (int b = 0; b < 4; ++b) sum += Qs[a][b] * H4[cc][b];
        Em[a][cc] = u2[a] * cd{sum, 0.0};
      }
  } else {
    double l1 = lam[0], l2 = lam[1], l3 = lam[2], l4 = lam[3];
    double th[4];
    if (l1 - l4 <= 1e-15 * fmax(l1, 1e-300)) {
      th[0] = 0; th[1] = M_PI / 4; th[2] = M_PI / 2; th[3] = 3 * M_PI / 4;
    } else {
      double base = l1 - l4, sp = 0.5 * (base + l2 + l3);
      double area2 = fmax(0.0, sp * (sp - base) * (sp - l2) * (sp - l3));
      double hh = 2.0 / base * sqrt(area2);
      double t2 = (l2 > 0) ? M_PI - asin(fmin(1.0, hh / l2)) : M_PI;
      double cr = (l4 - l1) - l2 * cos(t2), ci = -l2 * sin(t2);
      double t3 = (cr != 0.0 || ci != 0.0) ? atan2(ci, cr) : 0.0;
      th[0] = 0; th[1] = 0.5 * t2; th[2] = 0.5 * t3; th[3] = M_PI / 2;
    }
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int cc = 0; cc < 4; ++cc) Em[a][cc] = cd{cos(th[a]) * H4[a][cc], sin(th[a]) * H4[a][cc]};
  }
  // W = Vs[:, :rank] U_T E[:rank] + Vs[:, rank:r] E[rank:r]
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      cd acc = cz();
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        if (a < rank) {
          cd ue = cz();
#pragma unroll
          for (int k = 0; k < 4; ++k)
            if (k < rank) cfma(ue, UT[a][k], Em[k][j]);
          cfma(acc, Vs[i][a], ue);
        } else if (a < r) {
          cfma(acc, Vs[i][a], Em[a][j]);
        }
      }
      out.W[i][j] = i < r ? acc : cz();
    }
  out.conc = conc;
}

__device__ void mixed_ops(const cd (&K)[4][2][2], int r, const cd (&W)[4][4], const cd (&rho)[2][2],
                          cd (&Kp)[4][2][2], double (&p)[4]) {
  for (int j = 0; j < 4; ++j) {
    for (int a = 0; a < 2; ++a)
      for (int b = 0; b < 2; ++b) {
        cd acc = cz();
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (i < r) cfma(acc, W[i][j], K[i][a][b]);
        Kp[j][a][b] = acc;
      }
    double s = 0;
    for (int a = 0; a < 2; ++a) {
      // (K rho K^dag)[a][a] = sum_{m,n} K[a][m] rho[m][n] conj(K[a][n])
      cd acc = cz();
      for (int m = 0; m < 2; ++m)
        for (int nn = 0; nn < 2; ++nn) acc = acc + Kp[j][a][m] * rho[m][nn] * conj(Kp[j][a][nn]);
      s += acc.re;
    }
    p[j] = fmax(s, 0.0);
  }
}

}  // namespace

// ------------------------------------------------------------------ unravel_opt
// An item whose channel id lies outside 0..n_k-1 reads no channel: its U, p and eof are NaN.
__global__ __launch_bounds__(64) __attribute__((flatten)) void k_unravel_opt(int batch, const double* __restrict__ rho_q, const double* __restrict__ kraus,
                              int n_k, const int* __restrict__ kraus_id, int r, double* __restrict__ U,
                              double* __restrict__ p_out, double* __restrict__ eof) {
  int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= batch) return;
  const int kid = kraus_id ? kraus_id[b] : 0;
  if (kid < 0 || kid >= n_k) {
    const double nan = __builtin_nan("");
    for (int j = 0; j < 4; ++j) {
      p_out[b * 4 + j] = nan;
      for (int i = 0; i < 2 * r; ++i) U[((long long)b * 4 + j) * r * 2 + i] = nan;
    }
    eof[b] = nan;
    return;
  }
  cd rho[2][2];
#pragma unroll
  for (int x = 0; x < 4; ++x) rho[x >> 1][x & 1] = cd{rho_q[b * 8 + 2 * x], rho_q[b * 8 + 2 * x + 1]};
  cd K[4][2][2];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        if (i < r) {
          const double* kp = kraus + ((long long)kid * r + i) * 8 + 2 * (2 * a + c);
          K[i][a][c] = cd{kp[0], kp[1]};
        } else K[i][a][c] = cz();
      }
  UnravelOut o;
  optimal_mixing(rho, K, r, o);
  cd Kp[4][2][2];
  double p[4];
  mixed_ops(K, r, o.W, rho, Kp, p);
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    p_out[b * 4 + j] = p[j];
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (i < r) {
        U[((long long)b * 4 + j) * r * 2 + 2 * i] = o.W[i][j].re;
        U[((long long)b * 4 + j) * r * 2 + 2 * i + 1] = o.W[i][j].im;
      }
  }
  double c = fmin(fmax(o.conc, 0.0), 1.0);
  double x = 0.5 * (1.0 + sqrt(fmax(0.0, 1.0 - c * c)));
  double h = 0;
  if (x > 0 && x < 1) h = -x * log2(x) - (1 - x) * log2(1 - x);
  eof[b] = h;
}

hipError_t launch_unravel_opt(int batch, const double* rho_q, const double* kraus, int n_k, const int* kraus_id, int r,
                              double* U, double* p, double* eof, hipStream_t st) {
  hipLaunchKernelGGL(k_unravel_opt, dim3((batch + 63) / 64), dim3(64), 0, st, batch, rho_q, kraus, n_k, kraus_id, r, U, p,
                     eof);
  return hipGetLastError();
}

}  // namespace mpsb
