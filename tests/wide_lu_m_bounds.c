/* Host replica of the index arithmetic of the workgroup integration's LU and
 * triangular solves (lu_m, block_apply, factor_m and solve_w of the
 * large-mechanism integrator), for bounds checking under AddressSanitizer.
 * TEST INFRASTRUCTURE ONLY.
 *
 * Every buffer is allocated on its own, at exactly the size the kernel's layout
 * gives it: in LDS the panel (18 ld doubles), each wave's table (8 rows of 14),
 * the solves' block rows (16 rows of 18), the candidates and solved values (144
 * doubles), pos (ld ints) and the solve vectors (ld doubles each); in HBM the two
 * matrix slots (n columns of ld doubles). That the LDS buffers fit the region the
 * kernel gives them is checked too. Uninitialised buffers, registers and padding
 * rows hold NaN, so that any use of them shows in the results.
 *
 * The kernel's registers are arrays per thread. The 256 threads run one after the
 * other inside each phase between two barriers; a wave's lanes run in lock step
 * where they exchange values. The loads run where the kernel issues them (two
 * blocks ahead, across the panel's factorisation), so that a load of what is not
 * finished yet would show as well.
 *
 * Usage: wide_lu_m_bounds <out.bin> <n_lo> <n_hi> <pattern>
 * pattern 0: random matrices; 1: every pivot is the last row; 2: no pivoting;
 * 3: column n-1 zero; 4: column n/2 zero; 5: every column ties.
 * For each n it writes n, ld, info, the input g I - J (row-major), the factors in
 * logical row order, the logical position of each row and the solution of
 * A x = b for b_i = i + 1 (zeros for a singular matrix).
 */
#include <math.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

enum { T = 256, MB = 16, MS = 18, BK = 8, TW = 14, SB = 16, XS = 18, LS = 14, UB = 144, CAND = 2 + MB };

/* LDS */
static double *H, *TAB[4], *TS, *ub, *b, *x;
static int* pos;
/* registers */
static double C[T][4][4], Q[3][T][4][BK], V[3][T][SB], acc[T], P[T][MB];
static int PS[T][4], pq[T], pt[T];

static int imin(int a, int c) { return a < c ? a : c; }
static int imax(int a, int c) { return a > c ? a : c; }

static int slot_row(int lane, int s, int nt, int ld) { return s < nt - 1 ? lane + 64 * s : imin(lane + 64 * s, ld - 1); }

static void mult_load(const double* M, int ld, int nt, int kb, double q[T][4][BK]) {
  for (int t = 0; t < T; ++t)
    for (int j = 0; j < BK; ++j)
      for (int s = 0; s < nt; ++s) q[t][s][j] = M[(kb + j) * ld + slot_row(t & 63, s, nt, ld)];
}

static void cols_load(const double* J, int n, int ld, int nt, int k0) {
  for (int t = 0; t < T; ++t)
    for (int j = 0; j < 4; ++j)
      for (int s = 0; s < nt; ++s) C[t][s][j] = J[imin(k0 + 4 * (t >> 6) + j, n - 1) * ld + slot_row(t & 63, s, nt, ld)];
}

static void cols_form(double g, int n, int nt, int k0) {
  for (int t = 0; t < T; ++t)
    for (int s = 0; s < nt; ++s)
      for (int j = 0; j < 4; ++j) {
        const int q = (t & 63) + 64 * s, col = k0 + 4 * (t >> 6) + j;
        const double v = (q == col ? g : 0.0) - C[t][s][j];
        C[t][s][j] = q < n && col < n ? v : 0.0;
      }
}

static void block_apply(int w, int nt, double q[T][4][BK], int kb) {
  double* tab = TAB[w];
  for (int l = 0; l < 64; ++l) {
    const int t = 64 * w + l;
    for (int s = 0; s < nt; ++s) {
      const int r = PS[t][s] - kb;
      if (r >= 0 && r < BK) {
        for (int c = 0; c < 4; ++c) tab[r * TW + c] = C[t][s][c];
        for (int j = 0; j < BK; ++j) tab[r * TW + 4 + j] = q[t][s][j];
      }
    }
  }
  double xs[64], lr[64][BK], z[64];
  for (int l = 0; l < 64; ++l) {
    const double* d = tab + (l & (BK - 1)) * TW;
    xs[l] = d[l >> 4];
    for (int j = 0; j < BK; ++j) lr[l][j] = d[4 + j];
  }
  for (int l = 0; l < 64; ++l)
    for (int s = 0; s < nt; ++s)
      for (int j = 0; j < BK; ++j) q[64 * w + l][s][j] = PS[64 * w + l][s] - kb > j ? q[64 * w + l][s][j] : 0.0;
  for (int j = 0; j < BK - 1; ++j) {
    for (int l = 0; l < 64; ++l) z[l] = xs[(l & ~15) + j];
    for (int l = 0; l < 64; ++l) xs[l] = xs[l] - z[l] * ((l & 15) > j ? lr[l][j] : 0.0);
  }
  for (int j = 0; j < BK; ++j)
    for (int l = 0; l < 64; ++l)
      for (int s = 0; s < nt; ++s)
        for (int c = 0; c < 4; ++c) C[64 * w + l][s][c] = C[64 * w + l][s][c] - q[64 * w + l][s][j] * xs[16 * c + j];
}

static int factor_m(double* M, int n, int ld, int k0, int nb, int info) {
  for (int t = 0; t < T; ++t)
    for (int j = 0; j < MB; ++j) P[t][j] = H[(t < n ? t : 0) * MS + j];
  for (int c = 0; c < nb; ++c) {
    const int k = k0 + c;
    uint32_t key[T], lo[T];
    int code[T];
    for (int t = 0; t < T; ++t) {
      uint64_t bits;
      memcpy(&bits, &P[t][c], 8);
      lo[t] = (uint32_t)bits;
      key[t] = ((uint32_t)(bits >> 32) & 0x7fffffffu) + 1u;
      if (P[t][c] != P[t][c]) key[t] = pq[t] == k ? 0xffffffffu : 0u;
      if (pq[t] < k) key[t] = 0u;
      code[t] = pq[t] * 256 + t;
    }
    double* set = ub + (c & 1) * 4 * CAND;
    for (int w = 0; w < 4; ++w) {
      uint32_t mk = 0, ml = 0;
      int best = -1;
      for (int l = 0; l < 64; ++l) mk = key[64 * w + l] > mk ? key[64 * w + l] : mk;
      for (int l = 0; l < 64; ++l)
        if (key[64 * w + l] == mk && lo[64 * w + l] > ml) ml = lo[64 * w + l];
      for (int l = 0; l < 64; ++l) {
        const int t = 64 * w + l;
        if (key[t] != mk) continue;
        if (mk == 0) {                       /* no candidate: the first lane */
          best = t;
          break;
        }
        if (lo[t] == ml && (best < 0 || code[t] < code[best])) best = t;
      }
      double* slot = set + w * CAND;
      const int32_t word[4] = {(int32_t)lo[best], (int32_t)mk, code[best], 0};
      memcpy(slot, word, 16);
      for (int j = c / 2 * 2; j < MB; ++j) slot[2 + j] = P[best][j];
    }
    int bw = 0, bc = 0;
    uint64_t bk = 0;
    for (int w = 0; w < 4; ++w) {
      int32_t word[4];
      memcpy(word, set + w * CAND, 16);
      const uint64_t kw = (uint64_t)(uint32_t)word[1] << 32 | (uint32_t)word[0];
      if (w == 0 || kw > bk || (kw == bk && word[2] < bc)) {
        bk = kw;
        bc = word[2];
        bw = w;
      }
    }
    const int pv = bc >> 8, qs = bc & 255;
    if (qs >> 6 != bw) abort();
    double z[MB];
    for (int j = 0; j < MB; ++j) z[j] = set[bw * CAND + 2 + j];
    const double akk = z[c];
    if (akk == 0.0 && !info) info = k + 1;
    for (int t = 0; t < T; ++t) {
      if (t == qs) pq[t] = k;
      else if (pq[t] == k) pq[t] = pv;
      const double l = P[t][c] / akk;
      const int below = pq[t] > k && akk != 0.0;
      if (below) P[t][c] = l;
      for (int j = c + 1; j < MB; ++j) P[t][j] = P[t][j] - z[j] * (below ? l : 0.0);
      if (t < n) M[k * ld + t] = P[t][c];
    }
  }
  return info;
}

static int lu_m(double* M, const double* J, double g, int n, int ld) {
  const int nt = ld <= 128 ? 2 : (ld <= 192 ? 3 : 4), ahead = nt < 4;
  const int np = (n + MB - 1) / MB;
  int info = 0;
  for (int t = 0; t < T; ++t) pq[t] = t < n ? t : -1;
  cols_load(J, n, ld, nt, 0);
  for (int p = 0; p < np; ++p) {
    const int k0 = p * MB, nb = imin(MB, n - k0), nblk = k0 / BK;
    cols_form(g, n, nt, k0);
    if (p > 0) {
      for (int t = 0; t < T; ++t)
        for (int s = 0; s < nt; ++s) PS[t][s] = (t & 63) + 64 * s < ld ? pos[(t & 63) + 64 * s] : -1;
#define AT(B) (imin(B, nblk - 1) * BK)
#define APPLY(I, B) for (int w = 0; w < 4; ++w) block_apply(w, nt, Q[I], (B) * BK)
      if (p == 1 || !ahead) mult_load(M, ld, nt, 0, Q[0]);
      if (ahead) {
        mult_load(M, ld, nt, BK, Q[1]);
        for (int bl = 0; bl < nblk; bl += 3) {
          mult_load(M, ld, nt, AT(bl + 2), Q[2]);
          APPLY(0, bl);
          mult_load(M, ld, nt, AT(bl + 3), Q[0]);
          if (bl + 1 < nblk) APPLY(1, bl + 1);
          mult_load(M, ld, nt, AT(bl + 4), Q[1]);
          if (bl + 2 < nblk) APPLY(2, bl + 2);
        }
      } else {
        for (int bl = 0; bl < nblk; bl += 2) {
          mult_load(M, ld, nt, AT(bl + 1), Q[1]);
          APPLY(0, bl);
          mult_load(M, ld, nt, AT(bl + 2), Q[0]);
          APPLY(1, bl + 1);
        }
      }
    }
    for (int t = 0; t < T; ++t)
      for (int s = 0; s < nt; ++s) {
        const int q = (t & 63) + 64 * s;
        if (q < n)
          for (int c = 0; c < 4; ++c) H[q * MS + 4 * (t >> 6) + c] = C[t][s][c];
      }
    if (p + 1 < np) cols_load(J, n, ld, nt, k0 + MB);
    if (ahead && p > 0) mult_load(M, ld, nt, 0, Q[0]);
    info = factor_m(M, n, ld, k0, nb, info);
    for (int t = 0; t < T; ++t)
      if (t < ld) pos[t] = pq[t];
  }
  return info;
}

static void solve_load(const double* M, int n, int ld, int k0, int fwd, double v[T][SB]) {
  for (int t = 0; t < T; ++t) {
    const int need = fwd ? pt[t] >= k0 : (pt[t] >= 0 && pt[t] < k0 + SB);
    const double* p = M + k0 * ld + (need ? t : 0);
    for (int j = 0; j < SB; ++j) {
      v[t][j] = *p;
      p += k0 + j + 1 < n ? ld : 0;
    }
  }
}

static void solve_block(int fwd, int part, int k0, int nb, double v[T][SB]) {
  for (int t = 0; t < T; ++t) {
    const int rel = pt[t] - k0;
    if (rel >= 0 && rel < SB) {
      for (int j = 0; j < SB; ++j) TS[rel * XS + j] = v[t][j];
      TS[rel * XS + SB] = acc[t];
    }
  }
  double lm[64][SB], xv[64], rdg[64], z[64];
  for (int t = 0; t < 64; ++t) {
    const int c = t & (SB - 1), r = imin(c, nb - 1);
    for (int j = 0; j < SB; ++j) lm[t][j] = TS[r * XS + j];
    xv[t] = c < nb ? TS[r * XS + SB] : 0.0;
    rdg[t] = fwd ? 1.0 : 1.0 / TS[r * (XS + 1)];
  }
  if (fwd) {
    for (int j = 0; j < SB - 1; ++j) {
      for (int t = 0; t < 64; ++t) z[t] = xv[(t & ~15) + j];
      for (int t = 0; t < 64; ++t) xv[t] = xv[t] - z[t] * ((t & 15) > j ? lm[t][j] : 0.0);
    }
  } else {
    for (int j = SB - 1; j >= 0; --j) {
      for (int t = 0; t < 64; ++t) z[t] = xv[(t & ~15) + j] * rdg[(t & ~15) + j];
      for (int t = 0; t < 64; ++t) xv[t] = xv[t] - z[t] * ((t & 15) < j && (!part || j < nb) ? lm[t][j] : 0.0);
    }
    for (int t = 0; t < 64; ++t) xv[t] = xv[t] * rdg[t];
  }
  for (int t = 0; t < SB; ++t) ub[t] = xv[t];
  for (int t = 0; t < T; ++t) {
    const int rel = pt[t] - k0;
    if (rel >= 0 && rel < SB) acc[t] = ub[rel];
    else if (fwd ? rel >= 0 : rel < 0)
      for (int j = 0; j < SB; ++j)
        if (!part || j < nb) acc[t] = acc[t] - v[t][j] * ub[j];
  }
}

static void solve_w(const double* M, int n, int ld) {
  const int nblk = (n + SB - 1) / SB;
  for (int t = 0; t < T; ++t) {
    pt[t] = t < n ? pos[t] : -1;
    acc[t] = t < n ? b[t] : 0.0;
  }
#define F(I, B) solve_load(M, n, ld, imin(B, nblk - 1) * SB, 1, V[I])
#define G(I, B) solve_load(M, n, ld, imax(B, 0) * SB, 0, V[I])
  F(0, 0);
  F(1, 1);
  for (int i = 0; i < nblk; i += 3) {
    F(2, i + 2);
    solve_block(1, 0, i * SB, imin(SB, n - i * SB), V[0]);
    F(0, i + 3);
    if (i + 1 < nblk) solve_block(1, 0, (i + 1) * SB, imin(SB, n - (i + 1) * SB), V[1]);
    F(1, i + 4);
    if (i + 2 < nblk) solve_block(1, 0, (i + 2) * SB, imin(SB, n - (i + 2) * SB), V[2]);
  }
  G(2, nblk - 1);
  G(0, nblk - 2);
  G(1, nblk - 3);
  solve_block(0, 1, (nblk - 1) * SB, n - (nblk - 1) * SB, V[2]);
  for (int i = nblk - 2; i >= 0; i -= 3) {
    G(2, i - 2);
    solve_block(0, 0, i * SB, SB, V[0]);
    G(0, i - 3);
    if (i - 1 >= 0) solve_block(0, 0, (i - 1) * SB, SB, V[1]);
    G(1, i - 4);
    if (i - 2 >= 0) solve_block(0, 0, (i - 2) * SB, SB, V[2]);
  }
  for (int t = 0; t < T; ++t)
    if (pt[t] >= 0) x[pt[t]] = acc[t];
}

static uint64_t rng = 0x9e3779b97f4a7c15ull;
static double urand(void) {
  rng ^= rng << 13;
  rng ^= rng >> 7;
  rng ^= rng << 17;
  return (double)(rng >> 11) * (1.0 / 9007199254740992.0) * 2.0 - 1.0;
}

static double* nans(size_t k) {
  double* p = (double*)malloc(sizeof(double) * k);
  for (size_t i = 0; i < k; ++i) p[i] = NAN;
  return p;
}

/* L U with L's rows in the order arr */
static void product(int n, double* A, int ties) {
  double* L = (double*)malloc(sizeof(double) * (size_t)n * n);
  double* U = (double*)malloc(sizeof(double) * (size_t)n * n);
  int* arr = (int*)malloc(sizeof(int) * n);
  for (int i = 0; i < n; ++i)
    for (int j = 0; j < n; ++j) {
      const double l = urand(), u = urand();
      L[i * n + j] = i == j ? 1.0 : (i < j ? 0.0 : (ties ? (l < 0 ? -1.0 : 1.0) : 0.5 * l));
      U[i * n + j] = i > j ? 0.0 : (i == j ? (ties ? (u < 0 ? -1.0 : 1.0) : 2.0 + fabs(u)) : (ties ? floor(u + 0.5) : u));
    }
  for (int i = 0; i < n; ++i) arr[i] = i;
  if (!ties)
    for (int k = n - 2; k >= 0; --k) {
      const int tmp = arr[k];
      arr[k] = arr[n - 1];
      arr[n - 1] = tmp;
    }
  for (int i = 0; i < n; ++i)
    for (int j = 0; j < n; ++j) {
      double v = 0.0;
      for (int q = 0; q < n; ++q) v += L[arr[i] * n + q] * U[q * n + j];
      A[i * n + j] = v;
    }
  free(L); free(U); free(arr);
}

int main(int argc, char** argv) {
  if (argc != 5) return 2;
  const int n_lo = atoi(argv[2]), n_hi = atoi(argv[3]), pattern = atoi(argv[4]);
  const double g = 2.5;
  if (n_lo < 65 || n_hi > 256 || n_lo > n_hi || pattern < 0 || pattern > 5) return 2;
  FILE* f = fopen(argv[1], "wb");
  if (!f) return 2;
  for (int n = n_lo; n <= n_hi; ++n) {
    const int ld = (n + 15) & ~15;
    const int two = 2 * LS * ld, m = MS * ld + 4 * BK * TW, region = two > m ? two : m;
    if (LS * ld + SB * XS > region || 2 * 4 * CAND > UB) return 3;
    double *M = nans((size_t)n * ld), *J = nans((size_t)n * ld);
    double *A = (double*)malloc(sizeof(double) * (size_t)n * n), *Fo = nans((size_t)n * n);
    H = nans((size_t)MS * ld);
    for (int w = 0; w < 4; ++w) TAB[w] = nans(BK * TW);
    TS = nans(SB * XS);
    ub = nans(UB);
    b = nans(ld);
    x = nans(ld);
    pos = (int*)malloc(sizeof(int) * ld);
    for (int i = 0; i < ld; ++i) pos[i] = 1 << 20;
    for (size_t i = 0; i < sizeof(C) / 8; ++i) ((double*)C)[i] = NAN;
    for (size_t i = 0; i < sizeof(Q) / 8; ++i) ((double*)Q)[i] = NAN;
    for (size_t i = 0; i < sizeof(V) / 8; ++i) ((double*)V)[i] = NAN;
    if (pattern == 1 || pattern == 5) {
      product(n, A, pattern == 5);
    } else {
      for (int i = 0; i < n; ++i)
        for (int j = 0; j < n; ++j) {
          double v = urand();
          if (pattern == 2) v = i == j ? 4.0 * n : v;
          if ((pattern == 3 && j == n - 1) || (pattern == 4 && j == n / 2)) v = 0.0;
          A[i * n + j] = v;
        }
    }
    for (int i = 0; i < n; ++i)
      for (int j = 0; j < n; ++j) {
        J[j * ld + i] = (i == j ? g : 0.0) - A[i * n + j];
        A[i * n + j] = (i == j ? g : 0.0) - J[j * ld + i];
      }
    const int info = lu_m(M, J, g, n, ld);
    for (int i = 0; i < n; ++i) b[i] = i + 1.0;
    if (info == 0) solve_w(M, n, ld);
    else for (int i = 0; i < n; ++i) x[i] = 0.0;
    for (int q = 0; q < n; ++q)
      for (int j = 0; j < n; ++j) Fo[pos[q] * n + j] = M[j * ld + q];
    const int hdr[3] = {n, ld, info};
    fwrite(hdr, sizeof(int), 3, f);
    fwrite(A, sizeof(double), (size_t)n * n, f);
    fwrite(Fo, sizeof(double), (size_t)n * n, f);
    fwrite(pos, sizeof(int), n, f);
    fwrite(x, sizeof(double), n, f);
    free(M); free(J); free(A); free(Fo); free(H); free(TS); free(ub); free(b); free(x); free(pos);
    for (int w = 0; w < 4; ++w) free(TAB[w]);
  }
  fclose(f);
  return 0;
}
