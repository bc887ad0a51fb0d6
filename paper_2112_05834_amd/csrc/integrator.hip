// Per-cell stiff chemistry integration on CDNA4 (gfx950).
//
// One cell is owned by a group of G lanes of a 64-wide wavefront (G = 64: one
// cell per wave; G = 16: four cells per wave), with G >= n = Ns + 1. Lane i
// of the group owns state component i (0 = T, 1..Ns = Y_1..Y_Ns) and row i of
// the Rosenbrock matrix M = I/(gamma h) - J, kept in registers. The analytical
// Jacobian is assembled row-wise in an LDS area, from the mechanism image that
// every block stages in LDS. The area is the group's own, or (33 to 55
// components) shared by two waves, which is what lets two waves run on a SIMD.
// After a rejected step J is formed again above 32 components with the default
// options, where it goes straight into M, and wherever the area is shared; a
// group's own area keeps it otherwise.
//
// Arithmetic per cell does not depend on G, on the cell's position in the
// grid or on the schedule: reductions follow one fixed pairing tree over 64
// virtual lanes, pivots are chosen by value then lowest position, and every
// other operation is per element in a fixed order.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <type_traits>

#include "device_common.hpp"
#include "kernels.hpp"

namespace chemk {

namespace {

using namespace dev;

// LDS add whose result is not returned: nothing waits on it
__device__ __forceinline__ void lds_add(double* p, double v) {
  __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
}

__device__ __forceinline__ double readlane_d(double v, int lane) {
  const int lo = __builtin_amdgcn_readlane(__double2loint(v), lane);
  const int hi = __builtin_amdgcn_readlane(__double2hiint(v), lane);
  return __hiloint2double(hi, lo);
}

// ---------------------------------------------------------------------------
// lane-group primitives (one cell per group of G lanes, G in {16, 32, 64})
// ---------------------------------------------------------------------------
// (every pattern used here reads a lane inside the same row, so no lane is
// out of bounds; bound_ctrl lets the compiler skip initialising the
// destination's old value)
template <int CTRL>
__device__ __forceinline__ double dpp_d(double v) {
  const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xf, 0xf, true);
  return __hiloint2double(hi, lo);
}
template <int CTRL>
__device__ __forceinline__ int dpp_i(int v) {
  return __builtin_amdgcn_mov_dpp(v, CTRL, 0xf, 0xf, true);
}
constexpr int kXor1 = 0xB1;        // quad_perm [1,0,3,2]
constexpr int kXor2 = 0x4E;        // quad_perm [2,3,0,1]
constexpr int kHalfMirror = 0x141; // lane i <-> 7-i within 8
constexpr int kMirror = 0x140;     // lane i <-> 15-i within 16
constexpr int kRowBcast15 = 0x142; // lane 15 of each row into the next row
constexpr int kRowBcast31 = 0x143; // lane 31 into rows 2 and 3

// v of lane SRC of each 16-lane row, to every lane of that row
template <int SRC>
__device__ __forceinline__ double row_bcast(double v) {
  const long long b = __builtin_amdgcn_update_dpp(0ll, __double_as_longlong(v), 0x150 + SRC, 0xf, 0xf, true);
  return __longlong_as_double(b);
}

// DPP move into the rows of ROWMASK only; the other rows keep old
template <int CTRL, int ROWMASK>
__device__ __forceinline__ double dpp_rows_d(double old, double v) {
  const int lo = __builtin_amdgcn_update_dpp(__double2loint(old), __double2loint(v), CTRL, ROWMASK, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(__double2hiint(old), __double2hiint(v), CTRL, ROWMASK, 0xf, false);
  return __hiloint2double(hi, lo);
}
template <int CTRL, int ROWMASK>
__device__ __forceinline__ int dpp_rows_i(int old, int v) {
  return __builtin_amdgcn_update_dpp(old, v, CTRL, ROWMASK, 0xf, false);
}

// f(integral constants 0 .. N - 1) in order
template <int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (N > 0) {
    static_for<N - 1>(f);
    f(std::integral_constant<int, N - 1>{});
  }
}

template <int G>
struct Grp {
  static_assert(G == 16 || G == 32 || G == 64, "group width");
  __device__ static __forceinline__ int lane() { return static_cast<int>(__lane_id()); }
  __device__ static __forceinline__ int gl() { return lane() & (G - 1); }
  __device__ static __forceinline__ int base() { return lane() & ~(G - 1); }

  // the two 16-lane rows of a 32-lane group: the even rows' value on both,
  // and the odd rows' (v_permlane16_swap, no LDS round trip)
  __device__ static __forceinline__ void rows_i(int v, int& even, int& odd) {
    const auto r = __builtin_amdgcn_permlane16_swap(static_cast<unsigned>(v), static_cast<unsigned>(v), false, false);
    even = static_cast<int>(r[0]);
    odd = static_cast<int>(r[1]);
  }
  __device__ static __forceinline__ void rows(double v, double& even, double& odd) {
    int el, ol, eh, oh;
    rows_i(__double2loint(v), el, ol);
    rows_i(__double2hiint(v), eh, oh);
    even = __hiloint2double(eh, el);
    odd = __hiloint2double(oh, ol);
  }
  // value of v in group lane SRC, known at compile time: a readlane, or DPP
  // inside the 16-lane row (and the other row's by a row swap)
  template <int SRC>
  __device__ static __forceinline__ double bcast_c(double v) {
    if constexpr (G == 64) {
      return readlane_d(v, SRC);
    } else {
      const double z = row_bcast<SRC & 15>(v);
      if constexpr (G == 16) return z;
      double even, odd;
      rows(z, even, odd);
      return SRC < 16 ? even : odd;
    }
  }

  // value of v in group lane src (src equal across the group)
  __device__ static __forceinline__ double bcast(double v, int src) {
    if constexpr (G == 64) {
      return readlane_d(v, __builtin_amdgcn_readfirstlane(src));
    } else {
      return __shfl(v, base() + src, 64);
    }
  }
  // Sum over the 64 virtual lanes of a cell (lanes beyond the group add +0)
  // with one pairing tree for every G: xor 1, xor 2, then the 8-lane and
  // 16-lane mirrors inside a DPP row, then rows (0+1) + (2+3). With one cell
  // per wave the rows are combined by DPP row broadcasts: row 3 ends with
  // (r3 + r2) + (r1 + r0), the same value as (r0 + r1) + (r2 + r3) in every
  // bit (IEEE addition commutes), read from lane 63.
  __device__ static __forceinline__ double sum(double x) {
    x = x + dpp_d<kXor1>(x);
    x = x + dpp_d<kXor2>(x);
    x = x + dpp_d<kHalfMirror>(x);
    x = x + dpp_d<kMirror>(x);
    if constexpr (G == 64) {
      x = x + dpp_rows_d<kRowBcast15, 0xA>(0.0, x);   // rows 1, 3: + row 0, row 2
      x = x + dpp_rows_d<kRowBcast31, 0xC>(0.0, x);   // rows 2, 3: + row 1
      return readlane_d(x, 63);
    } else if constexpr (G == 32) {
      double even, odd;
      rows(x, even, odd);
      return (even + odd) + (0.0 + 0.0);
    } else {
      return (x + 0.0) + (0.0 + 0.0);
    }
  }
  __device__ static __forceinline__ double max(double x) {
    x = fmax(x, dpp_d<kXor1>(x));
    x = fmax(x, dpp_d<kXor2>(x));
    x = fmax(x, dpp_d<kHalfMirror>(x));
    x = fmax(x, dpp_d<kMirror>(x));
    if constexpr (G == 64) {
      x = fmax(x, dpp_rows_d<kRowBcast15, 0xA>(x, x));
      x = fmax(x, dpp_rows_d<kRowBcast31, 0xC>(x, x));
      return readlane_d(x, 63);
    } else if constexpr (G == 32) {
      double even, odd;
      rows(x, even, odd);
      return fmax(even, odd);
    } else {
      return x;
    }
  }
  __device__ static __forceinline__ int min_i(int x) {
    x = ::min(x, dpp_i<kXor1>(x));
    x = ::min(x, dpp_i<kXor2>(x));
    x = ::min(x, dpp_i<kHalfMirror>(x));
    x = ::min(x, dpp_i<kMirror>(x));
    if constexpr (G == 64) {
      x = ::min(x, dpp_rows_i<kRowBcast15, 0xA>(x, x));
      x = ::min(x, dpp_rows_i<kRowBcast31, 0xC>(x, x));
      return __builtin_amdgcn_readlane(x, 63);
    } else if constexpr (G == 32) {
      int even, odd;
      rows_i(x, even, odd);
      return ::min(even, odd);
    } else {
      return x;
    }
  }
  // largest of one 32-bit key per lane
  __device__ static __forceinline__ unsigned max_u32(unsigned x) {
    x = ::max(x, static_cast<unsigned>(dpp_i<kXor1>(static_cast<int>(x))));
    x = ::max(x, static_cast<unsigned>(dpp_i<kXor2>(static_cast<int>(x))));
    x = ::max(x, static_cast<unsigned>(dpp_i<kHalfMirror>(static_cast<int>(x))));
    x = ::max(x, static_cast<unsigned>(dpp_i<kMirror>(static_cast<int>(x))));
    if constexpr (G == 64) {
      x = ::max(x, static_cast<unsigned>(dpp_rows_i<kRowBcast15, 0xA>(0, static_cast<int>(x))));
      x = ::max(x, static_cast<unsigned>(dpp_rows_i<kRowBcast31, 0xC>(0, static_cast<int>(x))));
      return static_cast<unsigned>(__builtin_amdgcn_readlane(static_cast<int>(x), 63));
    } else if constexpr (G == 32) {
      int even, odd;
      rows_i(static_cast<int>(x), even, odd);
      return ::max(static_cast<unsigned>(even), static_cast<unsigned>(odd));
    } else {
      return x;
    }
  }
  // group-relative ballot
  __device__ static __forceinline__ unsigned long long ballot(bool p) {
    const unsigned long long b = __ballot(p);
    if constexpr (G == 64) {
      return b;
    } else {
      return (b >> base()) & ((1ull << G) - 1ull);
    }
  }
  __device__ static __forceinline__ bool any(bool p) { return ballot(p) != 0ull; }
  // the group lane where p holds (p true on exactly one lane)
  __device__ static __forceinline__ int first(bool p) {
    return __ffsll(static_cast<long long>(ballot(p))) - 1;
  }
};

// A block's LDS after the mechanism image: one Jacobian J [NN*NN] row-major
// per cell, or per pair of waves that take turns with it (below), then every
// cell's own area: the per-species vectors C, gRT, hRT [NN each; entry ns is
// the absent species of the reaction records (C = 1, g = h = 0), entries
// after it are zero, so column loops run without a bound check] and a
// reaction/species buffer RB. RB holds, for state sizes up to 32, the
// per-reaction rate of progress (and with the Jacobian kf*theta, kr*theta,
// q0*dtheta/d[M], dq/dT) read by the species pass [max(5*nr, 3*NN)]; above 32
// only the species sums omega, d omega/dT and sum nu q0 dtheta/d[M] [3*NN]
// that the reaction lanes add into.
// P holds the LU's pivot rows, and D (up to 32) takes the adds that the species
// pass has no element for.
struct CellArea {
  double* J;
  double* P;
  double* D;
  double* RB;
  double* C;
  double* gRT;
  double* hRT;
};

// The LU's pivot rows of one panel, interleaved (column j's four entries side
// by side, up to a multiple of 16 columns), sit at the start of the cell's own
// area, which holds nothing between two right-hand sides.
constexpr int kPanel = 4;
__host__ __device__ constexpr int lu_rows_doubles(int nn) { return kPanel * ((nn + 15) & ~15); }
// one pivot row, its reciprocal and its position (several cells per wave)
__host__ __device__ constexpr int lu_row_doubles(int nn) { return ((nn + 15) & ~15) + 2; }
// state sizes above 32 assemble rates and Jacobian reaction by reaction
__host__ __device__ constexpr bool reaction_major(int nn) { return nn > 32; }
__host__ __device__ constexpr int rbuf_doubles(int nn, int nr) {
  return reaction_major(nn) ? 3 * nn : (5 * nr > 3 * nn ? 5 * nr : 3 * nn);
}
__host__ __device__ constexpr int cell_doubles_c(int nn, int nr) {
  const int vec = 3 * nn + rbuf_doubles(nn, nr) + (reaction_major(nn) ? 0 : 1);
  return ((vec > lu_rows_doubles(nn) ? vec : lu_rows_doubles(nn)) + 1) & ~1;
}
__host__ __device__ constexpr int j_doubles_c(int nn) { return (nn * nn + 1) & ~1; }
// Sizes whose waves may share a Jacobian buffer in pairs: one cell per wave,
// and two blocks of four waves, each with two buffers, fit the LDS of a CU.
__host__ __device__ constexpr bool can_share_j(int nn) { return nn > 32 && nn <= 55; }

template <int NN>
__device__ __forceinline__ CellArea cell_area(double* J, double* base, int nr) {
  CellArea c;
  c.J = J;
  c.C = base;
  c.gRT = base + NN;
  c.hRT = base + 2 * NN;
  c.RB = base + 3 * NN;
  c.P = base;
  c.D = c.RB + rbuf_doubles(NN, nr);
  return c;
}

// Reaction-major assembly (state sizes above 32, one cell per wave): the
// lane of reaction rx adds nu_i q to om[i], and with the Jacobian nu_i dq/dT
// to wT[i] and nu_i q0 dtheta/d[M] to td[i], for every species i of the
// reaction (nu_i = -order on the reactant side, +order on the product side,
// so a species on both sides gets two adds). With the Jacobian it also forms
// the concentration partials once, dq/dC_j = kf theta dPf_j for reactants
// and -kr theta dPr_j for products, and adds nu_i dq/dC_j to J(1+i, 1+j) for
// every species i and j of the reaction, plus nu_i (alpha_k - 1) q0
// dtheta/d[M] for the listed third-body efficiencies. LDS adds that return
// nothing; the lane-to-reaction mapping is fixed, so the order of the adds
// into each element is fixed.
template <int NN, bool JAC>
__device__ __forceinline__ void rx_scatter(const MechLds& L, const double* C, const uint4 w, const RateOut& r,
                                           double* om, double* wT, double* td, double* J) {
  const int nre = (w.x >> 24) & 0xf, npr = (w.y >> 24) & 0xf;
  const int type = (w.x >> 28) & 3;
  double nu[6];
  int row[6];
  bool cv[6];
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    cv[j] = j < nre;
    cv[3 + j] = j < npr;
    row[j] = cv[j] ? (w.x >> (8 * j)) & 0xff : 0;
    row[3 + j] = cv[3 + j] ? (w.y >> (8 * j)) & 0xff : 0;
    nu[j] = -static_cast<double>((w.z >> (4 * j)) & 0xf);
    nu[3 + j] = static_cast<double>((w.z >> (12 + 4 * j)) & 0xf);
  }
#pragma unroll
  for (int a = 0; a < 6; ++a) {
    if (!cv[a]) continue;
    lds_add(&om[row[a]], nu[a] * r.q);
    if (JAC) {
      lds_add(&wT[row[a]], nu[a] * r.dqdT);
      if (type >= 1) lds_add(&td[row[a]], nu[a] * r.q0b);
    }
  }
  if (!JAC) return;
  double Pf, Pr, dPf[3], dPr[3];
  int sf[3], sr[3];
  mass_action(C, w.x, w.z, nre, Pf, dPf, sf);
  mass_action(C, w.y, w.z >> 12, npr, Pr, dPr, sr);
  double dq[6];
  int col[6];
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    dq[j] = r.kfT * dPf[j];
    dq[3 + j] = -(r.krT * dPr[j]);
    col[j] = sf[j];
    col[3 + j] = sr[j];
  }
#pragma unroll
  for (int a = 0; a < 6; ++a) {
    if (!cv[a]) continue;
    double* Jr = J + (1 + row[a]) * NN + 1;
#pragma unroll
    for (int b = 0; b < 6; ++b)
      if (cv[b]) lds_add(&Jr[col[b]], nu[a] * dq[b]);
  }
  if (type >= 1) {
    const int eoff = w.w & 0xffff, neff = (w.w >> 16) & 0xff;
    for (int e0 = 0; e0 < neff; e0 += kEffChunk) {
      int sp[kEffChunk];
      double am[kEffChunk];
#pragma unroll
      for (int q = 0; q < kEffChunk; ++q) {
        const int e = e0 + q < neff ? eoff + e0 + q : eoff;
        sp[q] = L.eff_sp[e];
        am[q] = L.eff_am1[e];
      }
#pragma unroll
      for (int a = 0; a < 6; ++a) {
        if (!cv[a]) continue;
        double* Jr = J + (1 + row[a]) * NN + 1;
        const double ab = nu[a] * r.q0b;
#pragma unroll
        for (int q = 0; q < kEffChunk; ++q)
          if (e0 + q < neff) lds_add(&Jr[sp[q]], ab * am[q]);
      }
    }
  }
}

// ---------------------------------------------------------------------------
// the Jacobian buffer that two waves of a block share
// ---------------------------------------------------------------------------
// A wave needs the buffer only from the start of a Jacobian's assembly until
// M = g I - J is in its registers, well under half of an attempted step, so
// two waves take turns with one. That halves the largest part of a cell's LDS
// and lets two waves run on every SIMD. The lock is a word of LDS (NULL: the
// buffer is the wave's own); a holder never waits for anything while it holds
// it, and gives it back on every path, so each wait ends. Both fences are for
// LDS only: a wave's global stores in flight need not end first.
__device__ __forceinline__ void j_acquire(int* lock) {
  if (!lock) return;
  for (;;) {
    int held = 0;
    if (__lane_id() == 0) held = __hip_atomic_exchange(lock, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    if (__builtin_amdgcn_readfirstlane(held) == 0) break;
    __builtin_amdgcn_s_sleep(8);
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}
__device__ __forceinline__ void j_release(int* lock) {
  if (!lock) return;
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  if (__lane_id() == 0) __hip_atomic_store(lock, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// ---------------------------------------------------------------------------
// one cell
// ---------------------------------------------------------------------------
template <int NN, int G>
struct Cell {
  static_assert(G >= NN, "one state component per lane");
  using Gp = Grp<G>;
  // Reaction-major assembly of the production rates and the Jacobian for
  // state sizes above 32 (only 64-lane groups exist there); smaller sizes,
  // which also run several cells per wave, keep the species-major passes,
  // whose order of additions does not depend on the group width.
  static constexpr bool kScatter = reaction_major(NN);

  // Reactions from the packed records: one lane per reaction, in the order of
  // the general words and with the same operations per reaction, so that both
  // give the same bits. The reaction-major assembly adds into the species sums
  // and J (as rx_scatter); smaller sizes keep the rates in RB for the species
  // pass. The records hold what the general words make every lane decode: LDS
  // offsets of the species slots (one register serves C, g, h and the sums, by
  // instruction offsets), factors of the mass-action products without selects
  // on the orders, orders as doubles. Products by orders 1 and 2 are exact, so
  // they may be fused. Third slots and factors are handled only in blocks that
  // have any; there the B of a side 2A + B, which the record keeps in the third
  // slot, takes the second species' place in every sum, and the sums are formed
  // again (kept to this branch, the other blocks pay nothing: with the exchange
  // ahead of the sums 65536 54-species cells took 141.9 ms, so 140.1, without
  // it 140.3).
  template <bool JAC>
  __device__ static __forceinline__ void reactions(const MechArgs& A, const MechLds& L, const CellArea& ca, double T,
                                                   double rT, double lnT, double lnRTp, double Ctot) {
    const int i = Gp::gl(), nr = A.nr;
    const double2* rec = A.rec + i;
    const int N = A.rec_n;
    char* const Cb = reinterpret_cast<char*>(ca.C);
    char* const Jb = reinterpret_cast<char*>(ca.J + NN + 1);
    constexpr int kG = 8 * NN, kH = 16 * NN, kOm = 24 * NN, kWT = 32 * NN, kTd = 40 * NN;   // byte offsets from C
    const auto at = [&](unsigned off, int arr) { return *reinterpret_cast<const double*>(Cb + off + arr); };
#pragma nounroll
    for (int r0 = 0; r0 < nr; r0 += G, rec += G) {
      const double2 k1 = rec[0], k2 = rec[N], n0 = rec[2 * N];
      double2 n1 = rec[3 * N];
      const uint4 w0 = reinterpret_cast<const uint4*>(rec)[5 * N];
      const int type = (w0.w >> 8) & 3;
      const bool rev = (w0.w >> 10) & 1;
      const bool third = __any(w0.w & (4u | 32u | 64u));    // uniform: a third slot or factor in this block
      double2 n2{0.0, 0.0};
      uint4 w1{0, 0, 0, 0};
      if (__any(type != 0) || third) w1 = reinterpret_cast<const uint4*>(rec)[6 * N];
      const unsigned f0 = w0.x & 0xffff, p0 = w0.y & 0xffff;
      unsigned f1 = w0.x >> 16, p1 = w0.y >> 16, f2 = 0, p2 = 0, on = w0.w;   // on: slots with a species
      const double cf0 = at(f0, 0), cp0 = at(p0, 0);
      const double cf1 = at(w0.z & 0xffff, 0), cp1 = at(w0.z >> 16, 0);
      const double lnkf = k1.x + k1.y * lnT - k2.x * rT;
      const double kf = exp(lnkf);
      // sum of nu v over slots 0 and 1 of both sides
      const auto sum01 = [&](int arr) {
        double v = fma(-n0.x, at(f0, arr), 0.0);
        v = fma(n0.y, at(p0, arr), v);
        v = fma(-n1.x, at(f1, arr), v);
        return fma(n1.y, at(p1, arr), v);
      };
      double sumg = sum01(kG), sumh = JAC ? sum01(kH) : 0.0;
      double Pf = cf0 * cf1, Pr = cp0 * cp1;
      double cf2 = 1.0, cp2 = 1.0;
      bool tf = false, tp = false;      // a side 2A + B: B is the second species, as in the general words
      if (third) {
        n2 = rec[4 * N];
        f2 = w1.x & 0xffff;
        p2 = w1.x >> 16;
        cf2 = at(w1.y & 0xffff, 0);
        cp2 = at(w1.y >> 16, 0);
        Pf = Pf * cf2;
        Pr = Pr * cp2;
        tf = (on & 6u) == 4u;
        tp = (on & 48u) == 32u;
        f1 = tf ? f2 : f1;
        p1 = tp ? p2 : p1;
        n1.x = tf ? n2.x : n1.x;
        n1.y = tp ? n2.y : n1.y;
        n2.x = tf ? 0.0 : n2.x;
        n2.y = tp ? 0.0 : n2.y;
        on ^= (tf ? 6u : 0u) | (tp ? 48u : 0u);
        sumg = fma(n2.y, at(p2, kG), fma(-n2.x, at(f2, kG), sum01(kG)));
        if (JAC) sumh = fma(n2.y, at(p2, kH), fma(-n2.x, at(f2, kH), sum01(kH)));
      }
      // kr = kf / Kc with Kc = exp(-sum nu g/RT) (p_atm/RT)^(sum nu)
      double kr = exp(fma(k2.y, lnRTp, lnkf + sumg));
      kr = rev ? kr : 0.0;
      const double q0 = kf * Pf - kr * Pr;
      const double dlnkf = (k1.y + k2.x * rT) * rT;
      double theta = 1.0, beta = 0.0, dthdT = 0.0;
      if (type >= 1) theta_of<JAC>(L, ca.C, type, w1.z, kf, dlnkf, T, rT, lnT, Ctot, theta, beta, dthdT);
      const double q = theta * q0;
      double kfT = 0.0, krT = 0.0, q0b = 0.0, dqdT = 0.0;
      if (JAC) {
        const double dlnkr = rev ? dlnkf - (sumh * rT - k2.y * rT) : 0.0;
        kfT = kf * theta;
        krT = kr * theta;
        q0b = q0 * beta;
        dqdT = theta * (kf * dlnkf * Pf - kr * dlnkr * Pr) + q0 * dthdT;
      }
      if constexpr (!kScatter) {
        const int rx = r0 + i;
        if (rx < nr) {
          ca.RB[rx] = q;
          if (JAC) {
            ca.RB[nr + rx] = kfT;
            ca.RB[2 * nr + rx] = krT;
            ca.RB[3 * nr + rx] = q0b;
            ca.RB[4 * nr + rx] = dqdT;
          }
        }
        continue;
      }
      // slots f0 f1 f2 p0 p1 p2: species sums, then J by row and column
      const double nu[6] = {-n0.x, -n1.x, -n2.x, n0.y, n1.y, n2.y};
      const unsigned off[6] = {f0, f1, f2, p0, p1, p2};
      const auto each = [&](auto&& fn) {
#pragma unroll
        for (int a = 0; a < 6; ++a) {
          if (a % 3 == 2 && !third) continue;
          if (on & (1u << a)) fn(a);
        }
      };
      each([&](int a) {
        double* om = reinterpret_cast<double*>(Cb + off[a] + kOm);
        lds_add(om, nu[a] * q);
        if (JAC) {
          lds_add(om + NN, nu[a] * dqdT);
          if (type >= 1) lds_add(om + 2 * NN, nu[a] * q0b);
        }
      });
      if (JAC) {
        double dq[6];
        dq[0] = kfT * (n0.x * cf1);
        dq[1] = kfT * cf0;
        dq[3] = -(krT * (n0.y * cp1));
        dq[4] = -(krT * cp0);
        dq[2] = dq[5] = 0.0;
        if (third) {
          dq[0] = kfT * (n0.x * cf1 * cf2);
          dq[1] = kfT * (cf0 * (tf ? cf1 : cf2));
          dq[2] = kfT * (cf0 * cf1);
          dq[3] = -(krT * (n0.y * cp1 * cp2));
          dq[4] = -(krT * (cp0 * (tp ? cp1 : cp2)));
          dq[5] = -(krT * (cp0 * cp1));
        }
        each([&](int a) {
          char* Jr = Jb + off[a] * NN;
#pragma unroll
          for (int b = 0; b < 6; ++b) {
            if (b % 3 == 2 && !third) continue;
            if (on & (1u << b)) lds_add(reinterpret_cast<double*>(Jr + off[b]), nu[a] * dq[b]);
          }
        });
        if (type >= 1) {
          const int eoff = w1.z & 0xffff, neff = (w1.z >> 16) & 0xff;
          for (int e0 = 0; e0 < neff; e0 += kEffChunk) {
            int sp[kEffChunk];
            double am[kEffChunk];
#pragma unroll
            for (int c = 0; c < kEffChunk; ++c) {
              const int e = e0 + c < neff ? eoff + e0 + c : eoff;
              sp[c] = 8 * L.eff_sp[e];
              am[c] = L.eff_am1[e];
            }
            each([&](int a) {
              char* Jr = Jb + off[a] * NN;
              const double ab = nu[a] * q0b;
#pragma unroll
              for (int c = 0; c < kEffChunk; ++c)
                if (e0 + c < neff) lds_add(reinterpret_cast<double*>(Jr + sp[c]), ab * am[c]);
            });
          }
        }
      }
    }
  }

  // Production rate and Jacobian row of one species (this lane's) from the
  // rates in RB, entry by entry of its reaction list: the partial derivatives
  // by the record's factors, added in the order of the general words. The next
  // entry's record is fetched before the current one is used.
  __device__ static __forceinline__ void species_row(const MechArgs& A, const MechLds& L, const CellArea& ca,
                                                     double* Jrow, int e0, int e1, double& om, double& wT,
                                                     double& td) {
    const int nr = A.nr, N = A.rec_n;
    const char* const Cb = reinterpret_cast<const char*>(ca.C);
    char* const Jb = reinterpret_cast<char*>(Jrow);
    const auto at = [&](unsigned off) { return *reinterpret_cast<const double*>(Cb + off); };
    const auto add = [&](unsigned off, double v) { lds_add(reinterpret_cast<double*>(Jb + off), v); };
    if (e0 >= e1) return;
    unsigned ent = L.sp_ent[e0];
    const double2* rec = A.rec + (ent & 0xfff);
    uint4 w0 = reinterpret_cast<const uint4*>(rec)[5 * N];
    double2 n0 = rec[2 * N];
#pragma nounroll
    for (int e = e0; e < e1; ++e) {
      const int rx = ent & 0xfff;
      const double nu = static_cast<double>(static_cast<int>(ent >> 12) - 8);
      const uint4 w = w0;
      const double2 n = n0;
      const double2* const cur = rec;
      ent = e + 1 < e1 ? L.sp_ent[e + 1] : ent;
      rec = A.rec + (ent & 0xfff);
      w0 = reinterpret_cast<const uint4*>(rec)[5 * N];
      n0 = rec[2 * N];
      const unsigned f0 = w.x & 0xffff, f1 = w.x >> 16, p0 = w.y & 0xffff, p1 = w.y >> 16;
      const double cf0 = at(f0), cp0 = at(p0), cf1 = at(w.z & 0xffff), cp1 = at(w.z >> 16);
      const double qr = ca.RB[rx], kfT = ca.RB[nr + rx], krT = ca.RB[2 * nr + rx], q0b = ca.RB[3 * nr + rx],
                   dqdT = ca.RB[4 * nr + rx];
      om = om + nu * qr;
      wT = wT + nu * dqdT;
      const double af = nu * kfT, ar = nu * krT;
      const int type = (w.w >> 8) & 3;
      uint4 w1{0, 0, 0, 0};
      if (type != 0 || (w.w & (4u | 32u | 64u))) w1 = reinterpret_cast<const uint4*>(cur)[6 * N];
      if (w.w & (4u | 32u | 64u)) {
        const double cf2 = at(w1.y & 0xffff), cp2 = at(w1.y >> 16);
        add(f0, af * (n.x * cf1 * cf2));
        if (w.w & 2u) add(f1, af * (cf0 * cf2));
        if (w.w & 4u) add(w1.x & 0xffff, af * (cf0 * cf1));
        add(p0, -(ar * (n.y * cp1 * cp2)));
        if (w.w & 16u) add(p1, -(ar * (cp0 * cp2)));
        if (w.w & 32u) add(w1.x >> 16, -(ar * (cp0 * cp1)));
      } else {
        add(f0, af * (n.x * cf1));
        if (w.w & 2u) add(f1, af * cf0);
        add(p0, -(ar * (n.y * cp1)));
        if (w.w & 16u) add(p1, -(ar * cp0));
      }
      if (type >= 1) {
        const double ab = nu * q0b;
        td = td + ab;
        const int eoff = w1.z & 0xffff, neff = (w1.z >> 16) & 0xff;
        for (int c = 0; c < neff; ++c) add(8 * L.eff_sp[eoff + c], ab * L.eff_am1[eoff + c]);
      }
    }
  }

  // The reaction-major assembly from the general records (any orders).
  template <bool JAC>
  __device__ static __forceinline__ void reactions_general(const MechArgs& A, const MechLds& L, const CellArea& ca,
                                                           double T, double rT, double lnT, double lnRTp,
                                                           double Ctot) {
    const int nr = A.nr, i = Gp::gl();
    double* const om = ca.RB;
#pragma nounroll
    for (int rx = i; rx < nr; rx += G) {
      const uint4 w = L.rint[rx];
      const RateOut r = reaction_rate<JAC, false>(L, w, ca.C, ca.gRT, ca.hRT, ca.RB, nr, rx, T, rT, lnT, lnRTp, Ctot);
      rx_scatter<NN, JAC>(L, ca.C, w, r, om, om + NN, om + 2 * NN, ca.J);
    }
  }

  // f = dy/dt at y (this lane's component); with JAC also the analytical
  // Jacobian df/dy: written row-major into ca.J (complete on return), or with
  // TOM straight into M = g I - J, this lane's row in registers. jlock guards
  // a shared ca.J: it is taken before the first write of ca.J, and given back
  // once M is formed, or (without TOM) by the caller.
  template <bool JAC>
  __device__ static __forceinline__ double rhs(const MechArgs& A, const MechLds& L, const CellArea& ca, double p,
                                               double y, int* jlock = nullptr) {
    double none[NN];
    return eval<JAC, false>(A, L, ca, p, y, jlock, 0.0, none);
  }

  template <bool JAC, bool TOM>
  __device__ static __forceinline__ double eval(const MechArgs& A, const MechLds& L, const CellArea& ca, double p,
                                                double y, int* jlock, double g, double (&M)[NN]) {
    const int ns = A.ns, nr = A.nr;
    const int i = Gp::gl();                 // state component of this lane
    const bool sp = i >= 1 && i <= ns;      // lane holds species i-1
    const int s = sp ? i - 1 : 0;
    const double T = Gp::template bcast_c<0>(y);
    const double rT = 1.0 / T;
    // ln T and ln(RT/p_atm) by one logarithm, on lanes 0 and 1
    const double lns = log(i == 1 ? kR * T / kPatm : T);
    const double lnT = Gp::template bcast_c<0>(lns), lnRTp = Gp::template bcast_c<1>(lns);
    // mixture state
    const double Ys = sp ? y : 0.0;
    const double rWs = sp ? L.rW[s] : 0.0;
    const double invWbar = Gp::sum(Ys * rWs);
    const double Wbar = 1.0 / invWbar;
    const double rho = p * Wbar / (kR * T);
    const double Cs = rho * Ys * rWs;
    const double Ctot = Gp::sum(Cs);
    // species thermo (NASA-7, range by T < Tmid)
    double cpR = 0.0, hRT = 0.0, dcpR = 0.0;
    if (sp) {
      double gRT;
      nasa7<JAC>(A.nasa + 16 * s, T, rT, lnT, cpR, hRT, gRT, dcpR);
      ca.C[s] = Cs;
      ca.gRT[s] = gRT;
      ca.hRT[s] = hRT;
    } else if (i < NN) {
      // the absent species, and the padding components of a padded state size
      const int k = i == 0 ? NN - 1 : i - 1;
      ca.C[k] = k == ns ? 1.0 : 0.0;
      ca.gRT[k] = 0.0;
      ca.hRT[k] = 0.0;
    }
    const double cp = Gp::sum(Ys * cpR * kR * rWs);
    double dcp = 0.0;
    // species sums of the reaction-major assembly
    double* const som = ca.RB;
    double* const swT = ca.RB + NN;
    double* const std_ = ca.RB + 2 * NN;
    if (kScatter && i < NN) {
      som[i] = 0.0;
      if (JAC) {
        swT[i] = 0.0;
        std_[i] = 0.0;
      }
    }
    if (JAC) {
      dcp = Gp::sum(Ys * dcpR * kR * rWs);
      j_acquire(jlock);
      if constexpr (kScatter) {
        double2* z = reinterpret_cast<double2*>(ca.J);
#pragma unroll
        for (int e = 0; e < j_doubles_c(NN) / 2; e += 64)
          if (e + 64 <= j_doubles_c(NN) / 2 || e + i < j_doubles_c(NN) / 2) z[e + i] = double2{0.0, 0.0};
      } else if (i < NN) {
#pragma unroll
        for (int j = 0; j < NN; ++j) ca.J[i * NN + j] = 0.0;
      }
    }
    wsync();

    // ---- reactions: one lane per reaction ----
    if constexpr (kScatter) {
      if (A.rec) {
        reactions<JAC>(A, L, ca, T, rT, lnT, lnRTp, Ctot);
      } else {
        reactions_general<JAC>(A, L, ca, T, rT, lnT, lnRTp, Ctot);
      }
    } else {
      if (A.rec) {
        reactions<JAC>(A, L, ca, T, rT, lnT, lnRTp, Ctot);
      } else {
        for (int rx = i; rx < nr; rx += G)
          reaction_rate<JAC>(L, ca.C, ca.gRT, ca.hRT, ca.RB, nr, rx, T, rT, lnT, lnRTp, Ctot);
      }
    }
    wsync();

    // ---- species: production rates (and sparse Jacobian rows d omega/dC) ----
    // Above 32 state components the sums were formed by the reaction lanes
    // and are read back. Otherwise each species lane walks its reactions'
    // records; the Jacobian row is accumulated with LDS adds that return
    // nothing (the lane owns its row, and one wave's LDS operations execute
    // in order, so the sum order is the program order), and the next
    // entry's records are fetched before the current one is processed.
    double om = 0.0, wT = 0.0, td = 0.0;
    if (kScatter) {
      if (sp) {
        om = som[s];
        if (JAC) {
          wT = swT[s];
          td = std_[s];
        }
      }
    } else if (sp) {
      const int e0 = L.sp_off[s], e1 = L.sp_off[s + 1];
      double* Jrow = ca.J + i * NN + 1;
      if (!JAC) {
#pragma unroll 4
        for (int e = e0; e < e1; ++e) {
          const unsigned ent = L.sp_ent[e];
          const double nu = static_cast<double>(static_cast<int>(ent >> 12) - 8);
          om = om + nu * ca.RB[ent & 0xfff];
        }
      } else if (A.rec) {
        species_row(A, L, ca, Jrow, e0, e1, om, wT, td);
      } else {
        unsigned ent = e0 < e1 ? L.sp_ent[e0] : 0u;
        uint4 w = L.rint[ent & 0xfff];
        for (int e = e0; e < e1; ++e) {
          const int rx = ent & 0xfff;
          const double nu = static_cast<double>(static_cast<int>(ent >> 12) - 8);
          const uint4 wc = w;
          // prefetch the next entry
          const unsigned ent_n = e + 1 < e1 ? L.sp_ent[e + 1] : ent;
          double qr = ca.RB[rx], kfT = ca.RB[nr + rx], krT = ca.RB[2 * nr + rx];
          double q0b = ca.RB[3 * nr + rx], dqdT = ca.RB[4 * nr + rx];
          asm volatile("" : "+v"(qr), "+v"(kfT), "+v"(krT), "+v"(q0b), "+v"(dqdT));
          const int nre = (wc.x >> 24) & 0xf, npr = (wc.y >> 24) & 0xf;
          double Pf, Pr, dPf[3], dPr[3];
          int sf[3], sr[3];
          mass_action(ca.C, wc.x, wc.z, nre, Pf, dPf, sf);
          mass_action(ca.C, wc.y, wc.z >> 12, npr, Pr, dPr, sr);
          w = L.rint[ent_n & 0xfff];
          ent = ent_n;
          om = om + nu * qr;
          wT = wT + nu * dqdT;
          const double af = nu * kfT, ar = nu * krT;
#pragma unroll
          for (int j = 0; j < 3; ++j) lds_add(j < nre ? &Jrow[sf[j]] : ca.D, af * dPf[j]);
#pragma unroll
          for (int j = 0; j < 3; ++j) lds_add(j < npr ? &Jrow[sr[j]] : ca.D, -(ar * dPr[j]));
          const int type = (wc.x >> 28) & 3;
          if (type >= 1) {
            const double ab = nu * q0b;
            td = td + ab;
            const int eoff = wc.w & 0xffff, neff = (wc.w >> 16) & 0xff;
            for (int q = 0; q < neff; ++q) lds_add(&Jrow[L.eff_sp[eoff + q]], ab * L.eff_am1[eoff + q]);
          }
        }
      }
    }
    const double fY = sp ? A.W[s] * om / rho : 0.0;
    const double Q = Gp::sum(hRT * kR * T * om);
    const double rcp = rho * cp;
    const double fT = -Q / rcp;
    const double f = (i == 0) ? fT : fY;
    if (!JAC) return f;

    // ---- Jacobian: chain rule from d(omega)/dC, d(omega)/dT to y = (T, Y) ----
    wsync();
    double sv = 0.0;
    if (sp) {
      const double* Jrow = ca.J + i * NN + 1;
      double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
      // columns from ns on are zero in J
#pragma unroll
      for (int k = 0; k < NN - 1; k += 4) {
        a0 = fma(Jrow[k], ca.C[k], a0);
        if (k + 1 < NN - 1) a1 = fma(Jrow[k + 1], ca.C[k + 1], a1);
        if (k + 2 < NN - 1) a2 = fma(Jrow[k + 2], ca.C[k + 2], a2);
        if (k + 3 < NN - 1) a3 = fma(Jrow[k + 3], ca.C[k + 3], a3);
      }
      sv = ((a0 + a1) + (a2 + a3)) + td * Ctot;
    }
    const double HS = Gp::sum(hRT * sv);
    const double HT = Gp::sum(hRT * td);
    const double dQdT = Gp::sum(sp ? cpR * kR * om + hRT * kR * T * (wT - sv / T) : 0.0);
    // T-row entry of column i (species i-1): lane i sums column i of D
    double JT = 0.0;
    if (sp) {
      double c0 = 0.0, c1 = 0.0, c2 = 0.0, c3 = 0.0;
      // rows beyond species ns - 1 are zero in J and in hRT
#pragma unroll
      for (int q = 0; q < NN - 1; q += 4) {
        c0 = fma(ca.hRT[q], ca.J[(1 + q) * NN + i], c0);
        if (q + 1 < NN - 1) c1 = fma(ca.hRT[q + 1], ca.J[(2 + q) * NN + i], c1);
        if (q + 2 < NN - 1) c2 = fma(ca.hRT[q + 2], ca.J[(3 + q) * NN + i], c2);
        if (q + 3 < NN - 1) c3 = fma(ca.hRT[q + 3], ca.J[(4 + q) * NN + i], c3);
      }
      const double cs = (c0 + c1) + (c2 + c3);
      const double dQdY = kR * T * ((rho * rWs) * (cs + HT) - (Wbar * rWs) * HS);
      const double drcp = rho * cpR * kR * rWs - rcp * Wbar * rWs;
      JT = -(dQdY + fT * drcp) / rcp;
    }
    wsync();
    const double Wi_rho = sp ? A.W[s] / rho : 0.0;
    const double JcT = sp ? Wi_rho * (wT - sv / T) + fY / T
                          : (i == 0 ? -(dQdT + fT * (-rcp / T + rho * dcp)) / rcp : 0.0);   // column 0
    // rW is zero from ns on (up to 64 entries), which keeps the padding
    // columns of J zero
    if constexpr (TOM) {
      // The column factors rho/W_k, Wbar/W_k and 1/W_k, formed once by lane
      // k, are read back as broadcasts; -J goes straight into the rows of M,
      // g is added on the diagonal (one lane per instruction), and lane 0
      // reads its row, the T row, from where the other lanes left it.
      double* const fac = ca.C;     // C, g and h are not needed any more
      const double rWi = i < NN - 1 ? L.rW[i] : 0.0;
      if (i < NN - 1) *reinterpret_cast<double2*>(fac + 2 * i) = double2{rho * rWi, Wbar * rWi};
      if (sp) ca.J[i] = -JT;
      wsync();
      const double fYW = fY * Wbar;
      M[0] = -JcT;
      if (i < NN) {
        const double* Jrow = ca.J + i * NN;
#pragma unroll
        for (int k = 0; k < NN - 1; ++k) {
          const double2 ab = *reinterpret_cast<const double2*>(fac + 2 * k);
          const double D = Jrow[1 + k] + td;
          const double dw = ab.x * D - ab.y * sv;
          M[1 + k] = -(Wi_rho * dw + fYW * L.rW[k]);
        }
        if (i == 0) {
#pragma unroll
          for (int k = 1; k < NN; ++k) M[k] = ca.J[k];
        }
      } else {
#pragma unroll
        for (int k = 1; k < NN; ++k) M[k] = 0.0;
      }
      j_release(jlock);
      static_for<NN>([&](auto jc) {
        constexpr int j = decltype(jc)::value;
        add_on_lane<j>(M[j], g);
      });
    } else {
      if (sp) {
        double* Jrow = ca.J + i * NN;
#pragma unroll
        for (int k = 0; k < NN - 1; ++k) {
          const double rWk = L.rW[k];
          const double D = Jrow[1 + k] + td;
          const double dw = (rho * rWk) * D - (Wbar * rWk) * sv;
          Jrow[1 + k] = Wi_rho * dw + fY * Wbar * rWk;
        }
        ca.J[i] = JT;
      }
      if (sp || i == 0) ca.J[i * NN] = JcT;
      wsync();
    }
    return f;
  }

  // v += g on lane J alone (all 64 lanes active before and after)
  template <int J>
  __device__ static __forceinline__ void add_on_lane(double& v, double g) {
    asm volatile("s_bfm_b64 exec, 1, %2\n\tv_add_f64 %0, %0, %1\n\ts_mov_b64 exec, -1" : "+v"(v) : "v"(g), "n"(J));
  }

  // Without the bath gas (the last species, lane ns) its mass fraction is
  // 1 - the sum of the other species: this lane's value, with lane ns
  // replaced by that.
  __device__ static __forceinline__ double with_bath(int ns, double v) {
    const int i = Gp::gl();
    const double s = Gp::sum((i >= 1 && i < ns) ? v : 0.0);
    return i == ns ? 1.0 - s : v;
  }

  // The Jacobian of the state without the bath gas, from the full one in
  // ca.J: by the chain rule through Y_bath = 1 - sum_j Y_j every species
  // column loses the bath column. The bath's row and column are cleared, so
  // that its row of M is g e_ns, decoupled from the others.
  __device__ static __forceinline__ void reduce_bath(const CellArea& ca, int ns) {
    const int i = Gp::gl();
    wsync();
    if (i < ns) {
      double* Jr = ca.J + i * NN;
      const double jb = Jr[ns];
#pragma unroll
      for (int j = 1; j < NN; ++j)
        if (j < ns) Jr[j] = Jr[j] - jb;
      Jr[ns] = 0.0;
    } else if (i == ns) {
#pragma unroll
      for (int j = 0; j < NN; ++j) ca.J[i * NN + j] = 0.0;
    }
    wsync();
  }

  // one column into the last of M, the others moving up
  __device__ static __forceinline__ void shift_in(double (&M)[NN], double v) {
    static_for<NN - 1>([&](auto kc) { M[decltype(kc)::value] = M[decltype(kc)::value + 1]; });
    M[NN - 1] = v;
  }

  // Jacobian by forward differences: one more right-hand side per integrated
  // component (f0 = f(y) given). Every lane holds its component of the
  // perturbed state; lane j adds the increment. Without the bath gas the
  // perturbed state's bath lane is derived again, so the columns are those of
  // the reduced system, and the bath's row stays zero. J is written row-major
  // into ca.J, or (regs) its columns are shifted into the registers of M, so that
  // a buffer that two waves share is not held through n right-hand sides:
  // held, the two ran one after the other (3000 cells, 41 and 55 components: 194
  // and 540 ms so, 116 and 318 through M; with buffers of their own and one wave
  // per SIMD 144 and 428). What both ways share stands outside the branches:
  // stores to M and to ca.J in the two arms of one are merged into stores by
  // address, and M goes to scratch.
  __device__ static __forceinline__ void fd_jacobian(const MechArgs& A, const MechLds& L, const CellArea& ca, double p,
                                                     double y, double f0, bool nb, bool regs, double (&M)[NN]) {
    const int ns = A.ns;
    const int n = nb ? ns : ns + 1;
    const int i = Gp::gl();
    if (!regs && i < NN) {
#pragma unroll
      for (int j = 0; j < NN; ++j) ca.J[i * NN + j] = 0.0;
    }
#pragma unroll
    for (int j = 0; j < NN; ++j) M[j] = 0.0;
#pragma nounroll
    for (int j = 0; j < n; ++j) {
      const double yj = Gp::bcast(y, j);
      const double yp = yj + fd_increment(yj);
      const double d = yp - yj;
      double ypert = i == j ? yp : y;
      if (nb) ypert = with_bath(ns, ypert);
      const double fj = rhs<false>(A, L, ca, p, ypert);
      const bool row = i < NN && !(nb && i == ns);
      const double v = (fj - f0) / d;
      if constexpr (can_share_j(NN)) shift_in(M, row ? v : 0.0);
      if (!regs && row) ca.J[i * NN + j] = v;
    }
    if constexpr (can_share_j(NN)) {
#pragma nounroll
      for (int j = n; j < NN; ++j) shift_in(M, 0.0);
    }
    wsync();
  }

  // -------------------------------------------------------------------------
  // LU with partial pivoting of the rows in registers (row = lane). Rows are
  // not moved during the elimination: pos tracks each row's LAPACK position,
  // so the pivot of column k is the largest |a| among rows at positions >= k,
  // ties to the lowest position, exactly as a row-swapping getrf. At the end
  // every row is sent to the lane of its position (one ds_permute per dword),
  // so on return lane k holds row k of the packed factors (L left of the
  // diagonal, unit diagonal implied; U from the diagonal on) and rdiag =
  // 1/U_kk; pos keeps the position this lane's original row went to (used to
  // permute right-hand sides). With piv, lane k also receives the position
  // interchanged with k. Returns the first singular column + 1.
  // -------------------------------------------------------------------------
  __device__ static __forceinline__ int lu(double (&M)[NN], int& pos, double& rdiag, double* P, int n, int* piv) {
    if constexpr (G == 64) {
      return lu_wave(M, pos, rdiag, P, n, piv);
    } else {
      return lu_group(M, pos, rdiag, P, n, piv);
    }
  }

  // One cell per wave: panels of kPanel columns. Inside a panel only the
  // panel's own columns are updated, each pivot-row element broadcast by two
  // readlanes. The panel's pivot rows then go through the cell's LDS buffer P
  // to every 16-lane row (lane l of a row reads columns 16 J + l), solve their
  // unit lower triangle there, and every later column takes its kPanel updates
  // as fused multiply-adds whose multiplicand is broadcast along the 16-lane
  // row by DPP inside the instruction: one instruction per element where the
  // readlane form needs three. Each element receives the same fused
  // multiply-adds in the same order as column by column.
  // pivot search of one column by value, then position (every special case:
  // ties, zero columns, non-finite entries). Candidates are the rows at
  // positions k .. n - 1 (the rows that pad the matrix stay where they are), and
  // the lane returned always holds one, so that the positions stay a permutation
  // of the rows: a NaN is not chosen while another candidate compares, and where
  // none does the row at position k stays.
  __device__ static __forceinline__ int pivot_exact(double a, int pos, int k, int n, double& amax) {
    const bool cand = pos >= k && (pos < n || k >= n);
    const double key = cand ? fabs(a) : -1.0;
    amax = Gp::max(key);
    const bool tie = cand && key == amax;
    const int pmin = Gp::min_i(tie ? pos : kBig);
    return Gp::first(pos == (pmin < kBig ? pmin : k));
  }

  __device__ static __forceinline__ int lu_wave(double (&M)[NN], int& pos, double& rdiag, double* P, int n, int* piv) {
    unsigned long long zeros = 0;              // columns without a nonzero candidate
    const int i = Gp::lane();
    pos = i < NN ? i : -1;
    rdiag = 0.0;
    static_for<(NN + kPanel - 1) / kPanel>([&](auto pc) {
      constexpr int p0 = decltype(pc)::value * kPanel;
      constexpr int nb = NN - p0 < kPanel ? NN - p0 : kPanel;
      int own[kPanel];
      double ln[kPanel];                       // minus the multipliers (0 on rows above)
#pragma unroll
      for (int c = 0; c < nb; ++c) {
        const int k = p0 + c;
        const double a = M[k];
        // every lane forms its own element's reciprocal, beside the search
        // rather than after it: the hardware reciprocal refined by two Newton
        // steps (a shorter dependent chain than a correctly rounded division)
        double ra = __builtin_amdgcn_rcp(a);
        ra = fma(ra, fma(-a, ra, 1.0), ra);
        ra = fma(ra, fma(-a, ra, 1.0), ra);
        // the high words of |a| order the candidates except where they tie;
        // ties, zeros and non-finite entries take the exact search
        const unsigned hi = static_cast<unsigned>(__double2hiint(a)) & 0x7fffffffu;
        const unsigned key = pos >= k ? hi : 0u;
        const unsigned hmax = Gp::max_u32(key);
        const unsigned long long bal = __ballot(key == hmax);
        int owner = __builtin_ctzll(bal);
        double rp;
        if (__builtin_expect((bal & (bal - 1)) == 0 && hmax < 0x7ff00000u, 1)) {
          rp = readlane_d(ra, owner);
        } else {
          double amax;
          owner = __builtin_amdgcn_readfirstlane(pivot_exact(a, pos, k, n, amax));
          rp = readlane_d(ra, owner);
          if (amax == 0.0) {
            zeros |= 1ull << k;
            rp = 0.0;
          }
        }
        own[c] = owner;
        const int ppos = __builtin_amdgcn_readlane(pos, owner);
        pos = pos == k ? ppos : pos;
        pos = i == owner ? k : pos;
        if (piv) *piv = i == k ? ppos : *piv;
        rdiag = i == k ? rp : rdiag;
        const bool below = pos > k;
        const double l = below ? a * rp : 0.0;
        M[k] = below ? l : a;
        ln[c] = -l;
        // formed here, not carried along as masks and products
        asm volatile("" : "+v"(M[k]), "+v"(rdiag), "+v"(ln[c]));
#pragma unroll
        for (int j = k + 1; j < p0 + nb; ++j) M[j] = fma(ln[c], readlane_d(M[j], owner), M[j]);
      }
      if constexpr (p0 + kPanel < NN) {
        constexpr int j0 = p0 + kPanel;        // first column right of the panel
        const int r = pos - p0;
        if (static_cast<unsigned>(r) < static_cast<unsigned>(kPanel)) {
          double* row = P + r;
#pragma unroll
          for (int j = j0; j < NN; ++j) row[kPanel * j] = M[j];
        }
        // multipliers among the pivot rows (negated)
        const double n10 = readlane_d(ln[0], own[1]);
        const double n20 = readlane_d(ln[0], own[2]), n21 = readlane_d(ln[1], own[2]);
        const double n30 = readlane_d(ln[0], own[3]), n31 = readlane_d(ln[1], own[3]),
                     n32 = readlane_d(ln[2], own[3]);
        wsync();
        static_for<(NN + 15) / 16 - j0 / 16>([&](auto tc) {
          constexpr int J = j0 / 16 + decltype(tc)::value;
          const double* u = P + kPanel * (16 * J + (i & 15));
          const double x0 = u[0];
          double x1 = u[1], x2 = u[2], x3 = u[3];
          x1 = fma(n10, x0, x1);
          x2 = fma(n20, x0, x2);
          x3 = fma(n30, x0, x3);
          x2 = fma(n21, x1, x2);
          x3 = fma(n31, x1, x3);
          x3 = fma(n32, x2, x3);
          constexpr int ja = J * 16 > j0 ? J * 16 : j0;
          constexpr int jb = J * 16 + 16 < NN ? J * 16 + 16 : NN;
          static_for<(jb - ja + 3) / 4>([&](auto qc) {
            constexpr int j = ja + 4 * decltype(qc)::value;
            rank4<jb - j < 4 ? jb - j : 4, j & 15>(&M[j], x0, x1, x2, x3, ln);
          });
        });
        wsync();
      }
    });
    // rows to the lanes of their positions
    const int dst = 4 * (pos >= 0 ? pos : i);
#pragma unroll
    for (int j = 0; j < NN; ++j) M[j] = permute_d(M[j], dst);
    return zeros ? __builtin_ctzll(zeros) + 1 : 0;
  }

  // M[c] += sum_k l[k] (x_k of lane N + c of this 16-lane row), k ascending,
  // for NC columns. The leading s_nop covers the wait between a vector write
  // of x and its use as a DPP operand; the outputs are written before all inputs
  // are read, so they take registers of their own. The compiler does not see a
  // vector write here, so it adds no wait of its own behind the block: lane reads
  // of an output need one, and come only after the next panel's pivot search, which
  // works on the same block's first column.
  template <int NC, int N>
  __device__ static __forceinline__ void rank4(double* m, double x0, double x1, double x2, double x3,
                                               const double (&l)[kPanel]) {
#define CHEM_F(A, X, L, K) "v_fmac_f64_dpp " A ", " X ", " L " row_newbcast:" K " row_mask:0xf bank_mask:0xf\n\t"
    if constexpr (NC == 4) {
#define CHEM_R(X, L) CHEM_F("%0", X, L, "%12") CHEM_F("%1", X, L, "%13") CHEM_F("%2", X, L, "%14") CHEM_F("%3", X, L, "%15")
      asm("s_nop 1\n\t" CHEM_R("%4", "%8") CHEM_R("%5", "%9") CHEM_R("%6", "%10") CHEM_R("%7", "%11")
          : "+&v"(m[0]), "+&v"(m[1]), "+&v"(m[2]), "+&v"(m[3])
          : "v"(x0), "v"(x1), "v"(x2), "v"(x3), "v"(l[0]), "v"(l[1]), "v"(l[2]), "v"(l[3]), "n"(N), "n"(N + 1),
            "n"(N + 2), "n"(N + 3));
#undef CHEM_R
    } else if constexpr (NC == 3) {
#define CHEM_R(X, L) CHEM_F("%0", X, L, "%11") CHEM_F("%1", X, L, "%12") CHEM_F("%2", X, L, "%13")
      asm("s_nop 1\n\t" CHEM_R("%3", "%7") CHEM_R("%4", "%8") CHEM_R("%5", "%9") CHEM_R("%6", "%10")
          : "+&v"(m[0]), "+&v"(m[1]), "+&v"(m[2])
          : "v"(x0), "v"(x1), "v"(x2), "v"(x3), "v"(l[0]), "v"(l[1]), "v"(l[2]), "v"(l[3]), "n"(N), "n"(N + 1),
            "n"(N + 2));
#undef CHEM_R
    } else if constexpr (NC == 2) {
#define CHEM_R(X, L) CHEM_F("%0", X, L, "%10") CHEM_F("%1", X, L, "%11")
      asm("s_nop 1\n\t" CHEM_R("%2", "%6") CHEM_R("%3", "%7") CHEM_R("%4", "%8") CHEM_R("%5", "%9")
          : "+&v"(m[0]), "+&v"(m[1])
          : "v"(x0), "v"(x1), "v"(x2), "v"(x3), "v"(l[0]), "v"(l[1]), "v"(l[2]), "v"(l[3]), "n"(N), "n"(N + 1));
#undef CHEM_R
    } else {
#define CHEM_R(X, L) CHEM_F("%0", X, L, "%9")
      asm("s_nop 1\n\t" CHEM_R("%1", "%5") CHEM_R("%2", "%6") CHEM_R("%3", "%7") CHEM_R("%4", "%8")
          : "+&v"(m[0])
          : "v"(x0), "v"(x1), "v"(x2), "v"(x3), "v"(l[0]), "v"(l[1]), "v"(l[2]), "v"(l[3]), "n"(N));
#undef CHEM_R
    }
#undef CHEM_F
  }

  // Several cells per wave: column by column. The pivot row, its reciprocal
  // and its position go through the group's LDS buffer P to every 16-lane row
  // (lane l of a row reads columns 16 J + l), and each element's update is one
  // multiply-add whose pivot-row element is broadcast along the row by DPP: one
  // LDS round trip a column, where a lane shuffle per element needs two
  // through the LDS crossbar.
  __device__ static __forceinline__ int lu_group(double (&M)[NN], int& pos, double& rdiag, double* P, int n, int* piv) {
    constexpr int kRow = (NN + 15) & ~15;    // then the reciprocal and the position
    int info = 0;
    const int i = Gp::gl();
    pos = i < NN ? i : -1;
    rdiag = 0.0;
    static_for<NN>([&](auto kc) {
      constexpr int k = decltype(kc)::value;
      const double a = M[k];
      double ra = __builtin_amdgcn_rcp(a);
      ra = fma(ra, fma(-a, ra, 1.0), ra);
      ra = fma(ra, fma(-a, ra, 1.0), ra);
      const unsigned hi = static_cast<unsigned>(__double2hiint(a)) & 0x7fffffffu;
      const unsigned key = pos >= k ? hi : 0u;
      const unsigned hmax = Gp::max_u32(key);
      const unsigned long long bal = Gp::ballot(key == hmax);
      int owner = __builtin_ctzll(bal);
      bool zero = false;
      if (!__all((bal & (bal - 1)) == 0 && hmax < 0x7ff00000u)) {
        double amax;
        owner = pivot_exact(a, pos, k, n, amax);
        zero = amax == 0.0;
      }
      const bool is_owner = i == owner;
      wsync();
      if (is_owner) {
#pragma unroll
        for (int j = k + 1; j < NN; ++j) P[j] = M[j];
        P[kRow] = zero ? 0.0 : ra;
        P[kRow + 1] = __hiloint2double(0, pos);
      }
      wsync();
      const double rp = P[kRow];
      const int ppos = __double2loint(P[kRow + 1]);
      double u[kRow / 16];
#pragma unroll
      for (int J = (k + 1) / 16; J < kRow / 16; ++J) u[J] = P[16 * J + (i & 15)];
      if (zero && info == 0) info = k + 1;
      if (piv) *piv = i == k ? ppos : *piv;
      pos = pos == k ? ppos : pos;
      pos = is_owner ? k : pos;
      rdiag = is_owner ? rp : rdiag;
      const bool below = pos > k;
      double l = below ? a * rp : 0.0;
      M[k] = below ? l : a;
      // formed here, not carried along as masks and products
      asm volatile("" : "+v"(M[k]), "+v"(rdiag), "+v"(l), "+v"(pos));
      static_for<NN - 1 - k>([&](auto jc) {
        constexpr int j = k + 1 + decltype(jc)::value;
        M[j] = fma(-l, row_bcast<(j & 15)>(u[j / 16]), M[j]);
      });
    });
    wsync();      // the last row is read before the area holds anything else
    // rows to the lanes of their positions
    const int dst = 4 * (Gp::base() + (pos >= 0 ? pos : i));
#pragma unroll
    for (int j = 0; j < NN; ++j) M[j] = permute_d(M[j], dst);
    rdiag = permute_d(rdiag, dst);
    return info;
  }

  // lane gl() receives the value of the lane whose byte address it is sent to
  __device__ static __forceinline__ double permute_d(double v, int dst_addr) {
    const int lo = __builtin_amdgcn_ds_permute(dst_addr, __double2loint(v));
    const int hi = __builtin_amdgcn_ds_permute(dst_addr, __double2hiint(v));
    return __hiloint2double(hi, lo);
  }

  // Solve M x = b with the factors of lu(); b is this lane's equation (row
  // gl() of M), the return value is solution component gl(). The right-hand
  // side is first sent to position order; both substitutions then broadcast
  // from fixed lanes.
  __device__ static __forceinline__ double solve(const double (&M)[NN], int pos, double rdiag, double b) {
    int i = Gp::gl();
    // with one cell per wave the comparisons are formed at their use, one
    // instruction each, not hoisted out of the stages (which spilled them)
    if constexpr (G == 64) asm volatile("" : "+v"(i));
    b = permute_d(b, 4 * (Gp::base() + (pos >= 0 ? pos : i)));
    // the multipliers are masked rather than the update, which keeps the
    // selects off the chain of dependent broadcasts (a zero multiplier
    // leaves b unchanged for finite z)
    static_for<NN - 1>([&](auto jc) {
      constexpr int j = decltype(jc)::value;
      const double lm = i > j ? M[j] : 0.0;
      b = fma(-lm, Gp::template bcast_c<j>(b), b);
    });
    static_for<NN - 1>([&](auto jc) {
      constexpr int j = NN - 1 - decltype(jc)::value;
      const double um = i < j ? M[j] : 0.0;
      b = fma(-um, Gp::template bcast_c<j>(b * rdiag), b);
    });
    return b * rdiag;
  }

  // -------------------------------------------------------------------------
  // adaptive Rosenbrock integration (scheme SCHEME) over [0, dt] of one cell:
  // begin(), attempt() until it returns false, then St holds the result
  // -------------------------------------------------------------------------
  // GEN: honour the forward-difference Jacobian and the state without the
  // bath gas (run-time options); without it both are compiled out, so that
  // the kernels of the default options carry none of their code.
  struct St {
    double p, y;                // pressure; this lane's state component
    double h, hnext, t, f0;     // next substep, proposal, time, f at y
    int nacc, nrej, att, consec, status;
    int njac, nfev;             // evaluations of J and of f (a difference Jacobian's included)
    bool need;                  // J of the current y not yet evaluated
  };

  // h: first substep (<= 0: dt). Returns whether there is anything to do.
  template <bool GEN>
  __device__ static __forceinline__ bool begin(const MechArgs& A, const OptsDev& o, double p, double y, double h,
                                               double dt, St& c) {
    const int ns = A.ns;
    const bool nb = GEN && o.no_bath != 0;   // bath gas (lane ns) derived, not integrated
    const bool valid = Gp::gl() < (nb ? ns : ns + 1);
    if (nb) y = with_bath(ns, y);
    c = St{p, y, h > 0.0 ? h : dt, 0.0, 0.0, 0.0, 0, 0, 0, 0, 0, 0, 0, true};
    c.hnext = c.h;
    // a non-finite state, or a pressure that is not a positive number
    if (Gp::any((valid && !isfinite(y)) || !isfinite(p) || !(p > 0.0))) c.status = 3;
    return c.status == 0 && c.t < dt;
  }

  // One attempted step. Returns whether the integration goes on.
  template <int SCHEME, bool GEN>
  __device__ static __forceinline__ bool attempt(const MechArgs& A, const MechLds& L, const CellArea& ca, int* jlock,
                                                 const OptsDev& o, double dt, St& c) {
    using TB = Tab<SCHEME>;
    const int ns = A.ns;
    const bool nb = GEN && o.no_bath != 0;
    const int n = nb ? ns : ns + 1;       // integrated components
    const int i = Gp::gl();
    const bool valid = i < n;
    double M[NN];
    int pos;
    double rdiag;
    if (c.att >= o.max_steps) {
      c.status = 1;
      return false;
    }
    if (c.need) {
      ++c.njac;
      c.nfev += (GEN && o.jac_fd) ? 1 + n : 1;
    }
    const double rem = dt - c.t;
    double hc = c.h;
    bool clipped = false;
    if (hc >= rem) {
      hc = rem;
      clipped = true;
    }
    if (hc < kHMin) {
      c.status = 2;
      return false;
    }
    const double g = 1.0 / (TB::gamma * hc);
    if constexpr (kScatter && !GEN) {
      // f of the step start and M = g I - J, formed together; after a
      // rejected attempt (a few per cent) J is formed again
      c.f0 = eval<true, true>(A, L, ca, c.p, c.y, jlock, g, M);
      c.need = false;
    } else {
      // f and J of the step start. A buffer of the wave's own keeps J
      // across rejected attempts; a shared one may have been overwritten, and
      // is not used at all by forward differences
      const bool regs = GEN && can_share_j(NN) && o.jac_fd && jlock;
      if (!regs) j_acquire(jlock);
      if (c.need || jlock) {
        if (GEN && o.jac_fd) {
          c.f0 = rhs<false>(A, L, ca, c.p, c.y);
          fd_jacobian(A, L, ca, c.p, c.y, c.f0, nb, regs, M);
        } else {
          c.f0 = rhs<true>(A, L, ca, c.p, c.y);
          if (nb) reduce_bath(ca, ns);
        }
        c.need = false;
      }
      // (the subtraction for all lanes alike where regs may be, and faster with
      // one cell per wave: 9 species, 1024 cells 5.03 ms, in the branch 5.11; with
      // four 5.41 and 5.33)
      if constexpr (G == 64) {
        if (!regs) {
          if (i < NN) {
#pragma unroll
            for (int j = 0; j < NN; ++j) M[j] = ca.J[i * NN + j];
          } else {
#pragma unroll
            for (int j = 0; j < NN; ++j) M[j] = 0.0;
          }
          j_release(jlock);
        }
#pragma unroll
        for (int j = 0; j < NN; ++j) M[j] = (i == j ? g : 0.0) - M[j];
      } else if (i < NN) {
#pragma unroll
        for (int j = 0; j < NN; ++j) M[j] = (i == j ? g : 0.0) - ca.J[i * NN + j];
      } else {
#pragma unroll
        for (int j = 0; j < NN; ++j) M[j] = 0.0;
      }
    }
    const int info = lu(M, pos, rdiag, ca.P, n, nullptr);
    ++c.att;
    if (info) {
      c.status = 4;
      return false;
    }
    // stages: one right-hand side and one solve call site for all four;
    // every sum runs over j < st in ascending order with the scheme's
    // coefficients, zeros included, as the oracle forms it
    double u1 = 0.0, u2 = 0.0, u3 = 0.0, u4 = 0.0;
    double fs = c.f0;
#pragma nounroll
    for (int st = 0; st < 4; ++st) {
      const int src = tab_fsrc<SCHEME>(st);
      if (src == kFnew) {
        double ys = c.y;
        if (st > 0) ys = ys + tab_a<SCHEME>(st, 0) * u1;
        if (st > 1) ys = ys + tab_a<SCHEME>(st, 1) * u2;
        if (st > 2) ys = ys + tab_a<SCHEME>(st, 2) * u3;
        if (nb) ys = with_bath(ns, ys);
        fs = rhs<false>(A, L, ca, c.p, ys);
        ++c.nfev;
      } else if (src == kFy) {
        fs = c.f0;
      }
      double v = fs;
      if (st > 0) v = v + (tab_c<SCHEME>(st, 0) / hc) * u1;
      if (st > 1) v = v + (tab_c<SCHEME>(st, 1) / hc) * u2;
      if (st > 2) v = v + (tab_c<SCHEME>(st, 2) / hc) * u3;
      if (nb && i == ns) v = 0.0;         // the bath lane takes no step of its own
      const double x = solve(M, pos, rdiag, v);
      if (st == 0) u1 = x;
      else if (st == 1) u2 = x;
      else if (st == 2) u3 = x;
      else u4 = x;
    }
    // new solution and error estimate
    double yn = c.y + TB::m[0] * u1;
    yn = yn + TB::m[1] * u2;
    yn = yn + TB::m[2] * u3;
    yn = yn + TB::m[3] * u4;
    if (nb) yn = with_bath(ns, yn);
    double ev = 0.0 + TB::e[0] * u1;
    ev = ev + TB::e[1] * u2;
    ev = ev + TB::e[2] * u3;
    ev = ev + TB::e[3] * u4;
    const double sc = o.atol + o.rtol * fmax(fabs(c.y), fabs(yn));
    const double q = ev / sc;
    const double acc = Gp::sum(valid ? q * q : 0.0);
    double err = sqrt(acc / n);
    double hnew;
    if (Gp::any(valid && !isfinite(yn)) || !isfinite(err)) {
      err = INFINITY;
      hnew = hc * kFacRej;
    } else {
      double fac = step_factor<SCHEME>(err);
      fac = fmin(kFacMax, fmax(kFacMin, fac));
      hnew = hc * fac;
    }
    if (err <= 1.0) {
      if (c.consec > 0) hnew = fmin(hnew, hc);
      const double Tn = Gp::template bcast_c<0>(yn);
      if (!(Tn >= kTMin && Tn <= kTMax)) {
        c.status = 5;
        return false;
      }
      c.y = yn;
      ++c.nacc;
      c.t = clipped ? dt : c.t + hc;
      c.hnext = clipped ? fmax(hnew, c.h) : hnew;
      c.h = hnew;
      c.consec = 0;
      c.need = true;
    } else {
      ++c.nrej;
      ++c.consec;
      if (c.consec >= 2) hnew = hc * kFacRej;
      c.h = hnew;
    }
    return c.t < dt;
  }
};

// features for the learned cost model: (T-1500)/700, ln(p/1e5),
// mean log10 max(Y, 1e-30) / 10, log10(dt/1e-6)
template <int G>
__device__ __forceinline__ void cell_features(int ns, double y, double p, double dt, float (&ft)[4]) {
  const int i = Grp<G>::gl();
  const double lv = (i >= 1 && i <= ns) ? log10(fmax(y, 1e-30)) : 0.0;
  const double ell = Grp<G>::sum(lv) / ns;
  const double T = Grp<G>::bcast(y, 0);
  ft[0] = static_cast<float>((T - 1500.0) / 700.0);
  ft[1] = static_cast<float>(log(p / 1e5));
  ft[2] = static_cast<float>(ell / 10.0);
  ft[3] = static_cast<float>(log10(dt / 1e-6));
}

// ---------------------------------------------------------------------------
// kernels
// ---------------------------------------------------------------------------
// Read one cell and begin its integration; store its result.
template <int NN, int G, bool GEN>
__device__ __forceinline__ bool load_cell(const IntegrateArgs& a, long long cell, typename Cell<NN, G>::St& c,
                                          float (&ft)[4]) {
  const int ns = a.m.ns;
  const int i = Grp<G>::gl();
  const double* pin = a.phi_in + cell * (ns + 2);
  const double p = pin[1];
  const double y = i == 0 ? pin[0] : (i <= ns ? pin[1 + i] : 0.0);
  if (a.log.cap > 0) cell_features<G>(ns, y, p, a.dt, ft);
  return Cell<NN, G>::template begin<GEN>(a.m, a.o, p, y, a.h_io ? a.h_io[cell] : 0.0, a.dt, c);
}

template <int NN, int G>
__device__ __forceinline__ void store_cell(const IntegrateArgs& a, long long cell,
                                           const typename Cell<NN, G>::St& c, const float (&ft)[4]) {
  const int ns = a.m.ns;
  const int i = Grp<G>::gl();
  double* pout = a.phi_out + cell * (ns + 2);
  if (i == 0) {
    pout[0] = c.y;
    pout[1] = c.p;
  } else if (i <= ns) {
    pout[1 + i] = c.y;
  }
  if (i == 0) {
    if (a.h_io) a.h_io[cell] = c.status != 0 ? c.h : c.hnext;
    if (a.accumulate) {
      if (a.n_acc) a.n_acc[cell] += c.nacc;
      if (a.n_rej) a.n_rej[cell] += c.nrej;
      if (a.status && a.status[cell] == 0) a.status[cell] = static_cast<signed char>(c.status);
      if (a.n_jac) a.n_jac[cell] += c.njac;
      if (a.n_fev) a.n_fev[cell] += c.nfev;
    } else {
      if (a.n_acc) a.n_acc[cell] = c.nacc;
      if (a.n_rej) a.n_rej[cell] = c.nrej;
      if (a.status) a.status[cell] = static_cast<signed char>(c.status);
      if (a.n_jac) a.n_jac[cell] = c.njac;
      if (a.n_fev) a.n_fev[cell] = c.nfev;
    }
    if (a.log.cap > 0) {
      const unsigned long long k = atomicAdd(a.log.head, 1ull) % static_cast<unsigned long long>(a.log.cap);
      a.log.feats[4 * k + 0] = ft[0];
      a.log.feats[4 * k + 1] = ft[1];
      a.log.feats[4 * k + 2] = ft[2];
      a.log.feats[4 * k + 3] = ft[3];
      a.log.target[k] = logf(static_cast<float>(c.nacc + c.nrej > 0 ? c.nacc + c.nrej : 1));
    }
  }
}

template <int NN, int G, int SCHEME, bool GEN>
__device__ __forceinline__ void run_cell(const IntegrateArgs& a, const MechLds& L, const CellArea& ca, int* jlock,
                                         long long cell) {
  typename Cell<NN, G>::St c;
  float ft[4];
  bool go = load_cell<NN, G, GEN>(a, cell, c, ft);
  while (go) go = Cell<NN, G>::template attempt<SCHEME, GEN>(a.m, L, ca, jlock, a.o, a.dt, c);
  store_cell<NN, G>(a, cell, c, ft);
}

// the next run of a.chunk queue positions for this group
template <int G>
__device__ __forceinline__ bool pull(const IntegrateArgs& a, long long& q, long long& end) {
  unsigned long long idx = 0;
  if (Grp<G>::gl() == 0) idx = atomicAdd(a.head, static_cast<unsigned long long>(a.chunk));
  idx = static_cast<unsigned long long>(__shfl(static_cast<long long>(idx), Grp<G>::base(), 64));
  q = static_cast<long long>(idx);
  end = min(q + a.chunk, a.n);
  return idx < static_cast<unsigned long long>(a.n);
}

// Waves per SIMD that the register allocator plans for: two where pairs of
// waves share a Jacobian buffer and two blocks fit a CU's LDS (256 registers
// a lane), one for the other large state sizes.
template <int NN>
constexpr int min_waves_per_eu() { return can_share_j(NN) ? 2 : 1; }
template <int NN>
constexpr int max_waves_per_eu() { return NN >= 32 && !can_share_j(NN) ? 1 : 2; }

// Divide a block's LDS: this wave's (group's) areas, the lock of its Jacobian
// buffer (NULL: the buffer is its own), and the mechanism image staged.
template <int NN, int G>
__device__ __forceinline__ CellArea block_area(unsigned char* smem, const MechArgs& m, int wpb, int cell_doubles,
                                               int share, int*& jlock) {
  constexpr int CPW = 64 / G;
  const int wave = threadIdx.x / 64;
  const int grp = (threadIdx.x % 64) / G;
  double* const work = reinterpret_cast<double*>(smem + m.lds_bytes);
  const bool sh = can_share_j(NN) && share;
  const int nj = sh ? (wpb + 1) / 2 : wpb * CPW;     // Jacobian buffers
  const int jb = sh ? wave / 2 : wave * CPW + grp;
  double* const cells = work + nj * j_doubles_c(NN);
  jlock = nullptr;
  if (sh) {
    jlock = reinterpret_cast<int*>(cells + wpb * cell_doubles) + jb;
    if (threadIdx.x % 128 == 0) *jlock = 0;
  }
  stage_mech(smem, m);        // ends in a barrier
  return cell_area<NN>(work + jb * j_doubles_c(NN), cells + (wave * CPW + grp) * cell_doubles, m.nr);
}

template <int NN, int G, bool PERSIST, int SCHEME, bool GEN>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(min_waves_per_eu<NN>(), max_waves_per_eu<NN>())))
k_integrate(IntegrateArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  constexpr int CPW = 64 / G;
  const int wave = threadIdx.x / 64;
  const int grp = (threadIdx.x % 64) / G;
  int* jlock;
  const CellArea ca = block_area<NN, G>(smem, a.m, a.wpb, a.cell_doubles, a.share_j, jlock);
  const MechLds L = mech_views(smem, a.m);
  if (!PERSIST) {
    const long long cell = (static_cast<long long>(blockIdx.x) * a.wpb + wave) * CPW + grp;
    if (cell < a.n) run_cell<NN, G, SCHEME, GEN>(a, L, ca, jlock, cell);
  } else if constexpr (G == 64) {
    long long q, end;
    while (pull<G>(a, q, end))
      for (; q < end; ++q)
        run_cell<NN, G, SCHEME, GEN>(a, L, ca, jlock, a.perm ? static_cast<long long>(a.perm[q]) : q);
  } else {
    // Several cells per wave: a group that finishes its cell takes the next
    // one while the others go on, so the groups attempt steps together until
    // the queue is empty, not until the longest of each set of cells ends.
    typename Cell<NN, G>::St c;
    float ft[4];
    long long q = 0, end = 0, cell = 0;
    bool busy = false;
    for (;;) {
      if (!busy) {
        if (q >= end && !pull<G>(a, q, end)) break;
        cell = a.perm ? static_cast<long long>(a.perm[q]) : q;
        ++q;
        busy = load_cell<NN, G, GEN>(a, cell, c, ft);
        if (!busy) store_cell<NN, G>(a, cell, c, ft);
      }
      if (busy) {
        busy = Cell<NN, G>::template attempt<SCHEME, GEN>(a.m, L, ca, jlock, a.o, a.dt, c);
        if (!busy) store_cell<NN, G>(a, cell, c, ft);
      }
    }
  }
}

// Right-hand side and Jacobian of every cell. Rows of J leave LDS one per
// store, coalesced (each lane a column); with every lane storing its own row
// a store touched 55 lines for 8 bytes each (8192 54-species cells: 242 us).
template <int NN, int G>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(min_waves_per_eu<NN>()))) k_eval(EvalArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  using C = Cell<NN, G>;
  constexpr int CPW = 64 / G;
  const int wave = threadIdx.x / 64;
  const int grp = (threadIdx.x % 64) / G;
  int* jlock;
  const CellArea ca = block_area<NN, G>(smem, a.m, a.wpb, a.cell_doubles, a.share_j, jlock);
  const MechLds L = mech_views(smem, a.m);
  const int ns = a.m.ns, n = ns + 1;
  const int i = Grp<G>::gl();
  const long long stride = static_cast<long long>(gridDim.x) * a.wpb * CPW;
  for (long long cell = (static_cast<long long>(blockIdx.x) * a.wpb + wave) * CPW + grp; cell < a.n; cell += stride) {
    const double* pin = a.phi + cell * (ns + 2);
    const double p = pin[1];
    const double y = i == 0 ? pin[0] : (i <= ns ? pin[1 + i] : 0.0);
    const double f = a.J ? C::template rhs<true>(a.m, L, ca, p, y, jlock) : C::template rhs<false>(a.m, L, ca, p, y);
    if (i < n) {
      a.f[cell * n + i] = f;
      if (a.J) {
        double* out = a.J + cell * n * n + i;
#pragma unroll 8
        for (int r = 0; r < n; ++r) out[r * n] = ca.J[r * NN + i];
      }
    }
    if (a.J) j_release(jlock);
    wsync();
  }
}

// Batched LU. The matrices pass through LDS in runs of whole rows (of all the
// wave's matrices when it has several), so that global accesses are contiguous
// over the lanes; each lane then has its row. With every lane loading its own
// row, 16384 55 x 55 matrices took 826 us, the copy of A they are made in
// included.
constexpr int kLuRows = 28;          // rows per run (one matrix per wave)
__host__ __device__ constexpr int lu_stage_doubles(int nn, int g) {
  const int stage = (g == 64 ? (nn < kLuRows ? nn : kLuRows) * nn : 64 / g * nn * nn);
  const int rows = g == 64 ? lu_rows_doubles(nn) : 64 / g * lu_row_doubles(nn);
  return ((stage > rows ? stage : rows) + 1) & ~1;
}

template <int NN, int G>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(NN > 55 ? 2 : 3))) k_lu(LuArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  using C = Cell<NN, G>;
  constexpr int CPW = 64 / G;
  const int wave = threadIdx.x / 64;
  const int lane = threadIdx.x % 64, grp = lane / G;
  double* const S = reinterpret_cast<double*>(smem) + wave * lu_stage_doubles(NN, G);
  const long long m0 = (static_cast<long long>(blockIdx.x) * a.wpb + wave) * CPW;
  if (m0 >= a.batch) return;
  const long long m = m0 + grp;
  const bool on = m < a.batch;                 // the last wave's groups may be without a matrix
  const int n = a.n;
  const int i = Grp<G>::gl();
  double M[NN];
#pragma unroll
  for (int j = 0; j < NN; ++j) M[j] = i == j ? 1.0 : 0.0;
  // runs of rows: r0 .. r0 + nr - 1 of one matrix, or all rows of the wave's
  const int mats = static_cast<int>(min(static_cast<long long>(CPW), a.batch - m0));
  const int step = G == 64 ? kLuRows : NN;
  double* const A0 = a.A + m0 * n * n;
  for (int r0 = 0; r0 < n; r0 += step) {
    const int nr = min(step, n - r0);
    const int cnt = G == 64 ? nr * n : mats * n * n;
    wsync();
#pragma unroll 8
    for (int e = lane; e < cnt; e += 64) S[e] = A0[r0 * n + e];
    wsync();
    const int r = i - r0;
    if (on && r >= 0 && r < nr) {
      const double* row = S + (G == 64 ? r * n : (grp * n + i) * n);
      if (n == NN) {
#pragma unroll
        for (int j = 0; j < NN; ++j) M[j] = row[j];
      } else {
        // entries past the row's end are read (within S) and not used
#pragma unroll
        for (int j = 0; j < NN; ++j) {
          const double v = row[j];
          M[j] = j < n ? v : 0.0;
        }
      }
    }
  }
  wsync();
  int piv = 0;
  int pos;
  double rdiag;
  const int info = C::lu(M, pos, rdiag, S + (G == 64 ? 0 : grp * lu_row_doubles(NN)), n, &piv);
  for (int r0 = 0; r0 < n; r0 += step) {
    const int nr = min(step, n - r0);
    const int cnt = G == 64 ? nr * n : mats * n * n;
    const int r = i - r0;
    wsync();
    if (on && r >= 0 && r < nr) {
      double* row = S + (G == 64 ? r * n : (grp * n + i) * n);
#pragma unroll
      for (int j = 0; j < NN; ++j)
        if (j < n) row[j] = M[j];
    }
    wsync();
#pragma unroll 8
    for (int e = lane; e < cnt; e += 64) A0[r0 * n + e] = S[e];
  }
  if (!on) return;
  if (i < n) a.piv[m * n + i] = piv;
  if (i == 0) a.info[m] = info;
  if (a.b) {
    const double b = i < n ? a.b[m * n + i] : 0.0;
    const double x = C::solve(M, pos, rdiag, b);
    if (i < n) a.b[m * n + i] = x;
  }
}

}  // namespace

// ---------------------------------------------------------------------------
// dispatch
// ---------------------------------------------------------------------------
// The variants with one cell per wave are a compilation unit of their own
// (integrator_wave.hip), compiled without the machine-level hoisting of loop
// invariants: in their step loop it moves more 64-bit constants (of log and exp,
// mostly) into registers than there are, and each is reloaded from scratch at its
// use, one wait after the other (54 species: 89 spilled registers with it, 24
// without; 131 cells 16.0 ms with, 15.0 without; 32768 cells 79.6 and 76.7).
// Variants with several cells per wave have registers to spare and lose by it
// (9 species, 1024 cells, four a wave: 5.2 ms with, 5.4 without).
#define CHEM_VARIANTS(X) \
  X(10, 16)              \
  X(10, 64)              \
  X(16, 16)              \
  X(32, 32)              \
  X(55, 64)              \
  X(64, 64)
#define CHEM_GROUP_VARIANTS(X) \
  X(10, 16)                    \
  X(16, 16)                    \
  X(32, 32)
#define CHEM_WAVE_VARIANTS(X) \
  X(10, 64)                   \
  X(55, 64)                   \
  X(64, 64)
#ifdef CHEM_WAVE_UNIT
#define CHEM_UNIT_VARIANTS CHEM_WAVE_VARIANTS
#define CHEM_UNIT(name) wave_##name
#else
#define CHEM_UNIT_VARIANTS CHEM_GROUP_VARIANTS
#define CHEM_UNIT(name) group_##name
#endif

template <int NN, int G, bool P>
static void* integrate_fn(int scheme, bool gen) {
  if (gen)
    return scheme == dev::kRos4 ? reinterpret_cast<void*>(&k_integrate<NN, G, P, dev::kRos4, true>)
                                : reinterpret_cast<void*>(&k_integrate<NN, G, P, dev::kRodas3, true>);
  return scheme == dev::kRos4 ? reinterpret_cast<void*>(&k_integrate<NN, G, P, dev::kRos4, false>)
                              : reinterpret_cast<void*>(&k_integrate<NN, G, P, dev::kRodas3, false>);
}

// this unit's kernels; null for a variant of the other one
void* CHEM_UNIT(integrate_kernel)(const Variant& v, bool persistent, int scheme, bool gen) {
#define V(a, b)                                                                                        \
  if (v.nn == a && v.g == b)                                                                           \
    return persistent ? integrate_fn<a, b, true>(scheme, gen) : integrate_fn<a, b, false>(scheme, gen);
  CHEM_UNIT_VARIANTS(V)
#undef V
  return nullptr;
}

void* CHEM_UNIT(eval_kernel)(const Variant& v) {
#define V(a, b) \
  if (v.nn == a && v.g == b) return reinterpret_cast<void*>(&k_eval<a, b>);
  CHEM_UNIT_VARIANTS(V)
#undef V
  return nullptr;
}

void* CHEM_UNIT(lu_kernel)(const Variant& v) {
#define V(a, b) \
  if (v.nn == a && v.g == b) return reinterpret_cast<void*>(&k_lu<a, b>);
  CHEM_UNIT_VARIANTS(V)
#undef V
  return nullptr;
}

#ifndef CHEM_WAVE_UNIT
void* wave_integrate_kernel(const Variant& v, bool persistent, int scheme, bool gen);
void* wave_eval_kernel(const Variant& v);
void* wave_lu_kernel(const Variant& v);

int variants_for(int n, Variant* out, int max_out) {
  // exact sizes first, then the smallest padded size
  static const Variant all[] = {
#define V(a, b) {a, b},
      CHEM_VARIANTS(V)
#undef V
  };
  int cnt = 0, best_nn = 1 << 30;
  for (const Variant& v : all)
    if (v.nn >= n && v.nn < best_nn) best_nn = v.nn;
  for (const Variant& v : all)
    if (v.nn == best_nn && cnt < max_out) out[cnt++] = v;
  return cnt;
}

int cell_doubles(int nn, int nr, int ns) { return cell_doubles_c(nn, nr); }

size_t block_lds(const Variant& v, int nr, int ns, int mech_bytes, int wpb, bool share_j) {
  const int cpw = 64 / v.g;
  const size_t nj = share_j ? (wpb + 1) / 2 : wpb * cpw;
  return mech_bytes + sizeof(double) * (nj * j_doubles_c(v.nn) + static_cast<size_t>(wpb) * cpw * cell_doubles_c(v.nn, nr)) +
         (share_j ? 16 : 0);
}

bool share_j(const Variant& v, int nr, int ns, int mech_bytes, int wpb, size_t lds_per_cu) {
  // pays only where it brings a second block to the CU; one wave has none to
  // share with
  return v.g == 64 && can_share_j(v.nn) && wpb >= 2 && 2 * block_lds(v, nr, ns, mech_bytes, wpb, true) <= lds_per_cu;
}

static void* find_integrate(const Variant& v, bool persistent, int scheme, bool gen) {
  if (scheme != dev::kRodas3 && scheme != dev::kRos4) return nullptr;
  return v.g == 64 ? wave_integrate_kernel(v, persistent, scheme, gen) : group_integrate_kernel(v, persistent, scheme, gen);
}

hipError_t launch_integrate(const Variant& v, bool persistent, int grid, const IntegrateArgs& a,
                            size_t lds_bytes, hipStream_t st) {
  void* fn = find_integrate(v, persistent, a.o.scheme, a.o.jac_fd || a.o.no_bath);
  if (!fn) return hipErrorInvalidValue;
  hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds_bytes));
  if (e != hipSuccess) return e;
  dim3 block(64 * a.wpb);
  IntegrateArgs copy = a;
  void* args[] = {&copy};
  return hipLaunchKernel(fn, dim3(grid), block, args, lds_bytes, st);
}

int integrate_blocks_per_cu(const Variant& v, bool persistent, int wpb, size_t lds_bytes) {
  void* fn = find_integrate(v, persistent, dev::kRodas3, false);
  if (!fn) return 0;
  hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds_bytes));
  int nb = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, fn, 64 * wpb, lds_bytes) != hipSuccess) return 0;
  return nb;
}

hipError_t launch_eval(const Variant& v, int grid, const EvalArgs& a, size_t lds_bytes, hipStream_t st) {
  void* fn = v.g == 64 ? wave_eval_kernel(v) : group_eval_kernel(v);
  if (!fn) return hipErrorInvalidValue;
  hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds_bytes));
  if (e != hipSuccess) return e;
  EvalArgs copy = a;
  void* args[] = {&copy};
  return hipLaunchKernel(fn, dim3(grid), dim3(64 * a.wpb), args, lds_bytes, st);
}

hipError_t launch_lu(const Variant& v, int grid, const LuArgs& a, hipStream_t st) {
  void* fn = v.g == 64 ? wave_lu_kernel(v) : group_lu_kernel(v);
  if (!fn) return hipErrorInvalidValue;
  LuArgs copy = a;
  void* args[] = {&copy};
  const size_t lds = sizeof(double) * lu_stage_doubles(v.nn, v.g) * a.wpb;
  hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));
  if (e != hipSuccess) return e;
  return hipLaunchKernel(fn, dim3(grid), dim3(64 * a.wpb), args, lds, st);
}

static __global__ void k_fill_u64(unsigned long long* p, unsigned long long v) { *p = v; }

static __global__ void k_copy_f64(double* dst, const double* src, long long n) {
  for (long long i = blockIdx.x * static_cast<long long>(blockDim.x) + threadIdx.x; i < n;
       i += static_cast<long long>(gridDim.x) * blockDim.x)
    dst[i] = src[i];
}

hipError_t launch_fill_u64(unsigned long long* p, unsigned long long v, hipStream_t st) {
  hipLaunchKernelGGL(k_fill_u64, dim3(1), dim3(1), 0, st, p, v);
  return hipGetLastError();
}

hipError_t launch_copy_f64(double* dst, const double* src, long long n, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  long long blocks = (n + 255) / 256;
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(k_copy_f64, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, st, dst, src, n);
  return hipGetLastError();
}

#endif  // CHEM_WAVE_UNIT

}  // namespace chemk
