// Host-side mechanism: parser, validation, and the packed images the kernels
// read (an LDS image staged by every block, plus global thermo tables).
#pragma once
#include <cstdint>
#include <string>
#include <vector>

namespace chem {

constexpr int kMaxSide = 3;        // distinct species per reaction side on the device
constexpr int kMaxSpecies = 255;   // species index fits in a byte of the reaction word
constexpr int kMaxReactions = 4095;

struct Rxn {
  int type = 0;   // 0 elementary, 1 third body, 2 Troe falloff
  int rev = 1;
  std::vector<std::pair<int, int>> reac, prod;   // (species, order), distinct species
  double A = 0, b = 0, Ea = 0;
  std::vector<std::pair<int, double>> eff;        // (species, alpha)
  double A0 = 0, b0 = 0, Ea0 = 0, ta = 0, T3 = 1, T1 = 1, T2 = 0;
  bool has_T2 = false;
};

struct MechHost {
  int ns = 0, nr = 0, ne = 0;
  std::vector<int> elem;                 // [ns][ne] atoms of each element per molecule
  std::vector<double> W;                 // kg/mol
  std::vector<double> tmid;              // NASA range boundary per species
  std::vector<double> lo, hi;            // [ns][7]
  std::vector<Rxn> rx;
};

// Parse the text format; on failure returns false with a message.
bool parse_mechanism(const std::string& path, MechHost& m, std::string& err);

// Algorithmic work per right-hand side and per Jacobian (beyond its RHS).
struct Work { double f_rhs, f_jac, t_rhs, t_jac; };
Work count_work(const MechHost& m);

// Packed image. The LDS blob is a byte array whose sections start at the
// offsets below (all 16-byte aligned); the kernel copies it into LDS verbatim.
struct Packed {
  std::vector<uint8_t> blob;
  int off_lnA, off_b, off_EaR, off_rint, off_troe, off_eff_sp, off_eff_am1, off_sp_off, off_sp_ent,
      off_rW;
  int lds_bytes;    // leading part of blob staged in LDS
  int ntroe, neff, nent;
  // Reaction records of the per-wave kernel (up to 64 state components, 63
  // species): seven arrays of rec_n 16-byte entries (nr rounded up to 64, absent
  // reactions without species):
  //   (ln A, b), (Ea/R, sum nu), (order of reactant 0, of product 0), (of 1,
  //   of 1), (of 2, of 2) as doubles; then two of 32-bit words
  //   w0 = slot offsets f0 | f1 << 16, r0 | r1 << 16, second factors ef | er << 16, flags
  //   w1 = slot offsets f2 | r2 << 16, third factors ef | er << 16, efficiency and Troe word, 0
  // An offset is 8 times a species index; absent slots hold 8 ns, where the
  // kernel keeps a concentration of 1 and zero g and h. A side's mass-action
  // product is C[slot 0] * C[second] * C[third]. Flags: bits 0..5 slot present
  // (f0 f1 f2 r0 r1 r2), 6 a side with three factors, 8..9 type, 10 reversible.
  // The second species of a side 2A + B is in slot 2; the sums take it second.
  // Empty if a side does not fit (a total order above 3, a species of order 2
  // after another, order 3): such mechanisms use the general records.
  std::vector<uint8_t> rec;
  int rec_n = 0;
  std::vector<double> nasa;   // [ns][16]: lo a1..a7, tmid, hi a1..a7, 0
  std::vector<double> W, rW;  // [ns]
};
Packed pack(const MechHost& m);

}  // namespace chem
