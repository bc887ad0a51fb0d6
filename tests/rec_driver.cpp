// Decodes the per-wave kernel's reaction records (mech.hpp, Packed::rec) of
// every mechanism file given and compares them with the parsed reactions.
// Prints "records" or "general" (no records) per file. TEST INFRASTRUCTURE ONLY.
#include <algorithm>
#include <cstdio>
#include <cstring>
#include <map>
#include <string>

#include "mech.hpp"

static int bad(const char* what, int r) {
  std::printf("mismatch: %s of record %d\n", what, r);
  return 1;
}

int main(int argc, char** argv) {
  for (int f = 1; f < argc; ++f) {
    chem::MechHost m;
    std::string err;
    if (!chem::parse_mechanism(argv[f], m, err)) {
      std::printf("error %s\n", err.c_str());
      return 1;
    }
    const chem::Packed P = chem::pack(m);
    if (P.rec.empty()) {
      std::printf("general\n");
      continue;
    }
    const int N = P.rec_n;
    if (N % 64 || N < m.nr || N >= m.nr + 64 || P.rec.size() != static_cast<size_t>(N) * 112) return bad("size", -1);
    const double* d = reinterpret_cast<const double*>(P.rec.data());
    const uint32_t* w = reinterpret_cast<const uint32_t*>(P.rec.data() + static_cast<size_t>(N) * 80);
    const uint32_t none = 8u * m.ns;
    std::vector<int> order(m.nr);
    for (int r = 0; r < m.nr; ++r) order[r] = r;
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return m.rx[a].type < m.rx[b].type; });
    for (int r = 0; r < N; ++r) {
      const uint32_t* a = w + 4 * r;
      const uint32_t* b = w + 4 * (N + r);
      const uint32_t slot[6] = {a[0] & 0xffff, a[0] >> 16, b[0] & 0xffff, a[1] & 0xffff, a[1] >> 16, b[0] >> 16};
      const uint32_t fac[2][2] = {{a[2] & 0xffff, b[1] & 0xffff}, {a[2] >> 16, b[1] >> 16}};
      for (uint32_t s : slot)
        if (s % 8 || s > none) return bad("offset", r);
      if (r >= m.nr) {
        if (a[3]) return bad("padding flags", r);
        for (uint32_t s : slot)
          if (s != none) return bad("padding slot", r);
        continue;
      }
      const chem::Rxn& x = m.rx[order[r]];
      if (((a[3] >> 8) & 3) != static_cast<uint32_t>(x.type) || ((a[3] >> 10) & 1) != (x.rev ? 1u : 0u))
        return bad("type or direction", r);
      uint32_t w3;
      std::memcpy(&w3, P.blob.data() + P.off_rint + 16 * r + 12, 4);
      if (b[2] != w3) return bad("efficiency word", r);
      double dnu = 0;
      bool three = false;
      for (int sd = 0; sd < 2; ++sd) {
        const auto& v = sd ? x.prod : x.reac;
        std::map<uint32_t, int> want, got, factors;
        for (auto& p : v) {
          want[8u * p.first] = p.second;
          dnu += (sd ? 1 : -1) * p.second;
        }
        // distinct species in their order, each with its order
        size_t at = 0;
        for (int k = 0; k < 3; ++k) {
          const bool on = (a[3] >> (3 * sd + k)) & 1;
          const double nu = d[2 * ((2 + k) * N + r) + sd];
          if (on != (slot[3 * sd + k] != none) || (!on && nu != 0)) return bad("slot", r);
          if (!on) continue;
          if (at >= v.size() || slot[3 * sd + k] != 8u * v[at].first || nu != v[at].second) return bad("order", r);
          ++at;
        }
        if (at != v.size()) return bad("species count", r);
        // factors of the product: slot 0, second, third
        for (uint32_t s : {slot[3 * sd], fac[sd][0], fac[sd][1]})
          if (s != none) ++factors[s];
        if (factors != want) return bad("factors", r);
        if (fac[sd][1] != none) three = true;
        if (slot[3 * sd + 2] != fac[sd][1]) return bad("third factor", r);
      }
      if (d[2 * (N + r) + 1] != dnu) return bad("sum nu", r);
      if (((a[3] >> 6) & 1) != (three ? 1u : 0u)) return bad("third flag", r);
      if (d[2 * r + 1] != x.b) return bad("b", r);
    }
    std::printf("records\n");
  }
  return 0;
}
