// Writes fixed_masks_o4.hpp: the compile-time descriptor masks and label
// cycles of the 39 fourth-order diagrams (the generator's, in plain loop
// order), for the fourth-order sample kernels.  Built against the library and run
// from the repository root:
//
//   hipcc -std=c++17 -I include -I paper_2603_24532_amd/csrc \
//     paper_2603_24532_amd/csrc/gen_fixed_masks.cpp \
//     -L paper_2603_24532_amd -lmbpt_vegas -Wl,-rpath,$PWD/paper_2603_24532_amd \
//     -o /tmp/gen_fixed_masks && /tmp/gen_fixed_masks > paper_2603_24532_amd/csrc/fixed_masks_o4.hpp
//
// The library checks these tables against its generator whenever a task set
// or server is created, so a stale header is refused, not used.
#include <cstdio>
#include <cstdlib>

#include "device_types.hpp"
#include "diagrams.hpp"
#include "runtime.hpp"

using namespace mbpt;

int main() {
  constexpr int O = 4, NL = 2 * O, L = O + 1, NC = O - 1;
  const int n = num_diagrams(O);
  std::printf("// Generated by gen_fixed_masks.cpp: compile-time descriptor masks and label\n");
  std::printf("// cycles of the %d fourth-order diagrams (variant V = diagram id).\n", n);
  std::printf("#pragma once\n\n");
  std::printf("namespace mbpt {\n");
  for (int id = 0; id < n; ++id) {
    DiagDev d{};
    fill_diag_dev(*get_diagram(O, id), d, false);
    std::printf("template <>\nstruct FixedMasks<4, %d> {\n", id);
    std::printf("  static constexpr bool kFixed = true;\n");
    std::printf("  static constexpr uint32_t line_mask = 0x%Xu, part_mask = 0x%Xu;\n", d.line_mask,
                d.part_mask);
    std::printf("  static constexpr uint32_t lmask[%d] = {", NL);
    for (int l = 0; l < NL; ++l) std::printf("%s0x%Xu", l ? ", " : "", d.lmask[l]);
    std::printf("};\n  static constexpr uint32_t pmask_v[%d] = {", O);
    for (int v = 0; v < O; ++v) std::printf("%s0x%Xu", v ? ", " : "", d.pmask_v[v]);
    std::printf("};\n  static constexpr uint32_t qmask_v[%d] = {", O);
    for (int v = 0; v < O; ++v) std::printf("%s0x%Xu", v ? ", " : "", d.qmask_v[v]);
    std::printf("};\n  static constexpr uint32_t cut_hole[%d] = {", NC);
    for (int c = 0; c < NC; ++c) std::printf("%s0x%Xu", c ? ", " : "", d.cut_hole[c]);
    std::printf("};\n  static constexpr uint32_t cut_part[%d] = {", NC);
    for (int c = 0; c < NC; ++c) std::printf("%s0x%Xu", c ? ", " : "", d.cut_part[c]);
    std::printf("};\n  static constexpr int loop_part[%d] = {", L);
    for (int j = 0; j < L; ++j) std::printf("%s%d", j ? ", " : "", d.loop_part[j]);
    // per vertex-term choice E: its cycle set | its cycle count << 24
    const CycleTables ct = cycle_tables(*get_diagram(O, id), false);
    if (ct.masks.size() > 24 || ct.of_e.size() != (1u << O)) {
      std::fprintf(stderr, "diagram %d: %zu cycles do not fit the 32-bit words\n", id,
                   ct.masks.size());
      return EXIT_FAILURE;
    }
    std::printf("};\n  static constexpr uint32_t cyc_e32[%d] = {", 1 << O);
    for (int E = 0; E < (1 << O); ++E)
      std::printf("%s0x%Xu", E ? ", " : "",
                  static_cast<uint32_t>(ct.of_e[E] | static_cast<uint64_t>(ct.n_of_e[E]) << 24));
    std::printf("};\n};\n");
  }
  std::printf("}  // namespace mbpt\n");
  return 0;
}
