// Device code of the sample kernels for gfx950 (CDNA4): VEGAS Monte Carlo of
// MBPT energy diagrams.  Templates only (plus two small constant tables, one
// copy per code object); kernels_inst.hip instantiates them per order and
// matter, kernels.hip holds the iteration-end, HF and init kernels.
//
// One thread evaluates one sample at a time: Philox4x32-10 words -> VEGAS
// bins and fractions (grid in LDS) -> spherical loop momenta -> line momenta
// from the compiled descriptor -> Pauli factors (n_k for holes, 1 - n_k for
// particles) -> energy denominators (eq:Dijkabc, free spectrum) ->
// antisymmetrised matrix elements per vertex -> explicit spin(-isospin) label
// sum -> weight.  Sums of (w - c) and (w - c)^2 are kept per thread as plain
// sums (at most spt terms), merged across the wavefront, the block and the
// work items with compensated pair merges in a fixed order; refinement
// histograms of w^2 are privatised in LDS and merged with fp64 atomics.  The integrand is
// elementwise with no contraction, so it runs on the vector ALUs (no MFMA).
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

#include "device_types.hpp"
#include "turn_table.hpp"
#include "kernels.hpp"

namespace mbpt {

// ---------------------------------------------------------------------------
// Philox4x32-10 (Salmon et al., SC'11)

__device__ __forceinline__ void philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                              uint32_t k0, uint32_t k1, uint32_t *out) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    // 32 x 32 -> 64-bit products (one v_mad_u64_u32 each)
    const uint64_t p0 = static_cast<uint64_t>(0xD2511F53u) * c0;
    const uint64_t p1 = static_cast<uint64_t>(0xCD9E8D57u) * c2;
    // three-input XOR in one v_bitop3_b32 (truth table 0x96)
    const uint32_t n0 = __builtin_amdgcn_bitop3_b32(static_cast<uint32_t>(p1 >> 32), c1, k0, 0x96);
    const uint32_t n2 = __builtin_amdgcn_bitop3_b32(static_cast<uint32_t>(p0 >> 32), c3, k1, 0x96);
    c0 = n0;
    c1 = static_cast<uint32_t>(p1);
    c2 = n2;
    c3 = static_cast<uint32_t>(p0);
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
  out[0] = c0;
  out[1] = c1;
  out[2] = c2;
  out[3] = c3;
}

// sin and cos of 2 pi k / MBPT_TURN_STEPS (copied into LDS by every sample
// kernel).
struct alignas(16) SinCos {
  double s, c;
};
constexpr int kTurnEntries = MBPT_TURN_STEPS + 1;
static __constant__ SinCos kTurnDev[kTurnEntries] = {MBPT_TURN_TABLE_INIT};
// 2^(j / 64), j = 0..63 (the table-driven exponential, copied into LDS beside
// the turn table)
constexpr int kExp2Entries = 64;
static __constant__ double kExp2Dev[kExp2Entries] = {MBPT_EXP2_TABLE_INIT};

__device__ __forceinline__ void load_turn_table(SinCos *dst, double *ex) {
  for (int i = threadIdx.x; i < kTurnEntries; i += blockDim.x) dst[i] = kTurnDev[i];
  for (int i = threadIdx.x; i < kExp2Entries; i += blockDim.x) ex[i] = kExp2Dev[i];
}

// What the integrand reads from LDS: the turn table, the 2^(j/64) table, the
// HF spline entries of the task (ntab isospin tables of kHfEntries x 4
// doubles, absent with the free spectrum) and the grid pairs of grid_pair.
// Block layout: turn table, 2^(j/64) table, HF tables, grid pairs, then
// the kernel's own scratch.
struct SampleLds {
  const SinCos *turn;
  const double *ex;
  const double *hf;
  const double2 *g;
  const void *cyc;  // label table(s) of the item's diagram(s) (see LabelForm)
};

// Fourth-order nuclear-matter single diagrams with the free spectrum, the
// quartic regulator and the polynomial label sums: the sample kernels branch
// per work item to code with the diagram's masks as compile-time constants
// (all 39 diagrams in one kernel, see with_variant).
// One launch covers every diagram, so its last, partly filled round of blocks
// is paid once per iteration: 39 launches, one per diagram, left the device
// idle at the end of each.  585 tasks, MI355X: 2^21 samples fp32 34.3 -> 24.8
// ms per iteration, 500 009 samples fp64 21.3 -> 7.1 ms; one task per launch
// (2^18 samples, fp32) 52 -> 45 us per iteration against the
// descriptor-driven code.
constexpr int kFixed4Diagrams = 39;
template <int ORDER, int Q, int P, bool X, int HE>
constexpr bool fixed4() {
  return ORDER == 4 && Q == 4 && (P == 0 || P == 1) && !X && HE == 2;
}

// The descriptor-driven single-diagram sample kernels of orders 4 and 5 read
// the loop coefficients of their momentum sums decoded in the descriptor
// (DiagDev::coef_d / coef_f) through the scalar cache, instead of decoding
// them from the bit masks per sum and sample on the scalar unit (so do the
// group kernels, per member).  Measured on MI355X against the masks: 9-13%
// faster at fourth order (per task, with components, neutron matter), 6-10%
// at fifth order, and 5-10% in the persistent kernels; against a table of
// the same values in LDS, 2-9% faster.
template <int ORDER, int P>
constexpr bool desc_coef() {
  return ORDER >= 4 && !(P == 3 || P == 4 || P == 6);  // not the group modes
}

// Label-cycle bit vectors: bit k of CycWord<ORDER> stands for cycle k of a
// diagram (at most 17 at fourth order, 33 at fifth).
template <int ORDER>
using CycWord = std::conditional_t<(ORDER >= 5), uint64_t, uint32_t>;

// Fifth-order diagrams with at most 24 label cycles (696 of the 840) run the
// variant kNarrowCycles of the cycle-form kernels, with 32-bit cycle words
// (the packing of DiagDev::cyc_e32): half the scalar registers for the
// per-E words and single-word bit operations per term.
constexpr int kNarrowCycles = -4;
constexpr int kNarrowCycleMax = 24;
template <int ORDER, int V>
using CycWordV = std::conditional_t<(ORDER >= 5 && V != kNarrowCycles), uint64_t, uint32_t>;

// The nuclear-matter label sum runs in the cycle form (see label_sum) for
// single diagrams with the free spectrum and the factorised label sum.
template <int ORDER, int Q, bool G, bool X, bool HF>
constexpr bool cycle_form() {
  return Q == 4 && ORDER >= 2 && !G && !X && !HF;
}
// Diagram groups of orders 3 and 4 run the cycle form per member, with one
// cycle table per member in LDS (kGroupCycleTables of them).
template <int ORDER, int Q, bool X, bool HF>
constexpr bool group_cycle_form() {
  return Q == 4 && (ORDER == 3 || ORDER == 4) && !X && !HF;
}

// How a kernel evaluates the label sum: kConfigs, one polynomial per isospin
// configuration (or the assignment list); kCycles, the cycle form from the
// label cycles left open (label_sum_cycles); kCounts, the cycle form with all
// the counts read from a table in LDS (label_sum_counts), which holds 2^{2n}
// entries of 2^n bytes: 4 KB at fourth order, but 32 KB at fifth and one per
// member for groups, so those take the cycles.
enum LabelForm { kConfigs, kCycles, kCounts };
template <int ORDER, int Q, bool G, bool X, bool HF>
constexpr LabelForm label_form() {
  if (G) return group_cycle_form<ORDER, Q, X, HF>() ? kCycles : kConfigs;
  if (!cycle_form<ORDER, Q, G, X, HF>()) return kConfigs;
  return ORDER <= 4 ? kCounts : kCycles;
}

// Entry of the count table: the counts of the 2^ORDER vertex-term choices, a
// byte each, as fp8 e5m2 (powers of two up to 2^15 and 0 are exact, and one
// instruction turns a pair into floats).
template <int ORDER>
struct alignas(1 << ORDER) LabelCounts {
  uint32_t w[(1 << ORDER) / 4];
};
template <int ORDER>
__host__ __device__ constexpr size_t count_table_bytes() {
  return sizeof(LabelCounts<(ORDER >= 2 && ORDER <= 4) ? ORDER : 2>) << (2 * ORDER);
}

// Bytes of the label-cycle table: one CycWord per set of lines.
template <int ORDER>
__host__ __device__ constexpr size_t cycle_table_bytes() {
  return (size_t{1} << (2 * ORDER)) * sizeof(CycWord<ORDER>);
}

// tab[s] = the cycles of diagram D that contain no line of the line set s
// (bit k set if (s & cycle k) = 0); built by the whole block.
template <typename W>
__device__ __forceinline__ void fill_cycle_table(const DiagDev *__restrict__ D, int nsets,
                                                 W *tab) {
  const int K = D->ncyc;
  for (int s = threadIdx.x; s < nsets; s += blockDim.x) {
    W w = 0;
    for (int k = 0; k < K; ++k)
      w |= (static_cast<uint32_t>(s) & D->cyc_mask[k]) == 0u ? (W(1) << k) : W(0);
    tab[s] = w;
  }
}
// In the words of the variant with_variant picks for D: 32 bits for a
// fifth-order diagram of at most kNarrowCycleMax cycles.
template <int ORDER>
__device__ __forceinline__ void build_cycle_table(const DiagDev *__restrict__ D, void *tab) {
  constexpr int NS = 1 << (2 * ORDER);
  if (ORDER >= 5 && D->ncyc <= kNarrowCycleMax)
    fill_cycle_table(D, NS, static_cast<uint32_t *>(tab));
  else
    fill_cycle_table(D, NS, static_cast<CycWord<ORDER> *>(tab));
}

// Count table of diagram D (kCounts), built by the whole block.  Entry s: every
// line of the set s is open to one isospin only (a hole line to the one with
// the larger Fermi momentum, a particle line to the other), every other line
// to both; choice E counts 2 spin states times the isospins open to all of the
// cycle's lines, per label cycle of E.  (The count is the same with neutrons
// and protons exchanged, so the table serves either asymmetry.)
template <int ORDER>
__device__ __forceinline__ void build_count_table(const DiagDev *__restrict__ D,
                                                  LabelCounts<ORDER> *tab) {
  constexpr int NS = 1 << (2 * ORDER), NW = (1 << ORDER) / 4;
  const int K = D->ncyc;
  const uint32_t part = D->part_mask;
  for (int s = threadIdx.x; s < NS; s += blockDim.x) {
    const uint32_t ps = static_cast<uint32_t>(s) & part, hs = static_cast<uint32_t>(s) & ~part;
    uint32_t cA = 0, cB = 0;  // cycles open to the isospin of larger / smaller kF
    for (int k = 0; k < K; ++k) {
      cA |= (ps & D->cyc_mask[k]) == 0u ? (1u << k) : 0u;
      cB |= (hs & D->cyc_mask[k]) == 0u ? (1u << k) : 0u;
    }
    const uint32_t ab = cA | cB, both = cA & cB;
    LabelCounts<ORDER> r;
#pragma unroll
    for (int i = 0; i < NW; ++i) {
      uint32_t w = 0;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const uint32_t c = D->cyc_e32[4 * i + j], m = c & 0xFFFFFFu, n = c >> 24;
        const uint32_t e5m2 = (15u + n + static_cast<uint32_t>(__popc(both & m))) << 2;
        w |= ((ab & m) == m ? e5m2 : 0u) << (8 * j);
      }
      r.w[i] = w;
    }
    tab[s] = r;
  }
}

// Bytes of the fixed tables at the start of a sample kernel's LDS.
__host__ __device__ constexpr size_t fixed_lds_bytes() {
  return kTurnEntries * sizeof(SinCos) + kExp2Entries * sizeof(double);
}

__host__ __device__ constexpr size_t hf_lds_doubles(int ntab) {
  return static_cast<size_t>(ntab) * kHfEntries * 4;
}

// HF splines in LDS: the (a, b) coefficients of every entry of the ntab tables,
// then the (c, d): a gather of 16-byte pairs spreads over all the banks, where
// pairs of a 32-byte entry fall on half of them.
template <int NTAB>
__device__ __forceinline__ void load_hf(double *hf, const double *__restrict__ src) {
  constexpr int n = NTAB * kHfEntries;
  double2 *ab = reinterpret_cast<double2 *>(hf), *cd = ab + n;
  const double2 *e = reinterpret_cast<const double2 *>(src);
  for (int i = threadIdx.x; i < n; i += blockDim.x) {
    ab[i] = e[2 * i];
    cd[i] = e[2 * i + 1];
  }
}
// HF self-energies of the NTAB isospin tables at |k| = kk from the LDS splines
// (constant beyond the last node).
template <int NTAB>
__device__ __forceinline__ void hf_sigma(const double *__restrict__ hf, double kk, double inv_h,
                                         double *sigma) {
  const double u = kk * inv_h;
  int i = static_cast<int>(u);
  double t = u - static_cast<double>(i);
  if (i >= kHfIntervals) {
    i = kHfIntervals;
    t = 0.0;
  }
  const double2 *ab = reinterpret_cast<const double2 *>(hf), *cd = ab + NTAB * kHfEntries;
#pragma unroll
  for (int tau = 0; tau < NTAB; ++tau) {
    const double2 p = ab[tau * kHfEntries + i], q = cd[tau * kHfEntries + i];
    sigma[tau] = fma(t, fma(t, fma(t, q.y, q.x), p.y), p.x);
  }
}

// Carves the block's dynamic LDS; returns the first free double after the
// grid pairs and fills the pointers.  Copies the turn and HF tables (the grid
// pairs are the caller's).
template <int ntab>
__device__ __forceinline__ double *carve_lds(const KArgs &a, const TaskDev *__restrict__ T,
                                             int nd, double *smem, SampleLds &L,
                                             double2 *&g) {
  SinCos *turn = reinterpret_cast<SinCos *>(smem);
  double *ex = reinterpret_cast<double *>(turn + kTurnEntries);
  double *hf = ex + kExp2Entries;
  g = reinterpret_cast<double2 *>(hf + hf_lds_doubles(ntab));
  load_turn_table(turn, ex);
  if constexpr (ntab > 0) load_hf<ntab>(hf, a.hf + 4 * static_cast<size_t>(T->hf_off));
  L.turn = turn;
  L.ex = ex;
  L.hf = ntab ? hf : nullptr;
  L.g = g;
  L.cyc = nullptr;
  return reinterpret_cast<double *>(g + nd * a.phys.nb);
}

// sin and cos of 2 pi u / 128 for u in [0, 128]: the nearest table angle
// 2 pi k / 128 rotated by the residual d, |d| <= pi / 128, whose sine and
// cosine - 1 come from their Taylor series (first omitted terms below 4e-19
// relative to sin d and 4e-18 absolute for cos d).
__device__ __forceinline__ void sincos_turn(const SinCos *__restrict__ tab, double u, double &s,
                                            double &c) {
  const double kf = rint(u);
  const double d = (u - kf) * (2.0 * M_PI / MBPT_TURN_STEPS);  // u - kf exact
  const double z = d * d;
  double ps = fma(z, -1.0 / 5040.0, 1.0 / 120.0);
  ps = fma(z, ps, -1.0 / 6.0);
  const double sd = fma(d * z, ps, d);
  double pc = fma(z, -1.0 / 720.0, 1.0 / 24.0);
  pc = fma(z, pc, -0.5);
  const double cm = z * pc;
  const SinCos t = tab[static_cast<int>(kf)];
  s = fma(t.s, cm, fma(t.c, sd, t.s));
  c = fma(t.c, cm, fma(-t.s, sd, t.c));
}

template <typename F>
__device__ __forceinline__ F fma_t(F x, F y, F z) {
  return __builtin_fma(x, y, z);
}
template <>
__device__ __forceinline__ float fma_t<float>(float x, float y, float z) {
  return __builtin_fmaf(x, y, z);
}

// Coefficient c in {0, +-1, +-2} of loop j in the uniform bitmask m (bits
// 0-7: +1, 8-15: -1, 16-23: +2, 24-31: -2) in precision F, built from its bit
// pattern with scalar instructions only.
template <typename F>
__device__ __forceinline__ F mask_coef(uint32_t m, int j);
template <>
__device__ __forceinline__ double mask_coef<double>(uint32_t m, int j) {
  uint32_t hi = 0u;
  hi = (m & (1u << j)) ? 0x3FF00000u : hi;
  hi = (m & (1u << (8 + j))) ? 0xBFF00000u : hi;
  hi = (m & (1u << (16 + j))) ? 0x40000000u : hi;
  hi = (m & (1u << (24 + j))) ? 0xC0000000u : hi;
  return __hiloint2double(static_cast<int>(hi), 0);
}
template <>
__device__ __forceinline__ float mask_coef<float>(uint32_t m, int j) {
  uint32_t bits = 0u;
  bits = (m & (1u << j)) ? 0x3F800000u : bits;
  bits = (m & (1u << (8 + j))) ? 0xBF800000u : bits;
  bits = (m & (1u << (16 + j))) ? 0x40000000u : bits;
  bits = (m & (1u << (24 + j))) ? 0xC0000000u : bits;
  return __uint_as_float(bits);
}

// out = sum_j c_j v_j over loops j < L, the terms in loop order, from coef(j).
// SKIP0: the coefficients are compile-time constants, so zero terms are left
// out and the first one is taken as it is (under IEEE rules neither a product
// with zero nor a sum with zero folds).
template <int L, bool SKIP0, typename F, typename C>
__device__ __forceinline__ void loop_sum(C &&coef, const F (*k)[3], F *out) {
  bool first = true;
#pragma unroll
  for (int i = 0; i < 3; ++i) out[i] = F(0);
#pragma unroll
  for (int j = 0; j < L; ++j) {
    const F c = coef(j);
    if (SKIP0 && c == F(0)) continue;
#pragma unroll
    for (int i = 0; i < 3; ++i) out[i] = first ? c * k[j][i] : fma_t<F>(c, k[j][i], out[i]);
    first = false;
  }
}
// Coefficients from the uniform bitmask m.
template <int L, bool SKIP0, typename F>
__device__ __forceinline__ void masked_sum(uint32_t m, const F (*k)[3], F *out) {
  loop_sum<L, SKIP0, F>([&](int j) { return mask_coef<F>(m, j); }, k, out);
}
// Coefficients from a row of the descriptor's decoded table: the operations of
// the mask they were decoded from.
template <int L, typename F>
__device__ __forceinline__ void table_sum(const F *c, const F (*k)[3], F *out) {
  loop_sum<L, false, F>([&](int j) { return c[j]; }, k, out);
}
template <typename F>
__device__ __forceinline__ const F *coef_row(const DiagDev *__restrict__ D, int row);
template <>
__device__ __forceinline__ const double *coef_row<double>(const DiagDev *__restrict__ D, int row) {
  return D->coef_d[row];
}
template <>
__device__ __forceinline__ const float *coef_row<float>(const DiagDev *__restrict__ D, int row) {
  return D->coef_f[row];
}

// Descriptor masks of diagram variant V: compile-time constants where
// FixedMasks<ORDER, V> has them, else read from the descriptor.
template <int ORDER, int V>
__device__ __forceinline__ uint32_t lmask_of(const DiagDev *__restrict__ D, int l) {
  if constexpr (FixedMasks<ORDER, V>::kFixed) return FixedMasks<ORDER, V>::lmask[l];
  else return D->lmask[l];
}
template <int ORDER, int V>
__device__ __forceinline__ uint32_t pmask_of(const DiagDev *__restrict__ D, int v) {
  if constexpr (FixedMasks<ORDER, V>::kFixed) return FixedMasks<ORDER, V>::pmask_v[v];
  else return D->pmask_v[v];
}
template <int ORDER, int V>
__device__ __forceinline__ uint32_t qmask_of(const DiagDev *__restrict__ D, int v) {
  if constexpr (FixedMasks<ORDER, V>::kFixed) return FixedMasks<ORDER, V>::qmask_v[v];
  else return D->qmask_v[v];
}
template <int ORDER, int V>
__device__ __forceinline__ uint32_t cut_hole_of(const DiagDev *__restrict__ D, int c) {
  if constexpr (FixedMasks<ORDER, V>::kFixed) return FixedMasks<ORDER, V>::cut_hole[c];
  else return D->cut_hole[c];
}
template <int ORDER, int V>
__device__ __forceinline__ uint32_t cut_part_of(const DiagDev *__restrict__ D, int c) {
  if constexpr (FixedMasks<ORDER, V>::kFixed) return FixedMasks<ORDER, V>::cut_part[c];
  else return D->cut_part[c];
}
template <int ORDER, int V>
__device__ __forceinline__ uint32_t line_mask_of(const DiagDev *__restrict__ D) {
  if constexpr (FixedMasks<ORDER, V>::kFixed) return FixedMasks<ORDER, V>::line_mask;
  else return D->line_mask;
}
template <int ORDER, int V>
__device__ __forceinline__ uint32_t part_mask_of(const DiagDev *__restrict__ D) {
  if constexpr (FixedMasks<ORDER, V>::kFixed) return FixedMasks<ORDER, V>::part_mask;
  else return D->part_mask;
}

// Runs f(std::integral_constant<int, V>) with the diagram variant of a task
// whose first descriptor is D: the one diagram of orders 1-2 (also as a
// single-member group), the diagram id at order 3 for single-diagram tasks,
// for the cycle form (CYF) at fifth order kNarrowCycles where the diagram
// has at most kNarrowCycleMax cycles, the diagram id at order 4 where the
// kernel holds them all (FX4, see fixed4), the generic path (-1) otherwise.
// The branch is uniform per work item.
template <typename Fn, int... I>
__device__ __forceinline__ void with_id(std::integer_sequence<int, I...>, int id, Fn &&f) {
  (void)((id == I ? (f(std::integral_constant<int, I>{}), true) : false) || ...);
}
template <int ORDER, bool G, bool CYF = false, bool FX4 = false, typename Fn>
__device__ __forceinline__ void with_variant(const DiagDev *__restrict__ D, Fn &&f) {
  if constexpr (ORDER <= 2) {
    f(std::integral_constant<int, 0>{});
  } else if constexpr (ORDER == 3 && !G) {
    // ids 0..2 are the order's only diagrams (the host validates task ids)
    if (D->id == 0) f(std::integral_constant<int, 0>{});
    else if (D->id == 1) f(std::integral_constant<int, 1>{});
    else f(std::integral_constant<int, 2>{});
  } else if constexpr (FX4) {
    with_id(std::make_integer_sequence<int, kFixed4Diagrams>{}, D->id, f);
  } else if constexpr (ORDER >= 5 && CYF) {
    if (D->ncyc <= kNarrowCycleMax) f(std::integral_constant<int, kNarrowCycles>{});
    else f(std::integral_constant<int, -1>{});
  } else {
    f(std::integral_constant<int, -1>{});
  }
}

// (p^2)^(reg_exp / 2) for the regulator exponent: HE > 0 is reg_exp / 2 fixed
// at compile time (the quartic regulator's kernels: no selects or loop, and
// vertices with equal momenta share their factors), HE = 0 takes it from the
// launch (a uniform loop).  Both multiply the same factors in the same order.
template <int HE, typename F>
__device__ __forceinline__ F reg_pow(F p2, int half_exp) {
  F r = p2;
  if constexpr (HE > 0) {
#pragma unroll
    for (int e = 1; e < HE; ++e) r *= p2;
  } else {
    for (int e = 1; e < half_exp; ++e) r *= p2;
  }
  return r;
}

// Square root of a finite a >= 0: hardware reciprocal square root refined by
// one coupled step on g = sqrt(a) and h = 1 / (2 sqrt(a)) (doubling its
// correct bits) and one Newton correction of g.  No rescaling: a is clamped to
// the smallest normal (so 0 gives 1.5e-154), and the squared momenta and
// (1 - c)(1 + c) that reach here are far from overflow.
__device__ __forceinline__ double sqrt_normal(double a) {
  a = fmax(a, 0x1p-1022);
  const double y = __builtin_amdgcn_rsq(a);
  double g = a * y;
  double h = 0.5 * y;
  const double r = fma(-g, h, 0.5);
  g = fma(g, r, g);
  h = fma(h, r, h);
  const double d = fma(-g, g, a);
  return fma(d, h, g);
}

// sin theta from its square a in fp32: rsq, then one Newton correction (within
// an ulp of the root), a clamped to 1e-30.  The hardware sine and cosine of the
// azimuth come out short, s^2 + c^2 = 1 - 6.5e-8 on average; the correction
// makes up for that, so the squared momenta are not all too small.
__device__ __forceinline__ float sin_theta_f(float a) {
  a = fmaxf(a, 1e-30f);
  const float y = __builtin_amdgcn_rsqf(a);
  const float g = a * y;
  return fmaf(fmaf(a, 6.5e-8f, fmaf(-g, g, a)), 0.5f * y, g);
}

// 1/d from the hardware reciprocal and two Newton steps (d normal and finite;
// within about one ulp).
__device__ __forceinline__ double rcp_newton(double d) {
  double r = __builtin_amdgcn_rcp(d);
  double e = fma(-d, r, 1.0);
  r = fma(r, e, r);
  e = fma(-d, r, 1.0);
  return fma(r, e, r);
}

// (s, c) += (s2, c2) with the rounding error of the leading parts kept
__device__ __forceinline__ void pair_merge(double &s, double &c, double s2, double c2) {
  const double t = s + s2;
  const double bp = t - s;
  const double err = (s - (t - bp)) + (s2 - bp);
  s = t;
  c = c + c2 + err;
}

// ---------------------------------------------------------------------------
// Per-sample integrand in fp64.  Returns the weight; writes the VEGAS bin of
// every dimension to bins[].

// Grid pair of bin b of dimension m (radius, cosine and azimuth of each loop
// in turn): with the bin's lower edge e, width w and a random word's fraction
// r = (f + 1/2) 2^-32, f whole, the mapped coordinate x = e + r w is one fma of
// f with the pair, scaled to what the loop momentum is built from: the radius
// R x0, the cosine 2 x1 - 1, and the azimuth in table steps of the turn (AZ),
// or in turns from -1/2 to 1/2 (fp32: half the rounding of 0 to 1).  Scaling
// here, once per work item, takes a multiplication per coordinate and the
// fraction's conversion to [0, 1) out of every sample; on MI355X (with the
// one-product bin split of vegas_map and the short fp32 root) orders 2+3, 36
// tasks x 2^24 fp32, 7.67 -> 6.95 ms per iteration, and the 585 fourth-order
// tasks fp32 (2^21) 24.8 -> 22.9 ms, fp64 (500 009) 7.1 -> 6.6 ms.
template <bool AZ>
__device__ __forceinline__ double2 grid_pair(int m, double e0, double e1, double R) {
  const double w = e1 - e0;
  const double e = fma(w, 0x1p-33, e0);
  const double ws = w * 0x1p-32;
  const int role = m % 3;
  if (role == 0) return make_double2(R * e, R * ws);
  if (role == 1) return make_double2(fma(2.0, e, -1.0), 2.0 * ws);
  return AZ ? make_double2(MBPT_TURN_STEPS * e, MBPT_TURN_STEPS * ws) : make_double2(e - 0.5, ws);
}

// Radius of the sphere loop j of the task's first descriptor D is drawn from.
__device__ __forceinline__ double loop_radius(const TaskDev *__restrict__ T,
                                              const DiagDev *__restrict__ D, int j) {
  return D->loop_part[j] ? T->Rp : T->Rh;
}

// Philox words -> VEGAS bins and scaled coordinates (see grid_pair; fp64,
// identical for both integrand precisions).  Returns jc times the product of
// the pairs' widths, the VEGAS Jacobian.
template <int ND>
__device__ __forceinline__ double vegas_map(const KArgs &a, const TaskDev *__restrict__ T,
                                            const double2 *__restrict__ g, double jc, uint64_t s,
                                            uint32_t iter, double *x, int *bins) {
  constexpr int NW = (ND + 3) / 4;
  const uint32_t nb = static_cast<uint32_t>(a.phys.nb);
  // counter (s lo, s hi, iteration, word block), key (seed, task)
  uint32_t wd[4 * NW];
#pragma unroll
  for (int j = 0; j < NW; ++j)
    philox4x32_10(static_cast<uint32_t>(s), static_cast<uint32_t>(s >> 32), iter,
                  static_cast<uint32_t>(j), a.phys.seed, T->key, wd + 4 * j);
  // w nb = b 2^32 + f: bin b and fraction f from one 32 x 32 product
  double jac = jc;
#pragma unroll
  for (int m = 0; m < ND; ++m) {
    const uint64_t y = static_cast<uint64_t>(wd[m]) * nb;
    const int b = static_cast<int>(y >> 32);
    const double2 ew = g[m * nb + b];
    x[m] = fma(static_cast<double>(static_cast<uint32_t>(y)), ew.y, ew.x);
    jac *= ew.y;
    bins[m] = b;
  }
  return jac;
}

// Sample-independent part of the Jacobian of a task (uniform, hoisted out of
// the sample loops): nb^ND prod_m w_m from the VEGAS map times 4 pi R_j rad_j^2
// per loop from the spherical map, times 1/n, where the product of the grid
// pairs' widths holds prod_m w_m 2^-32, R_j per radius, 2 per cosine and (AZ)
// MBPT_TURN_STEPS per azimuth, and rad_j^2 is per sample.  (The large power of
// two comes in first, so no partial product leaves the normal range.)
template <int ORDER, bool AZ>
__device__ __forceinline__ double jac_const(const KArgs &a, const TaskDev *__restrict__ T) {
  constexpr int L = ORDER + 1;
  double c = T->inv_density;
  const double nb = static_cast<double>(a.phys.nb) * 0x1p32;
#pragma unroll
  for (int m = 0; m < 3 * L; ++m) c *= nb;
#pragma unroll
  for (int j = 0; j < L; ++j) c *= (4.0 * M_PI) / (2.0 * (AZ ? MBPT_TURN_STEPS : 1.0));
  return c;
}

// Loop momenta of a sample: radius, cos theta and azimuth from the map, the
// squares of the radii, and the whole Jacobian.  The azimuth's sine and cosine
// come from the turn table in fp64 and from the hardware (in revolutions) in
// fp32.
template <int ORDER, bool AZ>
__device__ __forceinline__ double loop_momenta(const KArgs &a, const TaskDev *__restrict__ T,
                                               const SampleLds &Ls, double jc, uint64_t s,
                                               uint32_t iter, int *bins, double (*k)[3],
                                               double *r2) {
  constexpr int L = ORDER + 1;
  double x[3 * L];
  const double jac = vegas_map<3 * L>(a, T, Ls.g, jc, s, iter, x, bins);
  double rp = 1.0;
#pragma unroll
  for (int j = 0; j < L; ++j) {
    const double rad = x[3 * j], ct = x[3 * j + 1];
    const double st = sqrt_normal((1.0 - ct) * (1.0 + ct));
    double sp, cp;
    sincos_turn(Ls.turn, AZ ? x[3 * j + 2] : (x[3 * j + 2] + 0.5) * MBPT_TURN_STEPS, sp, cp);
    const double rs = rad * st;
    k[j][0] = rs * cp;
    k[j][1] = rs * sp;
    k[j][2] = rad * ct;
    r2[j] = rad * rad;
    rp = j == 0 ? rad : rp * rad;
  }
  return jac * (rp * rp);
}
template <int ORDER, bool AZ>
__device__ __forceinline__ double loop_momenta(const KArgs &a, const TaskDev *__restrict__ T,
                                               const SampleLds &Ls, double jc, uint64_t s,
                                               uint32_t iter, int *bins, float (*k)[3], float *r2) {
  static_assert(!AZ, "the fp32 azimuth is taken in revolutions");
  constexpr int L = ORDER + 1;
  double x[3 * L];
  const double jac = vegas_map<3 * L>(a, T, Ls.g, jc, s, iter, x, bins);
  double rp = 1.0;
#pragma unroll
  for (int j = 0; j < L; ++j) {
    const float rad = static_cast<float>(x[3 * j]), ct = static_cast<float>(x[3 * j + 1]);
    const float st = sin_theta_f((1.0f - ct) * (1.0f + ct));
    const float rev = static_cast<float>(x[3 * j + 2]);
    const float rs = -rad * st;  // half a turn from rev to the azimuth
    k[j][0] = rs * __builtin_amdgcn_cosf(rev);
    k[j][1] = rs * __builtin_amdgcn_sinf(rev);
    k[j][2] = rad * ct;
    r2[j] = rad * rad;
    rp = j == 0 ? x[3 * j] : rp * x[3 * j];
  }
  return jac * (rp * rp);
}

// m with the sign of t (1 if negative: k^2 below kF^2) shifted in at bit 0, one
// instruction.
__device__ __forceinline__ uint32_t push_sign(uint32_t m, float t) {
  return __builtin_amdgcn_alignbit(m, __float_as_uint(t), 31);
}
__device__ __forceinline__ uint32_t push_sign(uint32_t m, double t) {
  return __builtin_amdgcn_alignbit(m, static_cast<uint32_t>(__double2hiint(t)), 31);
}

// True if some label assignment survives the Pauli factors: neutron matter
// needs every line allowed as a neutron; nuclear matter needs one isospin
// configuration whose lines are all allowed.  A sample that fails does no
// further work (its weight is exactly zero); this also keeps structurally
// vanishing denominators (a one-particle-one-hole cut, where isospin
// conservation forces the same Fermi momentum on both lines) out of the
// division.
template <int Q>
__device__ __forceinline__ bool pauli_allowed(const KArgs &a, const DiagDev *__restrict__ D,
                                              uint32_t okN, uint32_t okP, uint32_t lmask) {
  if (Q == 2) return okN == lmask;
  const GroupDev *__restrict__ G = a.groups + D->group_off;
  bool any = false;
  for (int gi = 0; gi < D->ngroups; ++gi) {
    const uint32_t tau = G[gi].tau;
    any |= (((~tau & ~okN) | (tau & ~okP)) & lmask) == 0u;
  }
  return any;
}

// Spin(-isospin) label sum of one diagram, summed over the isospin
// configurations whose lines all pass the Pauli test.  Mode 0 evaluates each
// configuration's sum as the multilinear polynomial
//   sum_E c_E prod_{v not in E} V_d,v prod_{v in E} V_e,v
// (E: set of vertices taking the exchange term; c_E integer, compiled on the
// host from the nonzero label assignments): the monomials of the first
// ORDER/2 vertices and of the rest are tabulated once per sample, so a
// configuration costs 2^ORDER + 2^(ORDER - ORDER/2) multiply-adds however
// many assignments it holds.  Mode 1 walks the compressed assignment list.
// The 2^ORDER coefficients of a configuration in precision F (contiguous).
template <int ORDER, typename F>
__device__ __forceinline__ const F *coef_run(const double *block) {
  return block;
}
template <>
__device__ __forceinline__ const float *coef_run<1, float>(const double *block) {
  return reinterpret_cast<const float *>(block + 2);
}
template <>
__device__ __forceinline__ const float *coef_run<2, float>(const double *block) {
  return reinterpret_cast<const float *>(block + 4);
}
template <>
__device__ __forceinline__ const float *coef_run<3, float>(const double *block) {
  return reinterpret_cast<const float *>(block + 8);
}
template <>
__device__ __forceinline__ const float *coef_run<4, float>(const double *block) {
  return reinterpret_cast<const float *>(block + 16);
}
template <>
__device__ __forceinline__ const float *coef_run<5, float>(const double *block) {
  return reinterpret_cast<const float *>(block + 32);
}
template <typename F>
__device__ __forceinline__ F term_mult(const TermDev &t) {
  return t.mult;
}
template <>
__device__ __forceinline__ float term_mult<float>(const TermDev &t) {
  return t.multf;
}

// M[e] = prod_{v < NV} (bit v of e ? Ve[v] : Vd[v])
template <int NV, typename F>
__device__ __forceinline__ void monomials(const F *Vd, const F *Ve, F *M) {
  M[0] = F(1);
#pragma unroll
  for (int v = 0; v < NV; ++v) {
#pragma unroll
    for (int e = 0; e < (1 << v); ++e) {
      M[e + (1 << v)] = M[e] * Ve[v];
      M[e] = M[e] * Vd[v];
    }
  }
}

// Product of the energy denominators of one isospin configuration when the
// single-particle energies depend on isospin (HF spectrum in nuclear matter):
// D_c = Dn_c + sum over the cut's proton lines of +-(eps_p - eps_n), with
// Dn_c the denominator with every line a neutron.
template <int ORDER, int V>
__device__ __forceinline__ double group_den(const DiagDev *__restrict__ D, uint32_t tau,
                                            const double *Dn, const double *deps) {
  constexpr int NL = 2 * ORDER;
  double prod = 1.0;
#pragma unroll
  for (int c = 0; c < ORDER - 1; ++c) {
    const uint32_t hm = cut_hole_of<ORDER, V>(D, c) & tau, pm = cut_part_of<ORDER, V>(D, c) & tau;
    double Dc = Dn[c];
#pragma unroll
    for (int l = 0; l < NL; ++l) {
      uint32_t hi = (hm & (1u << l)) ? 0x3FF00000u : 0u;
      hi = (pm & (1u << l)) ? 0xBFF00000u : hi;
      Dc = fma(__hiloint2double(static_cast<int>(hi), 0), deps[l], Dc);
    }
    prod *= Dc;
  }
  return prod;
}

// Cycle set and cycle count of E (fourth order and below: at most 17
// cycles, the 32-bit packing).
template <int ORDER, int V = -1>
__device__ __forceinline__ void cycles_of_e(const DiagDev *__restrict__ D, int E,
                                            CycWordV<ORDER, V> &m, uint32_t &n) {
  if constexpr (ORDER >= 5 && V != kNarrowCycles) {
    const uint64_t w = D->cyc_e[E];
    m = w & ((uint64_t{1} << 56) - 1);
    n = static_cast<uint32_t>(w >> 56);
  } else {
    const uint32_t w = D->cyc_e32[E];
    m = w & 0xFFFFFFu;
    n = w >> 24;
  }
}

// True if some vertex-term choice E has every one of its label cycles
// allowed for at least one isospin (ab: cycles allowed as neutrons or as
// protons): exactly when some isospin configuration passes the Pauli test.
template <int ORDER, int V = -1>
__device__ __forceinline__ bool cycle_any(const DiagDev *__restrict__ D, CycWordV<ORDER, V> ab) {
  bool any = false;
#pragma unroll
  for (int E = 0; E < (1 << ORDER); ++E) {
    CycWordV<ORDER, V> m;
    uint32_t n;
    cycles_of_e<ORDER, V>(D, E, m, n);
    any |= (ab & m) == m;
  }
  return any;
}

// 2^e for 0 <= e <= 30 from its bit pattern
template <typename F>
__device__ __forceinline__ F pow2_bits(uint32_t e) {
  return __hiloint2double(static_cast<int>((1023u + e) << 20), 0);
}
template <>
__device__ __forceinline__ float pow2_bits<float>(uint32_t e) {
  return __uint_as_float((127u + e) << 23);
}

template <int ORDER, typename W>
__device__ __forceinline__ uint32_t popc_w(W x) {
  if constexpr (sizeof(W) == 8) return static_cast<uint32_t>(__popcll(x));
  else return static_cast<uint32_t>(__popc(x));
}

// Cycle form of the nuclear-matter label sum.  Expanding every vertex into
// its direct and exchange terms, the choice E (bit v: exchange at vertex v)
// contributes (-1)^{|E|} prod_{v not in E} V_d,v prod_{v in E} V_e,v times
// the number of labellings that keep each of E's label cycles uniform with
// every line allowed: 2 spin states times the isospins (neutron, proton)
// allowed on all of the cycle's lines, per cycle.  With cA / cB the cycles
// whose lines are all allowed as neutrons / protons, E's count is 0 if a
// cycle is allowed for neither, else 2^{cycles(E) + cycles allowed for both}.
// The monomials carry the sign (nVe = -V_e) and are tabulated as in the
// configuration form; the counts are integers, so the sum equals the sum over
// isospin configurations up to rounding.
template <int ORDER, typename F, bool ABS = false, int V = -1>
__device__ __forceinline__ F label_sum_cycles(const DiagDev *__restrict__ D, const F *Vd,
                                              const F *nVe, CycWordV<ORDER, V> cA,
                                              CycWordV<ORDER, V> cB, F *absum = nullptr) {
  using W = CycWordV<ORDER, V>;
  constexpr int H = ORDER / 2;
  constexpr int NA = 1 << H, NB = 1 << (ORDER - H);
  F MA[NA], MB[NB];
  monomials<H>(Vd, nVe, MA);
  monomials<ORDER - H>(Vd + H, nVe + H, MB);
  const W ab = cA | cB, both = cA & cB;
  F AA[ABS ? NA : 1], AB[ABS ? NB : 1];
  if constexpr (ABS) {
#pragma unroll
    for (int i = 0; i < NA; ++i) AA[i] = fabs(MA[i]);
#pragma unroll
    for (int i = 0; i < NB; ++i) AB[i] = fabs(MB[i]);
  }
  F acc = F(0), aacc = F(0);
#pragma unroll
  for (int eb = 0; eb < NB; ++eb) {
    F in = F(0), ain = F(0);
#pragma unroll
    for (int ea = 0; ea < NA; ++ea) {
      const int E = ea | (eb << H);
      W m;
      uint32_t n;
      cycles_of_e<ORDER, V>(D, E, m, n);
      const uint32_t e = popc_w<ORDER>(both & m) + n;
      const F c = (ab & m) == m ? pow2_bits<F>(e) : F(0);
      in = fma_t<F>(c, MA[ea], in);
      if constexpr (ABS) ain = fma_t<F>(c, AA[ea], ain);
    }
    acc = fma_t<F>(in, MB[eb], acc);
    if constexpr (ABS) aacc = fma_t<F>(ain, AB[eb], aacc);
  }
  if constexpr (ABS) *absum = aacc;
  return acc;
}

// The cycle form with the sample's counts from the count table.  Against the
// bit operations of label_sum_cycles (six per choice) the counts cost half an
// instruction per choice: 585 fourth-order tasks x 2^21 on MI355X fp32 21.8 ->
// 18.4 ms per iteration, 500 009 samples fp64 6.54 -> 6.22 ms (with the Pauli
// tests by sign, push_sign).
template <int ORDER, typename F, bool ABS = false>
__device__ __forceinline__ F label_sum_counts(const LabelCounts<ORDER> &t, const F *Vd,
                                              const F *nVe, F *absum = nullptr) {
  constexpr int H = ORDER / 2;
  constexpr int NA = 1 << H, NB = 1 << (ORDER - H);
  F c[NA * NB];
#pragma unroll
  for (int i = 0; i < NA * NB / 4; ++i) {
    const auto lo = __builtin_amdgcn_cvt_pk_f32_bf8(static_cast<int>(t.w[i]), false);
    const auto hi = __builtin_amdgcn_cvt_pk_f32_bf8(static_cast<int>(t.w[i]), true);
    c[4 * i] = lo[0];
    c[4 * i + 1] = lo[1];
    c[4 * i + 2] = hi[0];
    c[4 * i + 3] = hi[1];
  }
  F MA[NA], MB[NB];
  monomials<H>(Vd, nVe, MA);
  monomials<ORDER - H>(Vd + H, nVe + H, MB);
  F acc = F(0), aacc = F(0);
#pragma unroll
  for (int eb = 0; eb < NB; ++eb) {
    F in = c[eb * NA] * MA[0], ain = F(0);
#pragma unroll
    for (int ea = 1; ea < NA; ++ea) in = fma_t<F>(c[eb * NA + ea], MA[ea], in);
    if constexpr (ABS) {
#pragma unroll
      for (int ea = 0; ea < NA; ++ea) ain = fma_t<F>(c[eb * NA + ea], fabs(MA[ea]), ain);
      aacc = fma_t<F>(ain, fabs(MB[eb]), aacc);
    }
    acc = fma_t<F>(in, MB[eb], acc);
  }
  if constexpr (ABS) *absum = aacc;
  return acc;
}

// What the label sum needs of a sample's Pauli tests.
template <int ORDER, int V, LabelForm LF>
struct LabelState {};
template <int ORDER, int V>
struct LabelState<ORDER, V, kCycles> {
  CycWordV<ORDER, V> cA, cB;  // label cycles open as neutrons / protons
};
template <int ORDER, int V>
struct LabelState<ORDER, V, kCounts> {
  LabelCounts<ORDER> c;
};

// The label state of a sample whose lines are allowed as neutrons (okN) and
// protons (okP); false if no label assignment survives.
template <int ORDER, int Q, int V, LabelForm LF>
__device__ __forceinline__ bool label_state(const KArgs &a, const DiagDev *__restrict__ D,
                                            const SampleLds &Ls, uint32_t okN, uint32_t okP,
                                            LabelState<ORDER, V, LF> &st) {
  const uint32_t lmask = line_mask_of<ORDER, V>(D);
  if constexpr (LF == kCounts) {
    if ((okN | okP) != lmask) return false;  // a line open to neither
    st.c = static_cast<const LabelCounts<ORDER> *>(Ls.cyc)[okN ^ okP];
    uint32_t any = st.c.w[0];
#pragma unroll
    for (int i = 1; i < (1 << ORDER) / 4; ++i) any |= st.c.w[i];
    return any != 0u;
  } else if constexpr (LF == kCycles) {
    const CycWordV<ORDER, V> *tab = static_cast<const CycWordV<ORDER, V> *>(Ls.cyc);
    st.cA = tab[~okN & lmask];
    st.cB = tab[~okP & lmask];
    return cycle_any<ORDER, V>(D, st.cA | st.cB);
  } else {
    return pauli_allowed<Q>(a, D, okN, okP, lmask);
  }
}

// ISO: divide each configuration's sum by its own denominators (Dn, deps).
// X: the explicit assignment list instead of the polynomial (compile-time, so
// a kernel holds the state of one form only).
// ABS: also the same sum with every term in absolute value (*absum), the
// scale against which the fp32 integrand's cancellation is judged.
template <int ORDER, int Q, typename F, bool ISO, bool X, int V, bool ABS = false>
__device__ __forceinline__ F label_sum(const KArgs &a, const DiagDev *__restrict__ D,
                                       const F *Vd, const F *Ve, uint32_t okN, uint32_t okP,
                                       uint32_t lmask, uint32_t &units, const double *Dn,
                                       const double *deps, F *absum = nullptr) {
  const GroupDev *__restrict__ G = a.groups + D->group_off;
  const int ngroups = D->ngroups;
  F acc = F(0), aacc = F(0);
  if constexpr (!X) {
    constexpr int H = ORDER / 2;
    constexpr int NA = 1 << H, NB = 1 << (ORDER - H);
    F MA[NA], MB[NB];
    monomials<H>(Vd, Ve, MA);
    monomials<ORDER - H>(Vd + H, Ve + H, MB);
    F AA[ABS ? NA : 1], AB[ABS ? NB : 1];
    if constexpr (ABS) {
#pragma unroll
      for (int i = 0; i < NA; ++i) AA[i] = fabs(MA[i]);
#pragma unroll
      for (int i = 0; i < NB; ++i) AB[i] = fabs(MB[i]);
    }
    // one isospin configuration's polynomial sum_E c_E prod V
    auto add_config = [&](const F *c, uint32_t tau) {
      F gs = F(0);
#pragma unroll
      for (int eb = 0; eb < NB; ++eb) {
        F in = F(0);
#pragma unroll
        for (int ea = 0; ea < NA; ++ea) in = fma_t<F>(c[eb * NA + ea], MA[ea], in);
        gs = fma_t<F>(in, MB[eb], gs);
      }
      if constexpr (ABS) {
#pragma unroll
        for (int eb = 0; eb < NB; ++eb) {
          F in = F(0);
#pragma unroll
          for (int ea = 0; ea < NA; ++ea) in = fma_t<F>(fabs(c[eb * NA + ea]), AA[ea], in);
          aacc = fma_t<F>(in, AB[eb], aacc);
        }
      }
      if constexpr (ISO) gs *= rcp_newton(group_den<ORDER, V>(D, tau, Dn, deps));
      acc += gs;
    };
    if constexpr (Q == 2 && fixed_labels<FixedMasks<ORDER, V>>::value) {
      // neutron matter, a diagram of the fixed tables: its one configuration
      // with compile-time coefficients
      F c[NA * NB];
#pragma unroll
      for (int i = 0; i < NA * NB; ++i)
        c[i] = static_cast<F>(FixedMasks<ORDER, V>::label_coef_q2[i]);
      ++units;
      add_config(c, 0u);
    } else {
      for (int gi = 0; gi < ngroups; ++gi) {
        const uint32_t tau = G[gi].tau;
        bool ok = true;
        if (Q == 4) ok = (((~tau & ~okN) | (tau & ~okP)) & lmask) == 0u;
        if (ok) {
          ++units;
          const F *__restrict__ C = coef_run<ORDER, F>(a.gcoef + G[gi].coef_off);
          F c[NA * NB];  // one batch of scalar loads, then the multiply-adds
#pragma unroll
          for (int i = 0; i < NA * NB; ++i) c[i] = C[i];
          add_config(c, tau);
        }
      }
    }
  } else {
    for (int gi = 0; gi < ngroups; ++gi) {
      const uint32_t tau = G[gi].tau;
      const int first = G[gi].first, cnt = G[gi].count;
      bool ok = true;
      if (Q == 4) ok = (((~tau & ~okN) | (tau & ~okP)) & lmask) == 0u;
      if (ok) {
        units += cnt;
        F gs = F(0);
        for (int t = first; t < first + cnt; ++t) {
          const TermDev tm = a.terms[t];
          F prod = F(1), aprod = F(1);
#pragma unroll
          for (int v = 0; v < ORDER; ++v) {
            const uint32_t code = (tm.codes >> (2 * v)) & 3u;
            const F ca = code != 1u ? F(1) : F(0);
            const F cb = code != 0u ? F(-1) : F(0);
            prod *= fma_t<F>(ca, Vd[v], cb * Ve[v]);
            if constexpr (ABS) aprod *= fma_t<F>(ca, fabs(Vd[v]), -cb * fabs(Ve[v]));
          }
          gs = fma_t<F>(term_mult<F>(tm), prod, gs);
          if constexpr (ABS) aacc = fma_t<F>(fabs(term_mult<F>(tm)), aprod, aacc);
        }
        if constexpr (ISO) gs *= rcp_newton(group_den<ORDER, V>(D, tau, Dn, deps));
        acc += gs;
      }
    }
  }
  if constexpr (ABS) *absum = aacc;
  return acc;
}

// exp(x) for x <= 0 by Tang's table-driven method (ACM TOMS 15, 1989): with
// k = rint(64 x / ln 2) = 64 m + j, exp(x) = 2^m 2^(j/64) e^r, r = x - k ln2/64
// (|r| <= ln2/128, reduced with the split constant so k HI is exact), e^r - 1
// from its degree-6 Taylor polynomial (truncation below 3e-20) and 2^(j/64)
// from the LDS table.  Within about one ulp; arguments below -1000 give 0.
__device__ __forceinline__ double exp_nonpos(double x, const double *ex) {
  x = fmax(x, -1000.0);
  const double kd = __builtin_rint(x * MBPT_INV_LN2_64);
  const int k = static_cast<int>(kd);
  const double r = fma(-kd, MBPT_LN2_64_LO, fma(-kd, MBPT_LN2_64_HI, x));
  double q = fma(r, 1.0 / 720.0, 1.0 / 120.0);
  q = fma(q, r, 1.0 / 24.0);
  q = fma(q, r, 1.0 / 6.0);
  q = fma(q, r, 0.5);
  q = fma(q, r, 1.0);
  const double t = ex[k & 63];
  return __builtin_ldexp(fma(t, r * q, t), k >> 6);
}

// Vertices of one diagram at the loop momenta k.  With the relative momenta p
// and p', the antisymmetrised matrix element's terms are V_d = V(p, p') = V0 +
// Vy / dd and V_e = V(p, -p') = V0 + Vy / de up to their regulators, dd and de
// = p^2 + p'^2 -+ 2 p.p' + m^2.  Every label term takes one of them per vertex,
// so the products dd de of all vertices come out of the label sum:
//   Vd[v] = (V0 dd + Vy) de,  Ve[v] = (V0 de + Vy) dd  (NEG: -Ve[v]),
//   den = prod_v dd de,
// and one reciprocal per sample divides by den and the energy denominators
// together.  Inverting the 2n Yukawa denominators instead (prefix products
// around one reciprocal) took 3n more multiplications and held 4n values (with
// the loop sums' zero terms: 585 fourth-order tasks fp32 22.9 -> 21.8 ms per
// iteration of 2^21 samples on MI355X, orders 2+3 fp32 6.95 -> 6.73 ms).  The
// regulators come out too, as exp(-yreg), yreg = 4^n sum_v (p^n + p'^n) (n the
// regulator exponent).  V0, Vy: the interaction, in fp32 divided by
// Phys::vscale, so that one of them is 1 and the other at most 1.  KY: *ky adds
// the Yukawa denominators' condition numbers (s + 2 |p.p'|)(1 / dd + 1 / de), if
// rel (uniform).
template <int ORDER, int V, int HE, bool TD, bool NEG, bool KY, typename F>
__device__ __forceinline__ void vertex_terms(const KArgs &a, const DiagDev *__restrict__ D,
                                             const F (*k)[3], F V0, F Vy, F *Vd, F *Ve, F &den,
                                             F &yreg, bool rel = false, F *ky = nullptr) {
  constexpr int L = ORDER + 1;
  const F m2 = static_cast<F>(a.phys.m2);
#pragma unroll
  for (int v = 0; v < ORDER; ++v) {
    F p[3], q[3];  // 2 p and 2 p'
    if constexpr (TD) {
      table_sum<L, F>(coef_row<F>(D, 2 * ORDER + 2 * v), k, p);
      table_sum<L, F>(coef_row<F>(D, 2 * ORDER + 2 * v + 1), k, q);
    } else {
      masked_sum<L, FixedMasks<ORDER, V>::kFixed, F>(pmask_of<ORDER, V>(D, v), k, p);
      masked_sum<L, FixedMasks<ORDER, V>::kFixed, F>(qmask_of<ORDER, V>(D, v), k, q);
    }
    const F p2 = p[0] * p[0] + p[1] * p[1] + p[2] * p[2];
    const F q2 = q[0] * q[0] + q[1] * q[1] + q[2] * q[2];
    const F pq = p[0] * q[0] + p[1] * q[1] + p[2] * q[2];
    const F pn = reg_pow<HE>(p2, a.phys.half_exp), qn = reg_pow<HE>(q2, a.phys.half_exp);
    yreg = v == 0 ? pn + qn : yreg + (pn + qn);
    const F s2 = fma_t<F>(F(0.25), p2 + q2, m2);
    const F dd = fma_t<F>(F(-0.5), pq, s2), de = fma_t<F>(F(0.5), pq, s2);
    const F dde = dd * de;
    Vd[v] = fma_t<F>(V0, dd, Vy) * de;
    Ve[v] = (NEG ? fma_t<F>(-V0, de, -Vy) : fma_t<F>(V0, de, Vy)) * dd;
    den = v == 0 ? dde : den * dde;
    if constexpr (KY) {
      if (rel) {
        const F scale = fma_t<F>(F(0.5), fabs(pq), s2);
        *ky = fma_t<F>(scale, (dd + de) * __builtin_amdgcn_rcpf(dde), *ky);
      }
    }
  }
}

// (hbar^2 / 2m)^-NC, the unit of 1 / prod_c D_c with the denominators formed from
// the squared momenta (uniform).
template <int NC>
__device__ __forceinline__ double energy_unit(const KArgs &a) {
  double u = 1.0;
#pragma unroll
  for (int c = 0; c < NC; ++c) u *= a.phys.inv_hb2m;
  return u;
}

// Contribution of one diagram at the loop momenta k (prefactor, regulators,
// label sum and denominators; without the Jacobian and 1/n).  HF: single-
// particle energies of the Hartree-Fock spectrum (tables in LDS).
// REG: also add the regularised components w_k = w prod_c D_c / (D_c - k eta)
// to wr[k - 1].
template <int ORDER, int Q, bool HF, bool REG, bool X, int V, int HE, LabelForm LF,
          bool SCR = false, bool TD = false>
__device__ __forceinline__ double diag_weight64(const KArgs &a, const TaskDev *__restrict__ T,
                                                const DiagDev *__restrict__ D,
                                                const SampleLds &Ls, const double (*k)[3],
                                                const double *r2, uint32_t &npass,
                                                uint32_t &nterms, double *wr) {
  constexpr int L = ORDER + 1;
  constexpr int NL = 2 * ORDER;
  constexpr int NC = ORDER - 1;

  // line momenta -> occupation tests and energies
  double eps[NL], deps[NL];
  uint32_t inN = 0, inP = 0;  // bit l: line l inside the Fermi sphere
#pragma unroll
  for (int l = NL - 1; l >= 0; --l) {
    double kv[3];
    if (l < L) {
      // slot l < L carries loop momentum l itself
      kv[0] = k[l][0];
      kv[1] = k[l][1];
      kv[2] = k[l][2];
    } else {
      if constexpr (TD) table_sum<L, double>(D->coef_d[l], k, kv);
      else masked_sum<L, FixedMasks<ORDER, V>::kFixed, double>(lmask_of<ORDER, V>(D, l), k, kv);
    }
    // (a loop line's k^2 is its squared radius)
    const double k2 = l < L ? r2[l < L ? l : 0]
                            : kv[0] * kv[0] + kv[1] * kv[1] + kv[2] * kv[2];
    // the free spectrum's energies in units of hbar^2 / 2m (energy_unit)
    eps[l] = k2;
    deps[l] = 0.0;
    inN = push_sign(inN, k2 - T->kF2[0]);
    if (Q == 4) inP = push_sign(inP, k2 - T->kF2[1]);
  }
  // a hole line is allowed if occupied, a particle line if empty
  const uint32_t lmask = line_mask_of<ORDER, V>(D), pmask = part_mask_of<ORDER, V>(D);
  const uint32_t okN = (inN ^ pmask) & lmask;
  const uint32_t okP = (inP ^ pmask) & lmask;
  LabelState<ORDER, V, LF> ls;
  if (!label_state<ORDER, Q, V, LF>(a, D, Ls, okN, okP, ls)) return 0.0;
  if constexpr (SCR) return 1.0;  // the Pauli screen (see screen_on)
  ++npass;

  // HF: the energies in MeV plus the self-energy of a neutron, and for nuclear
  // matter the proton-neutron difference, of the samples that pass only (the
  // spline gathers are what the kernel waits for)
  if constexpr (HF) {
#pragma unroll
    for (int l = 0; l < NL; ++l) {
      double sigma[Q == 4 ? 2 : 1];
      hf_sigma<(Q == 4 ? 2 : 1)>(Ls.hf, sqrt_normal(eps[l]), T->hf_inv_h, sigma);
      eps[l] = fma(a.phys.hb2m, eps[l], sigma[0]);
      if constexpr (Q == 4) deps[l] = sigma[1] - sigma[0];
    }
  }

  // energy denominators (with every line a neutron when they depend on
  // isospin; the label sum then corrects them per configuration)
  constexpr bool iso_den = Q == 4 && HF;
  double dprod = 1.0;
  double Dn[NC > 0 ? NC : 1];
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const uint32_t hm = cut_hole_of<ORDER, V>(D, c), pm = cut_part_of<ORDER, V>(D, c);
    double Dc = 0.0;
#pragma unroll
    for (int l = 0; l < NL; ++l) {
      if constexpr (FixedMasks<ORDER, V>::kFixed) {
        if (hm & (1u << l)) Dc += eps[l];
        else if (pm & (1u << l)) Dc -= eps[l];
      } else {
        uint32_t hi = (hm & (1u << l)) ? 0x3FF00000u : 0u;
        hi = (pm & (1u << l)) ? 0xBFF00000u : hi;
        Dc = fma(__hiloint2double(static_cast<int>(hi), 0), eps[l], Dc);
      }
    }
    Dn[c] = Dc;
    dprod *= Dc;
  }

  double Vd[ORDER], Ve[ORDER], den, yreg;
  vertex_terms<ORDER, V, HE, TD, LF != kConfigs, false, double>(a, D, k, a.phys.V0, a.phys.Vy, Vd,
                                                                Ve, den, yreg);
  const double regall = exp_nonpos(-yreg * (a.phys.invLn * a.phys.quarter_n), Ls.ex);

  double acc;
  if constexpr (LF != kConfigs) {
    ++nterms;
    if constexpr (LF == kCounts) acc = label_sum_counts<ORDER, double>(ls.c, Vd, Ve);
    else acc = label_sum_cycles<ORDER, double, false, V>(D, Vd, Ve, ls.cA, ls.cB);
  } else {
    acc = label_sum<ORDER, Q, double, iso_den, X, V>(a, D, Vd, Ve, okN, okP, lmask, nterms, Dn,
                                                     deps);
  }
  const double pref = D->pref * (HF ? 1.0 : energy_unit<NC>(a));
  if constexpr (REG) {
    // Each component's shifted product (empty at first order) by its own
    // reciprocal. One reciprocal for all of them, from products of the shifted
    // products on either side, keeps these live across the components: fifth order
    // then fits one wave per SIMD instead of two (five nuclear diagrams x 2^23
    // samples, two components, on MI355X: 3.43 ms per iteration, 2.29 this way),
    // and the grouped fourth-order diagrams (15 points x 2^18, three components)
    // take 10.7 ms instead of 10.4.
    const double base = pref * regall * acc * rcp_newton(den);
#pragma unroll
    for (int r = 0; r < kMaxReg; ++r) {
      if (r < a.nreg) {
        const double eta = (r + 1) * (a.reg_eta * a.phys.inv_hb2m);
        double x = 1.0;
#pragma unroll
        for (int c = 0; c < NC; ++c) x *= Dn[c] - eta;
        // (a shift may be any finite energy: the product can overflow)
        wr[r] = fma(base, __builtin_isinf(x) ? 0.0 : rcp_newton(x), wr[r]);
      }
    }
    return base * rcp_newton(dprod);
  }
  // (with isospin-dependent energies the label sum holds the denominators)
  return pref * regall * acc * rcp_newton(iso_den ? den : den * dprod);
}

// One sample of a task: VEGAS map, loop momenta (radii from the first
// descriptor: the members of a diagram group share them), then the diagram,
// or (G) the task's T->ndiag group members summed.
// REG: the regularised components go to wr[0..nreg) (Jacobian and 1/n
// included).
template <int ORDER, int Q, bool HF, bool G, bool X, int V, bool REG = false, int HE = 0,
          bool SCR = false, bool TD = false, bool AZ = true>
__device__ __forceinline__ double eval_fp64(const KArgs &a, const TaskDev *__restrict__ T,
                                            const DiagDev *__restrict__ D,
                                            const SampleLds &Ls, double jc, uint64_t s,
                                            uint32_t iter, int *bins, uint32_t &npass,
                                            uint32_t &nterms, double *wr = nullptr) {
  constexpr int L = ORDER + 1;
  double k[L][3], r2[L];
  const double scale = loop_momenta<ORDER, AZ>(a, T, Ls, jc, s, iter, bins, k, r2);
  if constexpr (REG)
    for (int r = 0; r < kMaxReg; ++r) wr[r] = 0.0;
  double sum;
  if constexpr (G) {
    sum = 0.0;
    const int nd = T->ndiag;
    for (int di = 0; di < nd; ++di) {
      // the members' loop coefficients from their descriptors
      constexpr bool TDG = !FixedMasks<ORDER, V>::kFixed;
      if constexpr (group_cycle_form<ORDER, Q, X, HF>()) {
        SampleLds Lm = Ls;  // the member's cycle table
        Lm.cyc = static_cast<const char *>(Ls.cyc) + di * cycle_table_bytes<ORDER>();
        sum += diag_weight64<ORDER, Q, HF, REG, X, V, HE, kCycles, false, TDG>(
            a, T, D + di, Lm, k, r2, npass, nterms, wr);
      } else {
        sum += diag_weight64<ORDER, Q, HF, REG, X, V, HE, kConfigs, false, TDG>(
            a, T, D + di, Ls, k, r2, npass, nterms, wr);
      }
    }
  } else {
    constexpr LabelForm LF = label_form<ORDER, Q, false, X, HF>();
    sum = diag_weight64<ORDER, Q, HF, REG, X, V, HE, LF, SCR, TD>(a, T, D, Ls, k, r2, npass,
                                                                    nterms, wr);
    if constexpr (SCR) return sum;
  }
  if constexpr (REG)
    for (int r = 0; r < kMaxReg; ++r) wr[r] *= scale;
  return scale * sum;
}

// Largest product of a diagram's denominators that stays in fp32, its NC energy
// denominators without hbar^2 / 2m: 1e30 in MeV with nucleons' 20.75 MeV fm^2.
// Far below the range of a float, and not for its sake alone: beyond it the
// momenta are large, and the energy denominators of ring diagrams, differences
// of their squares, lose digits (third-order ring, cutoff 150 fm^-1: error 2.2e-6
// of W_cond rms, 5.3e-6 with 1e30 fm^-2NC).
template <int NC>
constexpr float fp32_den_max() {
  double m = 1e30;
  for (int c = 0; c < NC; ++c) m /= 20.75;
  return static_cast<float>(m);
}

// Per-sample integrand with fp32 arithmetic after the (fp64) VEGAS map; the
// Jacobian and the final weight stay fp64.  Sets `fallback` instead of
// returning a value when the sample lies in the band where fp32 cannot
// resolve the result to the target accuracy: a line within band_k kF^2 of a
// Fermi surface (the Pauli factor could flip), an energy denominator below
// band_d times the sum of its energies (cancellation), or a regulator exponent
// or reciprocal product outside the fp32 range.  The caller then evaluates the
// sample in fp64 from the same random words.
// fp32 contribution of one diagram at the loop momenta k (see
// diag_weight64); sets `fallback` instead when the sample needs fp64.
template <int ORDER, int Q, bool X, int V, int HE, LabelForm LF, bool SCR = false,
          bool TD = false>
__device__ __forceinline__ double diag_weight32(const KArgs &a, const TaskDev *__restrict__ T,
                                                const DiagDev *__restrict__ D,
                                                const SampleLds &Ls, const float (*k)[3],
                                                const float *r2, uint32_t &npass, uint32_t &nterms,
                                                bool &fallback) {
  constexpr int L = ORDER + 1;
  constexpr int NL = 2 * ORDER;
  constexpr int NC = ORDER - 1;
  const float kFn2 = static_cast<float>(T->kF2[0]), kFp2 = static_cast<float>(T->kF2[1]);
  const float bandk = static_cast<float>(T->band_k), bandd = static_cast<float>(T->band_d);
  float eps[NL];
  uint32_t inN = 0, inP = 0;
  float nearN = 3e38f, nearP = 3e38f;  // smallest distance to a Fermi surface
#pragma unroll
  for (int l = NL - 1; l >= 0; --l) {
    float kv[3];
    if (l < L) {
      kv[0] = k[l][0];
      kv[1] = k[l][1];
      kv[2] = k[l][2];
    } else {
      if constexpr (TD) table_sum<L, float>(D->coef_f[l], k, kv);
      else masked_sum<L, FixedMasks<ORDER, V>::kFixed, float>(lmask_of<ORDER, V>(D, l), k, kv);
    }
    // the Pauli tests take a loop line's squared radius; the energies take the
    // components, as the other lines do, so that the denominators' small
    // differences see one and the same set of momenta
    const float kk = kv[0] * kv[0] + kv[1] * kv[1] + kv[2] * kv[2];
    const float k2 = l < L ? r2[l < L ? l : 0] : kk;
    eps[l] = kk;  // in units of hbar^2 / 2m (energy_unit)
    const float tN = k2 - kFn2;
    nearN = fminf(nearN, fabsf(tN));
    inN = push_sign(inN, tN);
    if (Q == 4) {
      const float tP = k2 - kFp2;
      nearP = fminf(nearP, fabsf(tP));
      inP = push_sign(inP, tP);
    }
  }
  bool near = nearN < bandk * kFn2 || (Q == 4 && nearP < bandk * kFp2);
  if (near) {
    if constexpr (SCR) return 1.0;  // the Pauli screen (see screen_on)
    fallback = true;
    return 0.0;
  }
  const uint32_t lmask = line_mask_of<ORDER, V>(D), pmask = part_mask_of<ORDER, V>(D);
  const uint32_t okN = (inN ^ pmask) & lmask;
  const uint32_t okP = (inP ^ pmask) & lmask;
  LabelState<ORDER, V, LF> ls;
  if (!label_state<ORDER, Q, V, LF>(a, D, Ls, okN, okP, ls)) return 0.0;
  if constexpr (SCR) return 1.0;

  const bool rel = T->rel_target > 0.0;  // uniform
  float dprod = 1.0f;
  float kcut = 0.0f;  // (rel) sum of the cuts' condition numbers (sum |eps|) / |D|
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const uint32_t hm = cut_hole_of<ORDER, V>(D, c), pm = cut_part_of<ORDER, V>(D, c);
    float Dc = 0.0f, Dabs = 0.0f;
#pragma unroll
    for (int l = 0; l < NL; ++l) {
      if constexpr (FixedMasks<ORDER, V>::kFixed) {
        if (hm & (1u << l)) Dc += eps[l];
        else if (pm & (1u << l)) Dc -= eps[l];
        if ((hm | pm) & (1u << l)) Dabs += eps[l];
      } else {
        uint32_t bits = (hm & (1u << l)) ? 0x3F800000u : 0u;
        bits = (pm & (1u << l)) ? 0xBF800000u : bits;
        const float cf = __uint_as_float(bits);
        Dc = fmaf(cf, eps[l], Dc);
        Dabs = fmaf(fabsf(cf), eps[l], Dabs);
      }
    }
    near |= fabsf(Dc) < bandd * Dabs;
    if (rel) kcut = fmaf(Dabs, __builtin_amdgcn_rcpf(fabsf(Dc)), kcut);
    dprod *= Dc;
  }

  const float V0 = static_cast<float>(a.phys.V0 / a.phys.vscale);
  const float Vy = static_cast<float>(a.phys.Vy / a.phys.vscale);
  float Vd[ORDER], Ve[ORDER], den, yreg, ky = 0.0f;
  vertex_terms<ORDER, V, HE, TD, LF != kConfigs, true, float>(a, D, k, V0, Vy, Vd, Ve, den, yreg,
                                                              rel, &ky);
  // regulator exponent in powers of two, yreg times a constant in two parts:
  // one float's rounding of it alone moved every weight the same way (1.3e-7
  // on average at exponents up to 20)
  const double ylog2 = a.phys.invLn * a.phys.quarter_n * 1.4426950408889634;
  const float yhi = static_cast<float>(ylog2), ylo = static_cast<float>(ylog2 - yhi);
  const float y2 = yreg * yhi;
  const float yres = fmaf(yreg, ylo, fmaf(yreg, yhi, -y2));
  const float dall = den * dprod;
  // (y2 is NaN where p^n overflows a float and Lambda^-n underflows one)
  near |= !(fabsf(dall) > 1e-30f && fabsf(dall) < fp32_den_max<NC>() && den < 1e30f) ||
          !(y2 <= 115.0f);
  if (near) {
    fallback = true;
    return 0.0;
  }
  float inv = __builtin_amdgcn_rcpf(dall);
  inv = fmaf(inv, fmaf(-dall, inv, 1.0f), inv);  // one Newton step
  const float rexp = __builtin_amdgcn_exp2f(-y2);
  const float regall = fmaf(rexp, -0.693147181f * yres, rexp);

  float acc;
  const uint32_t nterms0 = nterms;
  if (rel) {
    // relative-accuracy target per value: a first-order bound on the fp32
    // evaluation's relative error, in units of the fp32 rounding unit u:
    // eight times the regulator exponent (its momenta carry a few u each), the cuts'
    // and the Yukawa denominators' condition numbers, the label sum's
    // cancellation (sum of |terms| / |sum|) and a constant for the rest
    float aabs;
    if constexpr (LF != kConfigs) {
      ++nterms;
      if constexpr (LF == kCounts)
        acc = label_sum_counts<ORDER, float, true>(ls.c, Vd, Ve, &aabs);
      else
        acc = label_sum_cycles<ORDER, float, true, V>(D, Vd, Ve, ls.cA, ls.cB, &aabs);
    } else {
      acc = label_sum<ORDER, Q, float, false, X, V, true>(a, D, Vd, Ve, okN, okP, lmask, nterms,
                                                          nullptr, nullptr, &aabs);
    }
    const float cancel = aabs * __builtin_amdgcn_rcpf(fabsf(acc));
    if (!(fabsf(acc) < 3e38f)) {  // out of the fp32 range
      nterms = nterms0;
      fallback = true;
      return 0.0;
    }
    const float bound =
        0x1p-24f * (5.5451774f * y2 + 4.0f * kcut + 4.0f * ky + 8.0f * cancel + 64.0f);
    if (!(bound <= static_cast<float>(T->rel_target))) {
      nterms = nterms0;
      fallback = true;
      return 0.0;
    }
  } else {
    if constexpr (LF != kConfigs) {
      ++nterms;
      if constexpr (LF == kCounts) acc = label_sum_counts<ORDER, float>(ls.c, Vd, Ve);
      else acc = label_sum_cycles<ORDER, float, false, V>(D, Vd, Ve, ls.cA, ls.cB);
    } else {
      acc = label_sum<ORDER, Q, float, false, X, V>(a, D, Vd, Ve, okN, okP, lmask, nterms,
                                                   nullptr, nullptr);
    }
    if (!(fabsf(acc) < 3e38f)) {  // out of the fp32 range
      nterms = nterms0;
      fallback = true;
      return 0.0;
    }
  }
  ++npass;
  double unit = energy_unit<NC>(a);  // times vscale^n (uniform)
#pragma unroll
  for (int v = 0; v < ORDER; ++v) unit *= a.phys.vscale;
  return (D->pref * unit) * static_cast<double>(regall) * static_cast<double>(acc) *
         static_cast<double>(inv);
}

template <int ORDER, int Q, bool G, bool X, int V, int HE = 0, bool SCR = false, bool TD = false>
__device__ __forceinline__ double eval_fp32(const KArgs &a, const TaskDev *__restrict__ T,
                                            const DiagDev *__restrict__ D,
                                            const SampleLds &Ls, double jc, uint64_t s,
                                            uint32_t iter, int *bins, uint32_t &npass,
                                            uint32_t &nterms, bool &fallback) {
  constexpr int L = ORDER + 1;
  float k[L][3], r2[L];
  const double scale = loop_momenta<ORDER, false>(a, T, Ls, jc, s, iter, bins, k, r2);
  double sum;
  if constexpr (G) {
    sum = 0.0;
    const int nd = T->ndiag;
    // members' counts are kept aside until every member has passed: a sample
    // that falls back is counted once, by its fp64 re-evaluation
    uint32_t gpass = 0, gterms = 0;
    for (int di = 0; di < nd; ++di) {
      constexpr bool TDG = !FixedMasks<ORDER, V>::kFixed;
      if constexpr (group_cycle_form<ORDER, Q, X, false>()) {
        SampleLds Lm = Ls;  // the member's cycle table
        Lm.cyc = static_cast<const char *>(Ls.cyc) + di * cycle_table_bytes<ORDER>();
        sum += diag_weight32<ORDER, Q, X, V, HE, kCycles, false, TDG>(a, T, D + di, Lm, k, r2,
                                                                      gpass, gterms, fallback);
      } else {
        sum += diag_weight32<ORDER, Q, X, V, HE, kConfigs, false, TDG>(a, T, D + di, Ls, k, r2,
                                                                       gpass, gterms, fallback);
      }
      if (fallback) return 0.0;  // the whole sample is re-evaluated in fp64
    }
    npass += gpass;
    nterms += gterms;
  } else {
    constexpr LabelForm LF = label_form<ORDER, Q, false, X, false>();
    sum = diag_weight32<ORDER, Q, X, V, HE, LF, SCR, TD>(a, T, D, Ls, k, r2, npass, nterms,
                                                         fallback);
    if constexpr (SCR) return sum;
    if (fallback) return 0.0;
  }
  return scale * sum;
}

// Kernel mode P: 0 fp64; 1 fp32 with the fp64 fallback; 2 fp64 with the
// Hartree-Fock spectrum (the fp32 integrand has the free spectrum only);
// 3 and 4: modes 0 and 1 for diagram groups (tasks of several descriptors);
// 5 and 6: fp64 with the regularised components, single diagrams / groups.
template <int P>
constexpr int prec_of() {
  return (P == 1 || P == 4) ? 1 : (P == 2 ? 2 : 0);
}
template <int P>
constexpr bool group_of() {
  return P == 3 || P == 4 || P == 6;
}
template <int P>
constexpr bool reg_of() {
  return P >= 5;
}
// Azimuths as steps of the turn table (see grid_pair): the fp64 kernels.
template <int P>
constexpr bool az_steps() {
  return prec_of<P>() != 1;
}
template <int ORDER, int Q, int P, bool X, int HE>
__device__ __forceinline__ double eval_sample(const KArgs &a, const TaskDev *__restrict__ T,
                                              const DiagDev *__restrict__ D,
                                              const SampleLds &Ls, uint64_t s,
                                              uint32_t iter, int *bins, uint32_t &npass,
                                              uint32_t &nterms, uint32_t &nfb) {
  constexpr int PP = prec_of<P>();
  constexpr bool G = group_of<P>();
  double w = 0.0;
  with_variant<ORDER, G, cycle_form<ORDER, Q, G, X, PP == 2>()>(D, [&](auto vt) {
    constexpr int V = decltype(vt)::value;
    constexpr bool AZ = az_steps<P>();
    const double jc = jac_const<ORDER, AZ>(a, T);
    if (PP != 1) {
      w = eval_fp64<ORDER, Q, PP == 2, G, X, V, false, HE, false, false, AZ>(
          a, T, D, Ls, jc, s, iter, bins, npass, nterms);
      return;
    }
    bool fb = false;
    w = eval_fp32<ORDER, Q, G, X, V, HE>(a, T, D, Ls, jc, s, iter, bins, npass, nterms, fb);
    if (fb) {
      ++nfb;
      w = eval_fp64<ORDER, Q, false, G, X, V, false, HE, false, false, AZ>(
          a, T, D, Ls, jc, s, iter, bins, npass, nterms);
    }
  });
  return w;
}

// Pauli screen of the sample loops in mode P: every sample first runs the
// integrand up to its Pauli test (the map, the momenta, the occupations and,
// in nuclear matter, the label cycles left open); a sample that fails adds
// its zero at once, and the others are queued per wavefront and evaluated 64
// at a time, from their random words again.  Most samples are Pauli-blocked,
// so whole wavefronts then run the denominators, interactions and label sum
// instead of wavefronts with most lanes idle.  The queued evaluation repeats
// the screen's arithmetic, so both take the same Pauli decision; a sample the
// fp32 screen finds within the fp64 band is queued, and its evaluation then
// falls back.  Fifth-order single diagrams (the free spectrum, the factorised
// label sums), where the work after the Pauli test dominates: measured on
// MI355X, nuclear matter fp32 and fp64 +25% (fp64 persistent +80%), neutron
// matter fp32 +18% and fp64 +8% (fp64 persistent -10%).  At fourth order it
// was slower (one diagram a launch -13%, persistent -10 to -17%).
template <int ORDER, int Q, int P, bool X>
constexpr bool screen_on() {
  return ORDER >= 5 && (P == 0 || P == 1) && !X;
}

// Words of a wavefront's LDS: the fp64 re-evaluation queue (fp32 kernels) and the
// Pauli screen's, 128 sample offsets each; the component sums of the regularised
// kernels, which have neither.
template <int ORDER, int Q, int P, bool X>
constexpr int wave_words() {
  return (prec_of<P>() == 1 ? 128 : 0) + (screen_on<ORDER, Q, P, X>() ? 128 : 0) +
         (reg_of<P>() ? 2 * kRegSums : 0);
}

// Appends the lanes with `flag` set to a wavefront's queue in LDS (ballot
// order, so the order is deterministic); n is wave-uniform.
__device__ __forceinline__ void wave_queue_push(uint32_t *q, int &n, bool flag, uint32_t v) {
  const uint64_t mask = __ballot(flag);
  if (flag) {
    const uint32_t below = __builtin_amdgcn_mbcnt_hi(
        static_cast<uint32_t>(mask >> 32), __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(mask), 0u));
    q[n + static_cast<int>(below)] = v;
  }
  n += __popcll(mask);
  __builtin_amdgcn_wave_barrier();
}

// Drops the first `take` entries of a wavefront's queue (take <= 64, at most
// 64 entries left behind them).
__device__ __forceinline__ void wave_queue_pop(uint32_t *q, int &n, int take, int lane) {
  __builtin_amdgcn_wave_barrier();
  const int rest = n - take;
  const uint32_t moved = (lane < rest) ? q[take + lane] : 0u;
  __builtin_amdgcn_wave_barrier();
  if (lane < rest) q[lane] = moved;
  __builtin_amdgcn_wave_barrier();
  n = rest;
}

// Bytes of the label tables a sample or dump kernel of mode P holds in LDS.
template <int ORDER, int Q, int P, bool X>
constexpr size_t label_lds_bytes() {
  constexpr LabelForm LF = label_form<ORDER, Q, group_of<P>(), X, prec_of<P>() == 2>();
  if (LF == kCounts) return count_table_bytes<ORDER>();
  if (LF == kCycles) return (group_of<P>() ? kGroupCycleTables : 1) * cycle_table_bytes<ORDER>();
  return 0;
}

// Builds the label table(s) of task T's diagram (one) or of its group's
// members (one per member, consecutive) at tab; the whole block takes part.
template <int ORDER, int Q, int P, bool X>
__device__ __forceinline__ void build_task_labels(const DiagDev *__restrict__ D,
                                                  const TaskDev *__restrict__ T, void *tab) {
  constexpr LabelForm LF = label_form<ORDER, Q, group_of<P>(), X, prec_of<P>() == 2>();
  if constexpr (LF == kCounts) {
    build_count_table<ORDER>(D, static_cast<LabelCounts<ORDER> *>(tab));
  } else if constexpr (LF == kCycles && group_of<P>()) {
    for (int di = 0; di < T->ndiag; ++di)
      build_cycle_table<ORDER>(D + di, static_cast<char *>(tab) + di * cycle_table_bytes<ORDER>());
  } else if constexpr (LF == kCycles) {
    build_cycle_table<ORDER>(D, tab);
  }
}

// HF spline tables held in LDS in mode P
template <int Q, int P>
constexpr int lds_tables() {
  return prec_of<P>() == 2 ? (Q == 4 ? 2 : 1) : 0;
}

// ---------------------------------------------------------------------------
// Work item: blockDim.x * spt consecutive samples of one task (HE: the
// regulator exponent's half fixed at compile time, or 0, see reg_pow)

// LDS of a sample block: turn and 2^(j/64) tables, HF tables, grid (e, width)
// pairs, histogram, reduction scratch, the wavefronts' queues (wave_words), label
// table(s).
struct BlockLds {
  SampleLds Ls;
  double2 *g;
  double *h;
  double *red;
};

// Carves the block's LDS and loads the task-independent tables.
template <int ORDER, int Q, int P, bool X>
__device__ __forceinline__ void block_lds(const KArgs &a, double *smem, BlockLds &B) {
  constexpr int ND = 3 * (ORDER + 1);
  constexpr int ntab = lds_tables<Q, P>();
  SinCos *turn = reinterpret_cast<SinCos *>(smem);
  double *ex = reinterpret_cast<double *>(turn + kTurnEntries);
  double *hf = ex + kExp2Entries;
  B.g = reinterpret_cast<double2 *>(hf + hf_lds_doubles(ntab));
  B.h = reinterpret_cast<double *>(B.g + ND * a.phys.nb);
  B.red = B.h + ND * a.phys.nb;
  const int nw = blockDim.x >> 6;
  B.Ls.turn = turn;
  B.Ls.ex = ex;
  B.Ls.hf = ntab ? hf : nullptr;
  B.Ls.g = B.g;
  size_t end = reinterpret_cast<char *>(B.red + 6 * nw) - reinterpret_cast<char *>(smem);
  end = (end + wave_words<ORDER, Q, P, X>() * nw * sizeof(uint32_t) + 15) & ~size_t{15};
  B.Ls.cyc = reinterpret_cast<char *>(smem) + end;
  load_turn_table(turn, ex);
}

// Loads task t's tables into the block's LDS: HF spline entries, grid pairs
// (grid_pair), a zeroed histogram and the label table(s) of
// its diagram(s).  The caller synchronises before and after.
template <int ORDER, int Q, int P, bool X>
__device__ __forceinline__ void task_lds(const KArgs &a, int t, BlockLds &B) {
  constexpr int ND = 3 * (ORDER + 1);
  constexpr int ntab = lds_tables<Q, P>();
  const TaskDev *__restrict__ T = a.tasks + t;
  const int nb = a.phys.nb;
  const int tid = threadIdx.x, bs = blockDim.x;
  if constexpr (ntab > 0)
    load_hf<ntab>(const_cast<double *>(B.Ls.hf), a.hf + 4 * static_cast<size_t>(T->hf_off));
  const double *ge = a.grids + T->grid_off;
  const DiagDev *__restrict__ D = a.diags + T->diag;
  for (int i = tid; i < ND * nb; i += bs) {
    const int m = i / nb, b = i - m * nb;
    const double e0 = ge[m * (nb + 1) + b], e1 = ge[m * (nb + 1) + b + 1];
    B.g[i] = grid_pair<az_steps<P>()>(m, e0, e1, loop_radius(T, D, m / 3));
    B.h[i] = 0.0;
  }
  build_task_labels<ORDER, Q, P, X>(D, T, const_cast<void *>(B.Ls.cyc));
}

// True if the iteration's histogram refines the grid afterwards; with a training
// phase the grid is frozen once the training iterations are done, and neither
// the samples nor the items touch the histograms (15 LDS atomics per sample and
// 750 memory-side ones per item at fourth order).  On trained grids, MI355X: 585
// fourth-order tasks x 2^21 fp32 18.9 -> 16.9 ms per iteration, orders 2+3, 36
// tasks x 2^24 fp32 6.62 -> 5.56 ms, one fourth-order task of 2^18 samples 33 ->
// 26 us.
__device__ __forceinline__ bool adapts(const TaskDev *__restrict__ T) {
  return T->train_iters <= 0 || T->it_done < T->train_iters;
}

// Adds the block's LDS histogram of task t to the task's histogram.
template <int ORDER>
__device__ __forceinline__ void hist_flush(const KArgs &a, int t, const double *h) {
  constexpr int ND = 3 * (ORDER + 1);
  if (!adapts(a.tasks + t)) return;
  double *hg = a.hists + a.tasks[t].hist_off;
  for (int i = threadIdx.x; i < ND * a.phys.nb; i += blockDim.x) {
    const double v = h[i];
    if (v != 0.0) atomicAdd(&hg[i], v);
  }
}

// The samples of one work item of task t (the task's tables in LDS): sums,
// histogram entries (LDS), and the item's partial sums and counters.
// FX4: the code of each fourth-order diagram (see fixed4).
template <int ORDER, int Q, int P, bool X, int HE, bool FX4 = false>
__device__ __forceinline__ void item_samples(const KArgs &a, int t, int item, const BlockLds &B) {
  constexpr int ND = 3 * (ORDER + 1);
  const TaskDev *__restrict__ T = a.tasks + t;
  const DiagDev *__restrict__ D = a.diags + T->diag;
  const int nb = a.phys.nb;
  const int tid = threadIdx.x, bs = blockDim.x;
  const SampleLds &Ls = B.Ls;
  double *h = B.h;
  double *red = B.red;

  const uint64_t N = T->nsamples;
  const uint32_t iter = T->iter;
  const int spt = T->spt;
  const double shift = T->shift;
  const bool hist = adapts(T);
  const uint64_t base = static_cast<uint64_t>(item - T->item_begin) * bs * spt;
  double s1 = 0.0, c1 = 0.0, s2 = 0.0, c2 = 0.0;
  uint32_t npass = 0, nterms = 0, nfb = 0;
  // regularised components: sum (w_k - shift) and sum (w_k - shift)^2 with
  // the main component's shift (a thread adds at most spt terms: plain sums)
  constexpr bool R = reg_of<P>();
  double rs[R ? kRegSums : 1];
#pragma unroll
  for (int j = 0; j < (R ? kRegSums : 1); ++j) rs[j] = 0.0;
  // a thread adds at most spt terms of the shifted sums: plain sums; the
  // merges across threads and items keep the rounding errors
  auto accumulate = [&](double w, const int *bins) {
    const double d = w - shift;
    s1 += d;
    s2 = fma(d, d, s2);
    if (hist) {
      const double w2 = w * w;
      if (w2 != 0.0) {
#pragma unroll
        for (int m = 0; m < ND; ++m) atomicAdd(&h[m * nb + bins[m]], w2);
      }
    }
  };
  // a sample that fails the Pauli screen: weight zero
  auto accumulate_zero = [&]() {
    const double d = -shift;
    s1 += d;
    s2 = fma(d, d, s2);
  };
  constexpr int PP = prec_of<P>();
  constexpr bool G = group_of<P>();
  constexpr bool SCR = screen_on<ORDER, Q, P, X>();
  const int lane = tid & 63;
  // per wavefront: the fp64 re-evaluation queue, then the Pauli screen's
  uint32_t *queue = reinterpret_cast<uint32_t *>(red + 6 * (bs >> 6)) +
                    wave_words<ORDER, Q, P, X>() * (tid >> 6);
  uint32_t *pqueue = queue + (PP == 1 ? 128 : 0);
  // the sample loops, specialised per diagram variant (uniform per item)
  auto loops = [&](auto vt) {
    constexpr int V = decltype(vt)::value;
    // the loop coefficients decoded in the descriptor (desc_coef)
    constexpr bool TD = desc_coef<ORDER, P>() && !FixedMasks<ORDER, V>::kFixed;
    constexpr bool AZ = az_steps<P>();
    const double jc = jac_const<ORDER, AZ>(a, T);
    if constexpr (SCR && PP == 0) {
      int pn = 0;  // wave-uniform
      auto drain_pass = [&](int take) {
        if (lane < take) {
          const uint64_t s = base + pqueue[lane];
          int bins[ND];
          const double w = eval_fp64<ORDER, Q, false, G, X, V, false, HE, false, TD, AZ>(
              a, T, D, Ls, jc, s, iter, bins, npass, nterms);
          accumulate(w, bins);
        }
        wave_queue_pop(pqueue, pn, take, lane);
      };
      for (int kk = 0; kk < spt; ++kk) {
        const uint64_t s = base + static_cast<uint64_t>(kk) * bs + tid;
        bool go = false;
        if (s < N) {
          int bins[ND];
          go = eval_fp64<ORDER, Q, false, G, X, V, false, HE, true, TD, AZ>(
                   a, T, D, Ls, jc, s, iter, bins, npass, nterms) != 0.0;
          if (!go) accumulate_zero();
        }
        wave_queue_push(pqueue, pn, go, static_cast<uint32_t>(s - base));
        if (pn >= 64) drain_pass(64);
      }
      while (pn > 0) drain_pass(pn < 64 ? pn : 64);
    } else if constexpr (PP != 1) {
      for (int kk = 0; kk < spt; ++kk) {
        const uint64_t s = base + static_cast<uint64_t>(kk) * bs + tid;
        if (s < N) {
          int bins[ND];
          if constexpr (R) {
            double wr[kMaxReg];
            const double w = eval_fp64<ORDER, Q, false, G, X, V, true, HE, false, TD, AZ>(
                a, T, D, Ls, jc, s, iter, bins, npass, nterms, wr);
            accumulate(w, bins);
            // the extrapolation's weights sum to one, so its shifted value
            // is the weighted sum of the components' shifted values
            double dx = 0.0;
#pragma unroll
            for (int r = 0; r < kMaxReg; ++r) {
              const double d = wr[r] - shift;
              rs[2 * r] += d;
              rs[2 * r + 1] += d * d;
              dx = fma(a.reg_coef[r], d, dx);
            }
            rs[2 * kMaxReg] += dx;
            rs[2 * kMaxReg + 1] += dx * dx;
          } else {
            const double w = eval_fp64<ORDER, Q, PP == 2, G, X, V, false, HE, false, TD, AZ>(
                a, T, D, Ls, jc, s, iter, bins, npass, nterms);
            accumulate(w, bins);
          }
        }
      }
    } else {
      // fp32 pass; samples in the fp64 band are queued per wavefront (ballot
      // order, so the accumulation order is deterministic) and re-evaluated in
      // fp64 by whole wavefronts, 64 at a time
      int qn = 0;  // wave-uniform
      auto drain = [&](int take) {
        if (lane < take) {
          const uint64_t s = base + queue[lane];
          int bins[ND];
          const double w = eval_fp64<ORDER, Q, false, G, X, V, false, HE, false, TD, AZ>(
              a, T, D, Ls, jc, s, iter, bins, npass, nterms);
          accumulate(w, bins);
        }
        __builtin_amdgcn_wave_barrier();
        const int rest = qn - take;
        uint32_t moved = (lane < rest) ? queue[take + lane] : 0u;
        __builtin_amdgcn_wave_barrier();
        if (lane < rest) queue[lane] = moved;
        __builtin_amdgcn_wave_barrier();
        qn = rest;
      };
      if constexpr (SCR) {
        int pn = 0;  // wave-uniform
        auto drain_pass = [&](int take) {
          bool fb = false;
          uint32_t off = 0u;
          if (lane < take) {
            off = pqueue[lane];
            int bins[ND];
            const double w = eval_fp32<ORDER, Q, G, X, V, HE, false, TD>(
                a, T, D, Ls, jc, base + off, iter, bins, npass, nterms, fb);
            if (!fb) accumulate(w, bins);
          }
          if (fb) ++nfb;
          wave_queue_push(queue, qn, fb, off);
          wave_queue_pop(pqueue, pn, take, lane);
          if (qn >= 64) drain(64);
        };
        for (int kk = 0; kk < spt; ++kk) {
          const uint64_t s = base + static_cast<uint64_t>(kk) * bs + tid;
          bool go = false;
          if (s < N) {
            int bins[ND];
            bool unused = false;
            go = eval_fp32<ORDER, Q, G, X, V, HE, true, TD>(a, T, D, Ls, jc, s, iter, bins,
                                                                 npass, nterms, unused) != 0.0;
            if (!go) accumulate_zero();
          }
          wave_queue_push(pqueue, pn, go, static_cast<uint32_t>(s - base));
          if (pn >= 64) drain_pass(64);
        }
        while (pn > 0) drain_pass(pn < 64 ? pn : 64);
      } else {
        for (int kk = 0; kk < spt; ++kk) {
          const uint64_t s = base + static_cast<uint64_t>(kk) * bs + tid;
          bool fb = false;
          if (s < N) {
            int bins[ND];
            const double w = eval_fp32<ORDER, Q, G, X, V, HE, false, TD>(
                a, T, D, Ls, jc, s, iter, bins, npass, nterms, fb);
            if (!fb) accumulate(w, bins);
          }
          const uint64_t mask = __ballot(fb);
          if (fb) {
            const int pos = qn + __builtin_amdgcn_mbcnt_hi(
                                     static_cast<uint32_t>(mask >> 32),
                                     __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(mask), 0u));
            queue[pos] = static_cast<uint32_t>(s - base);
            ++nfb;
          }
          qn += __popcll(mask);
          __builtin_amdgcn_wave_barrier();
          if (qn >= 64) drain(64);
        }
      }
      while (qn > 0) drain(qn < 64 ? qn : 64);
    }
  };
  with_variant<ORDER, G, cycle_form<ORDER, Q, G, X, PP == 2>(), FX4>(D, loops);
  // wavefront butterfly, then waves in order (compensated pairs s + c)
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    const double os1 = __shfl_xor(s1, off, 64), oc1 = __shfl_xor(c1, off, 64);
    const double os2 = __shfl_xor(s2, off, 64), oc2 = __shfl_xor(c2, off, 64);
    pair_merge(s1, c1, os1, oc1);
    pair_merge(s2, c2, os2, oc2);
    npass += __shfl_xor(npass, off, 64);
    nterms += __shfl_xor(nterms, off, 64);
    nfb += __shfl_xor(nfb, off, 64);
    if constexpr (R) {
#pragma unroll
      for (int j = 0; j < kRegSums; ++j) rs[j] += __shfl_xor(rs[j], off, 64);
    }
  }
  const int wave = tid >> 6;
  uint32_t *ured = reinterpret_cast<uint32_t *>(red + 4 * (bs >> 6));
  double *rred = red + 6 * (bs >> 6);
  if constexpr (R) {
    if (lane == 0) {
#pragma unroll
      for (int j = 0; j < kRegSums; ++j) rred[kRegSums * wave + j] = rs[j];
    }
  }
  if (lane == 0) {
    red[4 * wave + 0] = s1;
    red[4 * wave + 1] = c1;
    red[4 * wave + 2] = s2;
    red[4 * wave + 3] = c2;
    ured[3 * wave] = npass;
    ured[3 * wave + 1] = nterms;
    ured[3 * wave + 2] = nfb;
  }
  __syncthreads();
  if (tid == 0) {
    double S1 = red[0], C1 = red[1], S2 = red[2], C2 = red[3];
    uint64_t P1 = ured[0], P2 = ured[1], P0 = ured[2];
    for (int w = 1; w < (bs >> 6); ++w) {
      pair_merge(S1, C1, red[4 * w + 0], red[4 * w + 1]);
      pair_merge(S2, C2, red[4 * w + 2], red[4 * w + 3]);
      P1 += ured[3 * w];
      P2 += ured[3 * w + 1];
      P0 += ured[3 * w + 2];
    }
    const size_t store = static_cast<size_t>(T->store_begin) + (item - T->item_begin);
    double *part = a.partials + 4 * store;
    part[0] = S1;
    part[1] = C1;
    part[2] = S2;
    part[3] = C2;
    uint64_t *K = a.counters + kItemCounters * store;
    K[0] = P0;
    K[1] = P1;
    K[2] = P2;
    if constexpr (R) {
      double *cp = a.cpart + kRegSums * store;
      for (int j = 0; j < kRegSums; ++j) {
        double v = rred[j];
        for (int w = 1; w < (bs >> 6); ++w) v += rred[kRegSums * w + j];
        cp[j] = v;
      }
    }
  }
}

// One work item with its own setup and histogram merge.
template <int ORDER, int Q, int P, bool X, int HE>
__device__ __forceinline__ void process_item(const KArgs &a, int t, int item, double *smem) {
  BlockLds B;
  block_lds<ORDER, Q, P, X>(a, smem, B);
  task_lds<ORDER, Q, P, X>(a, t, B);
  __syncthreads();
  item_samples<ORDER, Q, P, X, HE, fixed4<ORDER, Q, P, X, HE>()>(a, t, item, B);
  __syncthreads();
  hist_flush<ORDER>(a, t, B.h);
}

// Waves per SIMD the sample kernels ask the compiler for (it then holds them
// within 512 / waves VGPRs, spilling the rest), as measured on MI355X:
// - fourth order: fp64, fp32, group and regularised kernels run 4-30% faster
//   at 3 waves (100-200 spilled bytes per thread) than at 2 without spills;
// - fifth order: fp32, group and explicit-list kernels gain at 3 waves; the
//   fp64 polynomial kernel (about 360 spilled bytes at 3) and the regularised
//   single-diagram kernel are faster at their natural occupancy; the
//   regularised group kernel stays within 256 VGPRs at 2;
// - HF kernels (isospin-dependent spectra keep per-line energy differences
//   live): 2 waves from third order on, 20-45% faster than at one, except
//   fifth-order neutron matter, which loses a third to ~520 spilled bytes.
// - third order (single diagrams specialised per diagram), by time per iteration:
//   4 waves with spilled bytes beat 3 without at large sizes (twelve tasks x
//   2^21, at 4 / 3 waves: nuclear fp32 371 / 393 us, neutron fp32 355 / 369;
//   at 5 the fp32 batch of orders 2 and 3 loses 12%); neutron-matter fp64 is
//   the faster at 3 at every size (2^18 samples 27 / 26 us, 2^23 166 / 160,
//   twelve tasks x 2^21 425 / 417), nuclear fp64 only at small ones (2^20 45 /
//   43 us, twelve tasks x 2^21 442 / 453);
// - fourth-order nuclear single diagrams with compile-time masks (fixed4): 3
//   waves; those that read the descriptor (other regulator exponents):
//   fp32 at 4 waves beats 3 by 1-6%, fp64 runs 4% faster at 3 than at 4;
// - fourth-order nuclear group kernels, whose per-member label tables leave
//   LDS for 3 blocks per CU, run 3-5% faster at 3 waves than at 4 and 8-13%
//   faster than at 2; the regularised ones spill 304 bytes at 3 (14.2 ms
//   against 11.9 at 2 for the fourth-order groups at 2^18 samples);
// - fifth-order nuclear matter with the Pauli screen: fp32 at 3 waves beats 4
//   by 8% and 2 by 11%, fp64 at 3 beats 2 by 11% and 4 by 16%.
// Other kernels fit their natural occupancy.
template <int ORDER, int Q, int P, bool X, int HE>
constexpr int min_waves() {
  if (fixed4<ORDER, Q, P, X, HE>()) return 3;
  if (P == 2) {
    if (ORDER == 2) return 3;
    if (ORDER == 3 || ORDER == 4) return 2;
    return (ORDER == 5 && Q == 4) ? 2 : 1;
  }
  if (Q == 4 && !X && (P == 0 || P == 1)) {
    if (ORDER == 4) return P == 1 ? 4 : 3;
    if (ORDER == 5) return 3;
  }
  if (ORDER == 3 && (P == 0 || P == 1)) return Q == 2 && P == 0 ? 3 : 4;
  if (ORDER == 4) return (P == 0 || P == 1 || P == 3 || P == 4 || P == 5) ? 3 : 2;
  if (ORDER == 5) {
    if (P == 1 || P == 3 || P == 4 || (P == 0 && X)) return 3;
    return P == 6 ? 2 : 1;
  }
  return 1;
}

// Waves per SIMD of the persistent kernels: their item loop leaves more
// registers live than a one-item kernel, and at the one-item kernels'
// occupancy the nuclear-matter kernels of orders 4 and 5 spilled 180-600
// bytes per lane.  Measured on MI355X (every third fourth-order diagram and
// every 42nd fifth-order one at the 15 nuclear-matter points, 2^22 samples
// per task): fourth order fp32 23.6 Gevals/s at 3 waves against 20.3 at 4,
// fp64 21.5 at 2 against 11.9 at 4; fifth order fp32 13.0 at 2 against 3.9 at
// 4, fp64 7.4 at 2 against 5.6 at 3.
template <int ORDER, int Q, int P, bool X>
constexpr int persistent_waves() {
  if (Q == 4 && !X && (P == 0 || P == 1)) {
    if (ORDER == 4) return P == 1 ? 3 : 2;
    if (ORDER == 5) return 2;
  }
  return min_waves<ORDER, Q, P, X, 0>();
}

// One launch over work items, one block per item.  k1 > k0: the items of the
// tasks of one order; olist[k0, k1) lists them as (first item, task) with
// ascending first item, their items are numbered contiguously from olist[k0].x,
// and block b takes item olist[k0].x + b.  One launch per order keeps each
// launch's register allocation that of its own order.  k1 < 0: the items of
// task k0 alone.
template <int ORDER, int Q, int P, bool X, int HE>
__global__ __launch_bounds__(256, (min_waves<ORDER, Q, P, X, HE>())) void sample_order(
    KArgs a, int k0, int k1) {
  extern __shared__ double smem[];
  int t = k0, item;
  if (k1 < 0) {
    item = a.tasks[t].item_begin + static_cast<int>(blockIdx.x);
  } else {
    const int2 *__restrict__ ol = a.olist;
    item = ol[k0].x + static_cast<int>(blockIdx.x);
    int lo = k0, hi = k1 - 1;  // last entry with first item <= item
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (ol[mid].x <= item) lo = mid;
      else hi = mid - 1;
    }
    t = ol[lo].y;
  }
  process_item<ORDER, Q, P, X, HE>(a, t, item, smem);
}

// Persistent launch over the work items of the tasks of one order (as
// sample_order, nitems items from olist[k0].x on): a grid of about as many
// blocks as are resident on the device at once; each block claims chunks of
// `chunk` consecutive items from the order's counter a.queue[ORDER] until all
// are taken.  Claims ascend, so a block meets the tasks in ascending order:
// it keeps the current task's grid, histogram and label-cycle table in LDS
// across that task's items and merges the histogram into the task's once per
// run of items (instead of once per item).  The counter starts at zero (task
// set initialisation) and the iteration end zeroes it for the next iteration.
template <int ORDER, int Q, int P, bool X, int HE>
__global__ __launch_bounds__(256, (persistent_waves<ORDER, Q, P, X>())) void sample_persistent(
    KArgs a, int k0, int k1, int nitems, int chunk) {
  extern __shared__ double smem[];
  __shared__ int claim;
  const int2 *__restrict__ ol = a.olist;
  const int first = ol[k0].x;
  BlockLds B;
  block_lds<ORDER, Q, P, X>(a, smem, B);
  int cur = -1, lo = k0;
  for (;;) {
    __syncthreads();  // every thread has read the previous claim
    if (threadIdx.x == 0) claim = atomicAdd(a.queue + ORDER, chunk);
    __syncthreads();
    const int c0 = claim;
    if (c0 >= nitems) break;
    const int c1 = min(c0 + chunk, nitems);
    for (int k = c0; k < c1; ++k) {
      const int item = first + k;
      while (lo + 1 < k1 && ol[lo + 1].x <= item) ++lo;
      const int t = ol[lo].y;
      __syncthreads();  // the previous item's reduction scratch has been read
      if (t != cur) {
        if (cur >= 0) hist_flush<ORDER>(a, cur, B.h);
        __syncthreads();
        task_lds<ORDER, Q, P, X>(a, t, B);
        __syncthreads();
        cur = t;
      }
      // opaque to the optimiser: nothing of one item's evaluation is kept
      // live into the next (the body then has the registers of a one-item
      // kernel)
      int tt = t, ii = item;
      asm volatile("" : "+s"(tt), "+s"(ii));
      item_samples<ORDER, Q, P, X, HE>(a, tt, ii, B);
    }
  }
  __syncthreads();
  if (cur >= 0) hist_flush<ORDER>(a, cur, B.h);
}

// ---------------------------------------------------------------------------
// Per-sample dump for parity checks: thread i evaluates sample first + i.

// Regularised modes: out_reg (if not null) receives the components,
// out_reg[i * nreg + k] for component k + 1.
template <int ORDER, int Q, int P, bool X, int HE>
__global__ __launch_bounds__(256) void dump_samples(KArgs a, int t, uint32_t iter, uint64_t first,
                                                   uint64_t count, double *out, double *out_reg) {
  extern __shared__ double smem[];
  constexpr int ND = 3 * (ORDER + 1);
  const TaskDev *T = a.tasks + t;
  const DiagDev *D = a.diags + T->diag;
  const int nb = a.phys.nb;
  SampleLds Ls;
  double2 *g;
  carve_lds<lds_tables<Q, P>()>(a, T, ND, smem, Ls, g);
  const double *ge = a.grids + T->grid_off;
  for (int i = threadIdx.x; i < ND * nb; i += blockDim.x) {
    const int m = i / nb, b = i - m * nb;
    const double e0 = ge[m * (nb + 1) + b], e1 = ge[m * (nb + 1) + b + 1];
    g[i] = grid_pair<az_steps<P>()>(m, e0, e1, loop_radius(T, D, m / 3));
  }
  Ls.cyc = g + ND * nb;
  build_task_labels<ORDER, Q, P, X>(D, T, g + ND * nb);
  __syncthreads();
  const uint64_t i = static_cast<uint64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < count) {
    int bins[ND];
    uint32_t np = 0, nt = 0, nf = 0;
    if constexpr (reg_of<P>()) {
      double wr[kMaxReg];
      with_variant<ORDER, group_of<P>(), cycle_form<ORDER, Q, group_of<P>(), X, false>()>(
          D, [&](auto vt) {
        constexpr int V = decltype(vt)::value;
        out[i] = eval_fp64<ORDER, Q, false, group_of<P>(), X, V, true, HE>(
            a, T, D, Ls, jac_const<ORDER, true>(a, T), first + i, iter, bins, np, nt, wr);
      });
      if (out_reg)
        for (int r = 0; r < a.nreg; ++r) out_reg[i * a.nreg + r] = wr[r];
    } else {
      out[i] = eval_sample<ORDER, Q, P, X, HE>(a, T, D, Ls, first + i, iter, bins, np, nt, nf);
    }
  }
}

// Mode of a sample kernel from the precision, spectrum, regularisation and
// grouping (see prec_of, group_of, reg_of); -1 if no kernel exists: the HF
// spectrum runs the fp64 integrand (mode 2) whatever the precision, the
// regularised components the fp64 integrand (modes 5, 6) with the free
// spectrum.
__host__ inline int mode_of(const KArgs &a, int prec, bool group) {
  if (a.nreg > 0) return a.phys.spectrum ? -1 : 5 + (group ? 1 : 0);
  if (a.phys.spectrum) return group ? -1 : 2;  // HF groups are not built
  return (prec ? 1 : 0) + (group ? 3 : 0);
}

}  // namespace mbpt
