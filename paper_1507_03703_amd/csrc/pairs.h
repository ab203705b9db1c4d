// Intramolecular nonbonded and implicit-solvent terms of a ligand
// (pairs.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace bpmf {

constexpr int kPairMaxAtoms = 128;
constexpr int kPairWords = kPairMaxAtoms / 32;  // mask words per atom

// LDS bytes of a ligand's staged pair parameters and per-evaluation pair
// scratch (eval_block): p0 (16 n), p1 (8 n), the excluded and 1-4 masks
// (2 x 16 n), Born radii and their chain-rule factors (2 x 4 n), and 16
// bytes for the alignment of their start
// plus, for a block of `waves` wavefronts, the per-slice partial sums of
// the three passes (pair_stage): S = waves / ceil(n / 64) slices of the
// partner range, 9 floats per slice and atom
__host__ __device__ inline int pair_slices(int n, int waves) {
  const int a = (n + 63) / 64;
  return waves / a > 0 ? waves / a : 1;
}
__host__ __device__ inline int pair_lds_bytes(int n, int waves) {
  return 64 * n + 16 + 36 * n * pair_slices(n, waves);
}

// Partners whose chains of a pass run side by side (pair_stage).  A replica's
// wavefronts share one CU and issue for some three quarters of the time, so
// what overlaps chains must not add instructions: 48 atoms on 8 wavefronts
// have 6 partners a thread, and 20 sweeps of 20 steps take 3.21 ms with 3 at
// a time, 3.36 with 2 or with 4 (two idle of 8), 3.40 with 6, 4.31 with 8;
// one at a time through branches 3.63 ms (12 to 100 atoms on 1 to 8 wavefronts:
// 1 to 42 % faster so, least where 32 atoms on 8 leave two of six idle).
// Ligands whose threads have no more than 2 partners take 2 at a time, in sweep
// kernels of their own (chosen by a branch, the longer slices lose 2 %): 8
// atoms, 64 replicas, 20 sweeps of 20 steps on 4 and 8 wavefronts 2.05 and 1.82
// ms, 2.52 and 2.08 ms with 3, 2.37 and 1.88 ms one at a time through branches.
constexpr int kPairAhead = 3, kPairShort = 2;
inline int pair_at_once(int n, int waves) {
  return waves > 1 && n <= kPairShort * pair_slices(n, waves) ? kPairShort
                                                              : kPairAhead;
}

constexpr float kObcA = 1.0f, kObcB = 0.8f, kObcC = 4.85f;

// Descreening integral H(r; a, s) of a ball of radius s at distance r outside
// radius a (Hawkins, Cramer, Truhlar), and dH/dr, from r^2 and ir = 1/r; ra =
// rcp(a).  The reciprocals and the logarithm are the hardware's (1 ulp);
// du/u = -u and dl/l = -+l are used as such.  Without branches: every lane of
// a wavefront has pairs on either side of each condition, so branches would
// be walked both ways, and partners' chains would not overlap.  Roundings are
// placed by hand, so that a use's bits do not depend on what the compiler makes
// of the code around it.  OWN, for the uses in which s is the atom's own for all
// partners: s^2 is rounded and r^2 is not, elsewhere the other way round; a
// trajectory's decisions follow from these bits, so both uses keep theirs.
//
// The logarithm is for normal arguments (u x is at least a / (r + s)): log2, by
// the hardware, times ln 2 in two parts, the rounding error of the leading
// product recovered by a fused multiply-add (the exact product of Dekker, 1971).
// That is what __logf gives there, without its scaling of subnormal arguments
// and its care of infinities.
__device__ __forceinline__ float hct_log(float v) {
  constexpr float kLn2 = 0x1.62e42ep-1f, kLn2Low = 0x1.efa39ep-25f;
  const float y = __builtin_amdgcn_logf(v);  // log2
  return fmaf(y, kLn2, fmaf(y, kLn2Low, fmaf(y, kLn2, -(y * kLn2))));
}
template <bool DERIV, bool OWN>
__device__ __forceinline__ void hct(float r2, float ir, float a, float ra,
                                    float s, float& H, float& dH) {
#pragma clang fp contract(off)
  const float r = r2 * ir, rps = fmaf(r2, ir, s), rs = r - s;
  const float ars = fabsf(rs);
  const bool shell = a > ars;  // the shells start at a, not at |r - s|
  const float u = __builtin_amdgcn_rcpf(rps);
  const float l = shell ? ra : __builtin_amdgcn_rcpf(ars);
  const float lg = hct_log(u * (shell ? a : ars));
  const float s2r2 = OWN ? fmaf(-r, r, s * s) : fmaf(s, s, -(r * r));
  const float uu = u * u;
  const float l2u2 = fmaf(l, l, -uu);
  const bool none = a >= rps, inside = a < s - r;
  float h = ir * (0.125f * s2r2 * l2u2);
  h = fmaf(0.5f, l - u, h);
  h = fmaf(ir, 0.25f * lg, h);
  h = inside ? h + (ra - l) : h;
  H = none ? 0.f : h;
  if (DERIV) {
    const float dll = shell ? 0.f : (rs > 0.f ? -l : l);
    const float dl = l * dll;
    float d = fmaf(ir, ir * (-0.125f * s2r2), -0.25f) * l2u2;
    d = fmaf(0.5f, fmaf(u, u, dl), d);
    d = fmaf(ir, 0.25f * s2r2 * fmaf(dl, l, u * uu), d);
    d = fmaf(ir, 0.25f * (-u - dll), d);
    d = fmaf(ir, ir * (-0.25f * lg), d);
    d = inside ? d - dl : d;
    dH = none ? 0.f : d;
  }
}

struct PairDev {
  int n;
  const float4* p0;       // n: q, sigma, sqrt(eps), rho
  const float2* p1;       // n: rt = rho - 0.09, S * rt
  const uint32_t* excl;   // n x kPairWords: bit j of row i = pair excluded
  const uint32_t* o14;    // n x kPairWords: bit j of row i = 1-4 pair
  float lj14, el14;
  float kc;    // k_e / eps_solute
  float kgb;   // -k_e (1/eps_solute - 1/eps_solvent)
  float sa;    // 4 pi gamma
  float probe;
};

// terms: N x 4 doubles (LJ, Coulomb, GB, SA); forces: N x n x 3 or null
hipError_t launch_pair_terms(const PairDev& P, const float* x, int64_t N,
                             double* terms, float* forces, hipStream_t st);

}  // namespace bpmf
