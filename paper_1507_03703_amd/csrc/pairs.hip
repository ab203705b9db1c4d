// Intramolecular nonbonded and implicit-solvent energy and forces of the
// ligand (Thermodynamic Cycle: the ligand force field with an OBC
// generalised-Born/surface-area solvent).
//   LJ 12-6 and Coulomb over pairs more than two bonds apart (Lorentz-
//   Berthelot; 1-4 pairs scaled), generalised Born over all ordered pairs
//   with f = sqrt(r^2 + R_i R_j exp(-r^2 / 4 R_i R_j)), Born radii from the
//   Hawkins-Cramer-Truhlar descreening integral through the OBC II
//   rescaling (Onufriev, Bashford, Case 2004), and the ACE surface term
//   4 pi gamma (rho + probe)^2 (rho / R)^6.
// One thread per atom, as many configurations to a workgroup as fill it:
// each thread sums its own row of pair terms (every pair is visited from both
// ends), so the forces need no atomics and the result does not depend on
// scheduling.  Three passes: (1) LJ, Coulomb, the descreening sum I_i and its
// derivatives; (2) the Born radii known, the GB energy, its explicit force
// and dE/dR_i; (3) the chain rule through dR_i/dI_i and dI/dr.
#include <hip/hip_runtime.h>
#include <math.h>

#include "pairs.h"

namespace bpmf {

namespace {

constexpr int kPairThreads = 256;
// to this size the derivatives of pass 1 are kept for pass 3
constexpr int kPairKeepAtoms = 64;

// LDS: the parameters of the ligand (p0, p1, masks), then per configuration
// positions, Born radii and chain-rule factors, then the kept derivatives
// (keep: n rows of n | 1 floats) or the threads' energies (4 doubles), which
// share the space
__host__ __device__ inline int pair_words(int n) { return (n + 31) / 32; }
__host__ __device__ inline int pair_head_bytes(int n) {
  return (24 * n + 8 * n * pair_words(n) + 15) & ~15;
}
__host__ __device__ inline int pair_conf_bytes(int n) { return 24 * n; }
__host__ __device__ inline int pair_keep_bytes(int n) {
  return 4 * n * (n | 1);
}

// What bounds it: instruction issue, some 160 vector instructions a pair end
// with forces.  Configurations are packed because 48 atoms fill 48 of a
// wavefront's 64 lanes (5 of them 240 of a block's 256); the descreening
// derivatives dH(r_ij; a_i, s_j) / r_ij of pass 1 are what pass 3 needs of
// both ends of a pair, so they are summed there for the thread's own atom and
// kept (KEEP) in LDS for the partner: pass 3 is then a product a pair instead
// of both integrals anew.  Above 64 atoms the n^2 floats would leave too few
// wavefronts, and the partner's integral is worked out again.  32000
// configurations of 48 atoms with forces: 310 us, one configuration to a
// wavefront and both integrals twice 530 us.
template <bool FORCES, bool KEEP>
__global__ __launch_bounds__(kPairThreads) void k_pair_terms(
    PairDev P, const float* __restrict__ xs, int64_t N, int G,
    double* __restrict__ terms, float* __restrict__ forces) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int n = P.n, nw = pair_words(n), ns = n | 1;
  const int tid = threadIdx.x, nthreads = blockDim.x;
  float4* s_p0 = reinterpret_cast<float4*>(smem);
  float2* s_p1 = reinterpret_cast<float2*>(s_p0 + n);
  uint32_t* s_ex = reinterpret_cast<uint32_t*>(s_p1 + n);
  uint32_t* s_14 = s_ex + n * nw;
  float4* s_xall = reinterpret_cast<float4*>(smem + pair_head_bytes(n));
  float* s_Rall = reinterpret_cast<float*>(s_xall + G * n);
  float* s_ball = s_Rall + G * n;
  float* s_keep = s_ball + G * n;
  const int64_t c0 = (int64_t)blockIdx.x * G;
  const int g = (int)(N - c0 < G ? N - c0 : G);  // the block's configurations
  const int cf = tid / n, i = tid - cf * n;
  const bool own = cf < g;
  const float* xc = xs + c0 * n * 3;
  for (int q = tid; q < n; q += nthreads) {
    s_p0[q] = P.p0[q];
    s_p1[q] = P.p1[q];
  }
  for (int q = tid; q < n * nw; q += nthreads) {
    const int a = q / nw, w = q - a * nw;
    s_ex[q] = P.excl[a * kPairWords + w];
    s_14[q] = P.o14[a * kPairWords + w];
  }
  float4 xi = make_float4(0.f, 0.f, 0.f, 0.f);
  if (own) {
    xi.x = xc[3 * tid];
    xi.y = xc[3 * tid + 1];
    xi.z = xc[3 * tid + 2];
    s_xall[tid] = xi;
  }
  __syncthreads();

  float e_lj = 0.f, e_c = 0.f, e_gb = 0.f, e_sa = 0.f;
  float fx = 0.f, fy = 0.f, fz = 0.f, vx = 0.f, vy = 0.f, vz = 0.f;
  float dRdI = 0.f, Ri = 0.f;
  float4 pi = make_float4(0.f, 0.f, 0.f, 0.f);
  float2 qi1 = make_float2(0.f, 0.f);
  const float4* s_x = s_xall + cf * n;
  float* s_R = s_Rall + cf * n;
  float* s_b = s_ball + cf * n;
  float* kept = s_keep + (KEEP ? (size_t)cf * n * ns : 0);
  // pass 1: LJ, Coulomb, descreening
  if (own) {
    pi = s_p0[i];
    qi1 = s_p1[i];
    const float ra = __builtin_amdgcn_rcpf(qi1.x);
    const float kq = P.kc * pi.x, ei4 = 4.f * pi.z;
    float I = 0.f;
    for (int w = 0; w < nw; ++w) {
      const uint32_t ex = s_ex[i * nw + w], o4 = s_14[i * nw + w];
      const int jn = n - 32 * w < 32 ? n - 32 * w : 32;
#pragma unroll 2
      for (int b = 0; b < jn; ++b) {
        const int j = 32 * w + b;
        const bool self = j == i;
        const float4 xj = s_x[j], pj = s_p0[j];
        const float dx = xi.x - xj.x, dy = xi.y - xj.y, dz = xi.z - xj.z;
        const float r2 = dx * dx + dy * dy + dz * dz;
        const float ir = __builtin_amdgcn_rsqf(r2);
        float H, dH = 0.f;
        hct<FORCES, false>(r2, ir, qi1.x, ra, s_p1[j].y, H, dH);
        I += self ? 0.f : H;
        if (FORCES) {
          const float h = self ? 0.f : dH * ir;
          vx += h * dx;
          vy += h * dy;
          vz += h * dz;
          if (KEEP) kept[j * ns + i] = h;
        }
        const bool off = self || ((ex >> b) & 1);
        const bool f14 = (o4 >> b) & 1;
        const float sg = 0.5f * (pi.y + pj.y), ep4 = ei4 * pj.z;
        const float ir2 = ir * ir;
        const float sr2 = sg * sg * ir2, sr6 = sr2 * sr2 * sr2;
        const float l14 = f14 ? P.lj14 : 1.f, c14 = f14 ? P.el14 : 1.f;
        const float lj = ep4 * (sr6 * sr6 - sr6) * l14;
        const float cl = kq * pj.x * ir;
        e_lj += 0.5f * (off ? 0.f : lj);
        e_c += 0.5f * (off ? 0.f : cl * c14);
        if (FORCES) {
          const float f = ir2 * (6.f * ep4 * (2.f * sr6 * sr6 - sr6) * l14 +
                                 cl * c14);
          const float fo = off ? 0.f : f;
          fx += fo * dx;
          fy += fo * dy;
          fz += fo * dz;
        }
      }
    }
    // OBC II Born radius
    const float psi = I * qi1.x;
    const float t = psi * (kObcA - psi * (kObcB - kObcC * psi));
    const float th = tanhf(t);
    Ri = 1.f / (1.f / qi1.x - th / pi.w);
    dRdI = Ri * Ri * (1.f - th * th) *
           (kObcA - psi * (2.f * kObcB - 3.f * kObcC * psi)) * qi1.x / pi.w;
    s_R[i] = Ri;
  }
  __syncthreads();
  // pass 2: GB energy, explicit GB force, dE/dR_i; surface term
  if (own) {
    const float qi = pi.x, kqi = P.kgb * qi;
    e_gb = 0.5f * P.kgb * qi * qi / Ri;
    float dEdR = -0.5f * P.kgb * qi * qi / (Ri * Ri);
#pragma unroll 4
    for (int j = 0; j < n; ++j) {
      const float4 xj = s_x[j];
      const float dx = xi.x - xj.x, dy = xi.y - xj.y, dz = xi.z - xj.z;
      const float r2 = dx * dx + dy * dy + dz * dz;
      const float Rj = s_R[j];
      const float RR = Ri * Rj;
      const float iRR = __builtin_amdgcn_rcpf(RR);
      const float t = 0.25f * r2 * iRR;
      const float D = __expf(-t);
      const float f2 = r2 + RR * D;
      const float invf = __builtin_amdgcn_rsqf(f2);  // f2 is normal
      const float invf3 = invf * invf * invf;
      const float kq = (j == i ? 0.f : kqi) * s_p0[j].x;
      e_gb += 0.5f * kq * invf;
      if (FORCES) {
        const float g2 = kq * (1.f - 0.25f * D) * invf3;
        fx += g2 * dx;
        fy += g2 * dy;
        fz += g2 * dz;
        dEdR -= 0.5f * kq * Rj * D * (1.f + t) * invf3;
      }
    }
    const float rp = pi.w + P.probe;
    const float q6 = pi.w / Ri, q3 = q6 * q6 * q6;
    e_sa = P.sa * rp * rp * q3 * q3;
    dEdR -= 6.f * e_sa / Ri;
    s_b[i] = dEdR * dRdI;
  }
  __syncthreads();
  // pass 3: chain rule through the Born radii
  if (FORCES && own) {
    const float bi = s_b[i];
    float gx = bi * vx, gy = bi * vy, gz = bi * vz;
#pragma unroll 4
    for (int j = 0; j < n; ++j) {
      const float4 xj = s_x[j];
      const float dx = xi.x - xj.x, dy = xi.y - xj.y, dz = xi.z - xj.z;
      float h;
      if (KEEP) {
        h = kept[i * ns + j];
      } else {
        const float r2 = dx * dx + dy * dy + dz * dz;
        const float ir = __builtin_amdgcn_rsqf(r2);
        const float aj = s_p1[j].x;
        float H, dH;
        hct<true, true>(r2, ir, aj, __builtin_amdgcn_rcpf(aj), qi1.y, H, dH);
        h = j == i ? 0.f : dH * ir;
      }
      h *= s_b[j];
      gx += h * dx;
      gy += h * dy;
      gz += h * dz;
    }
    float* fo = forces + (c0 * n + tid) * 3;
    fo[0] = fx - gx;
    fo[1] = fy - gy;
    fo[2] = fz - gz;
  }
  // energies: a configuration's atoms in order, in double
  double* red = reinterpret_cast<double*>(
      smem + pair_head_bytes(n) + ((G * pair_conf_bytes(n) + 15) & ~15));
  if (KEEP) __syncthreads();  // the kept derivatives are read
  if (own) {
    red[4 * tid] = (double)e_lj;
    red[4 * tid + 1] = (double)e_c;
    red[4 * tid + 2] = (double)e_gb;
    red[4 * tid + 3] = (double)e_sa;
  }
  __syncthreads();
  for (int q = tid; q < 4 * g; q += nthreads) {
    const double* v = red + (q >> 2) * n * 4 + (q & 3);
    double s = 0.0;
#pragma unroll 8
    for (int a = 0; a < n; ++a) s += v[4 * a];
    terms[c0 * 4 + q] = s;
  }
}

}  // namespace

hipError_t launch_pair_terms(const PairDev& P, const float* x, int64_t N,
                             double* terms, float* forces, hipStream_t st) {
  if (N <= 0) return hipSuccess;
  if (P.n < 1 || P.n > kPairMaxAtoms || N > 0x7fffffffll)
    return hipErrorInvalidValue;
  const int n = P.n;
  const bool keep = forces && n <= kPairKeepAtoms;
  // configurations per workgroup: what its threads and 64 KB hold
  int G = kPairThreads / n, lds = 0;
  for (;; --G) {
    const int tail = keep && G * pair_keep_bytes(n) > G * n * 32
                         ? G * pair_keep_bytes(n) : G * n * 32;
    lds = pair_head_bytes(n) + ((G * pair_conf_bytes(n) + 15) & ~15) + tail;
    if (G == 1 || lds <= 65536) break;
  }
  const int64_t most = (1ll << 24) - 1;  // workgroups of 256 threads a launch
  auto kern = !forces ? k_pair_terms<false, false>
              : keep  ? k_pair_terms<true, true>
                      : k_pair_terms<true, false>;
  for (int64_t c = 0; c < N; c += most * G) {
    const int64_t now = N - c < most * G ? N - c : most * G;
    hipLaunchKernelGGL(kern, dim3((unsigned)((now + G - 1) / G)),
                       dim3((G * n + 63) / 64 * 64), lds, st, P,
                       x + c * n * 3, now, G, terms + 4 * c,
                       forces ? forces + c * n * 3 : nullptr);
  }
  return hipGetLastError();
}

}  // namespace bpmf
