// Learned rigid-body pose proposal on gfx950: a conditional Gaussian-mixture
// density q(t, omega | tau) from an MLP 16 -> 256 -> 256 -> 104 (SiLU), its
// training (negative log-likelihood, Adam) and the independence
// Metropolis-Hastings pose move it drives.  The paper's own pose move is a
// random rotation about the centre of mass plus a Gaussian translation with
// Metropolis acceptance (Sampling section); here the proposal is learned and
// the acceptance carries the exact proposal density on SE(3).
//
// Dense layers run on the matrix cores: v_mfma_f32_16x16x32_bf16 with bf16
// operands rounded from fp32 (activations when they are formed, weights when
// they change) and fp32 accumulation.
#include <hip/hip_runtime.h>
#include <math.h>

#include <algorithm>
#include <type_traits>

#include "deferred.h"
#include "device.h"
#include "internal.h"
#include "mlp.h"

namespace bpmf {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// fp32 -> bf16 bits, round to nearest even (finite inputs); NaN stays NaN
__device__ __forceinline__ unsigned short bf16_bits(float f) {
  const unsigned int u = __float_as_uint(f);
  const unsigned int rn = (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;
  const unsigned int qn = (u >> 16) | 0x40u;
  return (unsigned short)((u & 0x7fffffffu) > 0x7f800000u ? qn : rn);
}

constexpr int kKStep = 32;  // K per MFMA
constexpr int kPad = 8;     // LDS row padding (bf16 elements)

__device__ __forceinline__ float silu(float z) { return z / (1.0f + expf(-z)); }
__device__ __forceinline__ float dsilu(float z) {
  const float s = 1.0f / (1.0f + expf(-z));
  return s * (1.0f + z * (1.0f - s));
}

// The three dense layers for kFRows rows per workgroup.  A row's path
// through the network does not involve the other rows, so one workgroup
// takes its rows through all layers with the activations held in LDS as the
// next layer's bf16 operand; each wave owns every kFWaves-th 16-column output
// tile.
constexpr int kFRows = 16;
constexpr int kFWaves = 16;  // wavefronts per workgroup
constexpr int kFLd = kNHid + kPad;  // LDS row length (bf16 elements)

// Operand layout of the 16x16x32 bf16 MFMA: lane l supplies row (l % 16) of A
// and column (l % 16) of B, each with the 8 consecutive k = 8 (l / 16) .. + 7;
// it receives D rows 4 (l / 16) .. + 3 of column l % 16.

// One 16 x 16 tile of A(16 x KIN) B: A in LDS (rows of LDA, valid below KV),
// b = the lane's first element of its column's KLD-long bf16 row.  k ascends
// in chunks of 32.  The B loads (every chunk's, one 16-byte load each) can be
// issued by tile_load before the barrier that completes A.
template <int KIN>
struct TileB {
  bf16x8 v[KIN / kKStep];
};
template <int KIN>
__device__ __forceinline__ void tile_load(const unsigned short* b,
                                          TileB<KIN>& t) {
  typedef const bf16x8 __attribute__((address_space(1))) gbf;
#pragma unroll
  for (int q = 0; q < KIN / kKStep; ++q) t.v[q] = *(gbf*)(b + kKStep * q);
}
template <int KIN, int KV, int LDA>
__device__ __forceinline__ f32x4 tile_mul(const unsigned short (*A)[LDA],
                                          const TileB<KIN>& t, int lane) {
  const int kg = (lane >> 4) * 8;
  f32x4 acc{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int q = 0; q < KIN / kKStep; ++q) {
    bf16x8 a;
    if (KV % kKStep == 0 || kKStep * q + kg < KV) {
      a = *reinterpret_cast<const bf16x8*>(&A[lane & 15][kKStep * q + kg]);
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e)
        a[e] = __builtin_bit_cast(__bf16, (unsigned short)0);
    }
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, t.v[q], acc, 0, 0, 0);
  }
  return acc;
}

// One layer: out(16 x N) = act(A(16 x KIN) W + bias), the weights from their
// bf16 transposed copy (row n of WT holds column n of W, KLD elements, zero
// past KIN and past N): a lane's eight k values of a tile are one 16-byte
// load.
template <int KIN, int KLD, int N, bool HIDDEN>
__device__ __forceinline__ void dense_rows_t(
    const unsigned short (*A)[kFLd], const unsigned short* __restrict__ WT,
    const float* __restrict__ bias, int row0, int B, float* __restrict__ H,
    unsigned short (*Hn)[kFLd], int lane, int wv) {
  constexpr int kTiles = (N + 15) / 16;
  constexpr int kTPW = (kTiles + kFWaves - 1) / kFWaves;
  typedef const bf16x8 __attribute__((address_space(1))) gbf;
  const int kg = (lane >> 4) * 8;
  f32x4 acc[kTPW];
#pragma unroll
  for (int i = 0; i < kTPW; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  // every k step's weight loads in flight at once (one 16-byte load per
  // tile and step): one round trip to L2 per layer
#pragma unroll
  for (int k0 = 0; k0 < KIN; k0 += kKStep) {
    bf16x8 b[kTPW];
#pragma unroll
    for (int i = 0; i < kTPW; ++i) {
      const int n = (wv + kFWaves * i) * 16 + (lane & 15);
      if (wv + kFWaves * i < kTiles)  // uniform over the wave
        b[i] = *(gbf*)(WT + (int64_t)n * KLD + k0 + kg);
    }
    bf16x8 a;
    if (k0 + kg < KIN) {
      a = *reinterpret_cast<const bf16x8*>(&A[lane & 15][k0 + kg]);
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) a[e] = __builtin_bit_cast(__bf16,
                                                           (unsigned short)0);
    }
#pragma unroll
    for (int i = 0; i < kTPW; ++i)
      if (wv + kFWaves * i < kTiles)
        acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b[i], acc[i], 0,
                                                         0, 0);
  }
#pragma unroll
  for (int i = 0; i < kTPW; ++i) {
    const int n = (wv + kFWaves * i) * 16 + (lane & 15);
    if (n >= N) continue;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int r = (lane >> 4) * 4 + q, m = row0 + r;
      const float v = acc[i][q] + bias[n];
      if (HIDDEN)
        Hn[r][n] = bf16_bits(silu(v));
      else if (m < B)
        H[(int64_t)m * N + n] = v;
    }
  }
}

__device__ float dihedral_angle(const float* x, int4 q);

// The network on the current configurations of pose-move tasks, for groups
// of up to 16 rows (row m = task m), group b with its own parameters (bf16
// transposed weights), outputs only; each row's features (sin and cos of
// the conditioning torsions, the dihedral angles of the replica's
// configuration) are computed in place, one thread per (row, torsion slot).
// Blocks past n_groups close a run of neighbour-scheme sweeps instead, one
// ligand of `fin` each (finish_ligand): the features need only positions,
// which that leaves unchanged.
__global__ __launch_bounds__(kFWaves * 64) void k_pose_network(
    const MlpGroup* __restrict__ groups, int n_groups,
    const LigDev* __restrict__ ligs, const PropDev* __restrict__ props,
    const PoseTask* __restrict__ tasks, float* __restrict__ out,
    const LigDev* __restrict__ fin, int exchange_every, int sample_every,
    uint64_t seed) {
  if ((int)blockIdx.x >= n_groups) {
    finish_ligand(fin[blockIdx.x - n_groups], exchange_every, sample_every,
                  seed);
    return;
  }
  __shared__ __align__(16) unsigned short S[2][kFRows][kFLd];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const MlpGroup gr = groups[blockIdx.x];
  const int row0 = gr.row0, B = gr.row0 + gr.rows;
  static_assert(kNFeat == 16, "eight torsion slots of sin, cos");
  for (int e = tid; e < kFRows * 8; e += kFWaves * 64) {
    const int r = e >> 3, q = e & 7, m = row0 + r;
    float sn = 0.f, cs = 0.f;
    if (m < B) {
      const PoseTask t = tasks[m];
      const LigDev& L = ligs[t.lig];
      const PropDev& P = props[t.lig];
      if (q < P.n_cond) {
        const float phi =
            dihedral_angle(L.x + (size_t)t.r * L.n * 3, P.cond[q]);
        sincosf(phi, &sn, &cs);
      }
    }
    S[0][r][2 * q] = bf16_bits(sn);
    S[0][r][2 * q + 1] = bf16_bits(cs);
  }
  __syncthreads();
  dense_rows_t<kNFeat, kT1Ld, kNHid, true>(S[0], gr.WT + kTOff1,
                                           gr.P + kOffB1, row0, B, nullptr,
                                           S[1], lane, wv);
  __syncthreads();
  dense_rows_t<kNHid, kT2Ld, kNHid, true>(S[1], gr.WT + kTOff2,
                                          gr.P + kOffB2, row0, B, nullptr,
                                          S[0], lane, wv);
  __syncthreads();
  dense_rows_t<kNHid, kT3Ld, kNOut, false>(S[0], gr.WT + kTOff3,
                                           gr.P + kOffB3, row0, B, out,
                                           nullptr, lane, wv);
}

// WT from the fp32 parameters: element (n, k) of each transposed matrix is
// the bf16 rounding of W[k][n] (0 in the padding); then the same of W2 and W3
// row by row
__global__ __launch_bounds__(256) void k_weights_bf16(
    const float* __restrict__ P, unsigned short* __restrict__ WT) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= kTSize) return;
  int off, ld, kin, nout;
  const float* W;
  bool rows = false;
  if (i < kTOff2) {
    off = kTOff1; ld = kT1Ld; kin = kNFeat; nout = kNHid; W = P + kOffW1;
  } else if (i < kTOff3) {
    off = kTOff2; ld = kT2Ld; kin = kNHid; nout = kNHid; W = P + kOffW2;
  } else if (i < kTOffR2) {
    off = kTOff3; ld = kT3Ld; kin = kNHid; nout = kNOut; W = P + kOffW3;
  } else if (i < kTOffR3) {
    off = kTOffR2; ld = kNHid; kin = kNHid; nout = kNHid; W = P + kOffW2;
    rows = true;
  } else {
    off = kTOffR3; ld = kR3Ld; kin = kNHid; nout = kNOut; W = P + kOffW3;
    rows = true;
  }
  const int a = (i - off) / ld, b = (i - off) - a * ld;
  const int n = rows ? b : a, k = rows ? a : b;
  WT[i] = (n < nout && k < kin) ? bf16_bits(W[(int64_t)k * nout + n])
                                : (unsigned short)0;
}

// network outputs of B rows of features
__global__ __launch_bounds__(kFWaves * 64) void k_mlp_forward(
    const float* __restrict__ P, const unsigned short* __restrict__ WT,
    const float* __restrict__ X, int B, float* __restrict__ out) {
  __shared__ __align__(16) unsigned short S[2][kFRows][kFLd];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int row0 = blockIdx.x * kFRows;
  for (int e = tid; e < kFRows * kNFeat; e += kFWaves * 64) {
    const int r = e / kNFeat, k = e - r * kNFeat, m = row0 + r;
    S[0][r][k] = bf16_bits(m < B ? X[(int64_t)m * kNFeat + k] : 0.f);
  }
  __syncthreads();
  dense_rows_t<kNFeat, kT1Ld, kNHid, true>(S[0], WT + kTOff1, P + kOffB1,
                                           row0, B, nullptr, S[1], lane, wv);
  __syncthreads();
  dense_rows_t<kNHid, kT2Ld, kNHid, true>(S[1], WT + kTOff2, P + kOffB2, row0,
                                          B, nullptr, S[0], lane, wv);
  __syncthreads();
  dense_rows_t<kNHid, kT3Ld, kNOut, false>(S[0], WT + kTOff3, P + kOffB3,
                                           row0, B, out, nullptr, lane, wv);
}

__device__ __forceinline__ float sigm(float z) { return 1.0f / (1.0f + expf(-z)); }

// Mixture parameters of one output row (13 numbers per component).
struct Mix {
  float lw[kNComp];  // raw logits (mix_lse normalises them)
  float mt[kNComp][3], mw[kNComp][3], st[kNComp][3], sw[kNComp][3];
};

// log-normaliser of the raw mixture logits (the log-softmax's lse, float)
__device__ __forceinline__ float mix_lse(const Mix& p) {
  float mx = -INFINITY;
  for (int j = 0; j < kNComp; ++j) mx = fmaxf(mx, p.lw[j]);
  float sm = 0.f;
  for (int j = 0; j < kNComp; ++j) sm += expf(p.lw[j] - mx);
  return mx + logf(sm);
}

// ----------------------------------------------------------------------------
// training: the gradient of the mean negative log-likelihood, Adam
// ----------------------------------------------------------------------------
// columns of the transposed activations a row block leaves for the weight
// gradients, by matrix
__device__ __forceinline__ unsigned short* act_of(const TrainArgs& a, int row) {
  return a.act + (int64_t)row * a.Bp;
}

// the sum over a 16-row block of a tile's column (double), to biasP
__device__ __forceinline__ void put_bias(const TrainArgs& a, int off, int n,
                                         const float (&v)[4], int lane) {
  double s = ((double)v[0] + (double)v[1]) + ((double)v[2] + (double)v[3]);
  s += __shfl_xor(s, 16);
  s += __shfl_xor(s, 32);
  if (lane < 16) a.biasP[(int64_t)blockIdx.x * kNBias + off + n] = s;
}

// four rows (bf16) of a tile's column into row `col` of the transposed matrix
__device__ __forceinline__ void put_act(const TrainArgs& a, int base, int col,
                                        int row0, const unsigned short (&h)[4],
                                        int lane) {
  ushort4 p;
  p.x = h[0];
  p.y = h[1];
  p.z = h[2];
  p.w = h[3];
  *reinterpret_cast<ushort4*>(act_of(a, base + col) + row0 +
                              4 * (lane >> 4)) = p;
}

// Forward and backward pass of 16 rows of a minibatch by one workgroup: the
// minibatch's rows drawn (row i of step s is training row philox(s, i) mod N,
// with replacement) or taken in order, the three layers, the mixture's
// likelihood gradient, and the two hidden layers' dZ.  Activations go from
// layer to layer through LDS, pre-activations stay in their wavefront's
// registers until the backward pass needs them; the bf16 activations and dZ
// (transposed, as the weight gradients' MFMA operands) and the block's bias
// and loss sums (double) are what leaves the block.  Rows past B are zero.
// Bound by latency (512 rows: 32 workgroups, seven dependent stages, the
// weights from L2): one launch of 19 us, where a gather, a forward kernel, a
// likelihood kernel of one thread per row, two GEMMs and three column sums
// took 150 us.
__global__ __launch_bounds__(kFWaves * 64) void k_train_rows(TrainArgs a) {
  __shared__ __align__(16) unsigned short S[2][kFRows][kFLd];
  __shared__ __align__(16) unsigned short D[kFRows][kR3Ld + kPad];
  __shared__ float O[kFRows][kNOut];
  __shared__ float ps[kFRows][6];
  __shared__ int64_t src[kFRows];
  __shared__ double lred[2];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int row0 = blockIdx.x * kFRows, B = a.B;
  const int c = lane & 15, n = wv * 16 + c;  // the wavefront's tile's column
  const int kg = (lane >> 4) * 8;
  if (tid < kFRows) {
    const int m = row0 + tid;
    int64_t j = m;
    if (a.gather) {
      const U4 o = philox4x32_10((uint32_t)m, (uint32_t)(a.step >> 32),
                                 (uint32_t)a.step, kBatch, (uint32_t)a.seed,
                                 (uint32_t)(a.seed >> 32));
      j = (int64_t)((((uint64_t)o.x << 32) | o.y) % (uint64_t)a.N);
    }
    src[tid] = j;
  }
  TileB<kT1Ld> w1;
  TileB<kNHid> w2;
  tile_load<kT1Ld>(a.WT + kTOff1 + (int64_t)n * kT1Ld + kg, w1);
  tile_load<kNHid>(a.WT + kTOff2 + (int64_t)n * kT2Ld + kg, w2);
  for (int e = tid; e < kFRows * (kR3Ld + kPad); e += kFWaves * 64)
    D[e / (kR3Ld + kPad)][e % (kR3Ld + kPad)] = 0;
  __syncthreads();
  if (tid < kFRows * kNFeat) {
    const int r = tid / kNFeat, k = tid - r * kNFeat;
    const unsigned short v =
        row0 + r < B ? bf16_bits(a.feats[src[r] * kNFeat + k])
                     : (unsigned short)0;
    S[0][r][k] = v;
    act_of(a, kActF + k)[row0 + r] = v;
  } else if (tid < kFRows * (kNFeat + 6)) {
    const int e = tid - kFRows * kNFeat, r = e / 6, q = e - 6 * r;
    ps[r][q] = row0 + r < B ? a.poses[src[r] * 6 + q] : 0.f;
  }
  __syncthreads();
  float z1[4], z2[4];
  unsigned short h[4];
  {
    const f32x4 v = tile_mul<kT1Ld, kNFeat, kFLd>(S[0], w1, lane);
    const float b = a.P[kOffB1 + n];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int r = (lane >> 4) * 4 + q;
      z1[q] = v[q] + b;
      h[q] = bf16_bits(silu(z1[q]));
      S[1][r][n] = h[q];
      if (row0 + r >= B) h[q] = 0;
    }
    put_act(a, kActH1, n, row0, h, lane);
  }
  TileB<kNHid> w3;
  if (wv < kT3Rows / 16)
    tile_load<kNHid>(a.WT + kTOff3 + (int64_t)n * kT3Ld + kg, w3);
  __syncthreads();
  {
    const f32x4 v = tile_mul<kNHid, kNHid, kFLd>(S[1], w2, lane);
    const float b = a.P[kOffB2 + n];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int r = (lane >> 4) * 4 + q;
      z2[q] = v[q] + b;
      h[q] = bf16_bits(silu(z2[q]));
      S[0][r][n] = h[q];
      if (row0 + r >= B) h[q] = 0;
    }
    put_act(a, kActH2, n, row0, h, lane);
  }
  TileB<kR3Ld> r3;
  tile_load<kR3Ld>(a.WT + kTOffR3 + (int64_t)n * kR3Ld + kg, r3);
  __syncthreads();
  if (wv < kT3Rows / 16) {
    const f32x4 v = tile_mul<kNHid, kNHid, kFLd>(S[0], w3, lane);
    if (n < kNOut) {
      const float b = a.P[kOffB3 + n];
#pragma unroll
      for (int q = 0; q < 4; ++q) O[(lane >> 4) * 4 + q][n] = v[q] + b;
    }
  }
  TileB<kNHid> r2;
  tile_load<kNHid>(a.WT + kTOffR2 + (int64_t)n * kNHid + kg, r2);
  __syncthreads();
  // negative log-likelihood and its gradient: component j of row r by thread
  // 8 r + j; the sums over a row's components run in component order
  if (tid < kFRows * kNComp) {
    const int r = tid / kNComp, j = tid - r * kNComp;
    const bool in = row0 + r < B;
    float* o = &O[r][13 * j];
    const float* pose = ps[r];
    const int l0 = lane & ~(kNComp - 1);
    auto row_lse = [&](float v) {  // log sum exp over the row's components
      float mx = -INFINITY;
#pragma unroll
      for (int q = 0; q < kNComp; ++q) mx = fmaxf(mx, __shfl(v, l0 + q));
      const float e = expf(v - mx);
      float t = 0.f;
#pragma unroll
      for (int q = 0; q < kNComp; ++q) t += __shfl(e, l0 + q);
      return mx + logf(t);
    };
    auto sub = [](float x, float y) {  // rounded by itself: no product fused
#pragma clang fp contract(off)
      return x - y;
    };
    const float lw = o[0] - row_lse(o[0]);
    float mt[3], mw[3], st[3], sw[3], zt[3], zw[3], th[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      mt[d] = o[1 + d];
      th[d] = tanhf(o[4 + d]);
      mw[d] = (float)M_PI * th[d];
      st[d] = kSt0 + (kSt1 - kSt0) * sigm(o[7 + d]);
      sw[d] = kSw0 + (kSw1 - kSw0) * sigm(o[10 + d]);
    }
    // One difference of the 24 is a single rounding of t - pi tanh, the others
    // of t - fl(pi tanh).  Nothing in the mathematics asks for it: an earlier
    // compilation fused that one product.  It is kept because a step's bits
    // decide those of the steps after it (bf16 roundings flip): with one form
    // for all, 20 steps end in other weights, as far from the 64-bit ones.
    const float last = fmaf(-(float)M_PI, th[2], pose[5]);
    float lg = lw - 3.0f * logf(2.0f * (float)M_PI);
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      zt[d] = (pose[d] - mt[d]) / st[d];
      zw[d] = (j == kNComp - 1 && d == 2 ? last : sub(pose[3 + d], mw[d])) /
              sw[d];
      lg += -0.5f * (zt[d] * zt[d] + zw[d] * zw[d]) - logf(st[d]) -
            logf(sw[d]);
    }
    const float ll = row_lse(lg);
    const float rj = expf(lg - ll), pi = expf(lw);
    float dj[13];
    dj[0] = -(rj - pi) * a.inv_b;
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      dj[1 + q] = -rj * zt[q] / st[q] * a.inv_b;
      dj[4 + q] = -rj * zw[q] / sw[q] * (float)M_PI * fmaf(-th[q], th[q], 1.f) *
                  a.inv_b;
      float sg = sigm(o[7 + q]);
      dj[7 + q] = -rj * fmaf(zt[q], zt[q], -1.f) / st[q] * (kSt1 - kSt0) * sg *
                  (1.f - sg) * a.inv_b;
      sg = sigm(o[10 + q]);
      dj[10 + q] = -rj * fmaf(zw[q], zw[q], -1.f) / sw[q] * (kSw1 - kSw0) * sg *
                   (1.f - sg) * a.inv_b;
    }
#pragma unroll
    for (int q = 0; q < 13; ++q) {
      o[q] = in ? dj[q] : 0.f;
      D[r][13 * j + q] = in ? bf16_bits(dj[q]) : (unsigned short)0;
    }
    // eight rows a wavefront, one value each
    const double l = wave_sum(j == 0 && in ? -(double)ll : 0.0);
    if (lane == 0) lred[wv] = l;
  }
  __syncthreads();
  if (tid == 0) a.lossP[blockIdx.x] = lred[0] + lred[1];
  // dZ2 = (dout W3^T) silu'(Z2), dZ1 = (dZ2 W2^T) silu'(Z1)
  {
    const f32x4 v = tile_mul<kR3Ld, kR3Ld, kR3Ld + kPad>(D, r3, lane);
    float dz[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      dz[q] = v[q] * dsilu(z2[q]);
      h[q] = bf16_bits(dz[q]);
      S[1][(lane >> 4) * 4 + q][n] = h[q];
    }
    put_act(a, kActZ2, n, row0, h, lane);
    put_bias(a, kNHid, n, dz, lane);
  }
  __syncthreads();
  {
    const f32x4 v = tile_mul<kNHid, kNHid, kFLd>(S[1], r2, lane);
    float dz[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      dz[q] = v[q] * dsilu(z1[q]);
      h[q] = bf16_bits(dz[q]);
    }
    put_act(a, kActZ1, n, row0, h, lane);
    put_bias(a, 0, n, dz, lane);
  }
  // the output layer's columns
  if (tid < kNOut) {
    double s = 0.0;
    for (int r = 0; r < kFRows; ++r) s += (double)O[r][tid];
    a.biasP[(int64_t)blockIdx.x * kNBias + 2 * kNHid + tid] = s;
  }
  for (int e = tid; e < kT3Rows * kFRows; e += kFWaves * 64) {
    const int col = e / kFRows, r = e - col * kFRows;
    act_of(a, kActD + col)[row0 + r] = D[r][col];
  }
}

// One parameter's gradient: stored, or taken as an Adam step (Kingma & Ba) on
// the fp32 master parameter
__device__ __forceinline__ float take_grad(const AdamArgs& w, int i, float g) {
  if (w.G) {
    w.G[i] = g;
    return 0.f;
  }
  const float mi = w.b1 * w.m[i] + (1.f - w.b1) * g;
  const float vi = w.b2 * w.v[i] + (1.f - w.b2) * g * g;
  w.m[i] = mi;
  w.v[i] = vi;
  const float p = w.P[i] - w.lr * (mi / w.c1) / (sqrtf(vi / w.c2) + w.eps);
  w.P[i] = p;
  return p;
}
// the updated weight (k, n) of matrix 1..3 in the bf16 copies
__device__ __forceinline__ void put_weight(unsigned short* WT, int mat, int k,
                                           int n, float p) {
  const unsigned short h = bf16_bits(p);
  if (mat == 1) {
    WT[kTOff1 + n * kT1Ld + k] = h;
  } else if (mat == 2) {
    WT[kTOff2 + n * kT2Ld + k] = h;
    WT[kTOffR2 + k * kNHid + n] = h;
  } else {
    WT[kTOff3 + n * kT3Ld + k] = h;
    WT[kTOffR3 + k * kR3Ld + n] = h;
  }
}
// the matrix, first row and first column of weight tile t (16 x 16)
__device__ __forceinline__ int weight_tile(int t, int& k0, int& n0) {
  constexpr int kHT = kNHid / 16, kOT = kT3Rows / 16;
  if (t < kHT * kHT) {
    k0 = t / kHT * 16;
    n0 = t % kHT * 16;
    return 2;
  }
  t -= kHT * kHT;
  if (t < kHT * kOT) {
    k0 = t / kOT * 16;
    n0 = t % kOT * 16;
    return 3;
  }
  k0 = 0;
  n0 = (t - kHT * kOT) * 16;
  return 1;
}

// Weight gradients H2^T dout, H1^T dZ2 and feats^T dZ1 (one wavefront per 16
// x 16 tile, over the rows in order; both operands are 16-byte loads of the
// transposed activations) with their Adam step or, for a split of many rows
// (blockIdx.y), the split's partial gradient.  The blocks past the tiles sum
// the biases' columns over the row blocks and, the last one, the loss (both
// once, in double).  Bound by latency at a minibatch's size (16 chunks of 32
// rows): 8.8 us with Adam, where three GEMMs whose 64 x 64 tiles left most of
// the chip idle and an update pass took 113 us.
constexpr int kTilesW = (kNHid / 16) * (kNHid / 16) +
                        (kNHid / 16) * (kT3Rows / 16) + kNHid / 16;
constexpr int kTileBlocks = kTilesW / 4;
constexpr int kBiasBlocks = (kNBias + 63) / 64;
static_assert(kTilesW % 4 == 0, "four tiles a block");
__global__ __launch_bounds__(256) void k_train_weights(TrainArgs a, AdamArgs w,
                                                       int n_split,
                                                       float* split,
                                                       double* loss) {
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  if ((int)blockIdx.x >= kTileBlocks) {
    if (blockIdx.y > 0) return;
    __shared__ double part[256];
    const int blk = blockIdx.x - kTileBlocks, nb = a.Bp / kFRows;
    double s = 0.0;
    if (blk < kBiasBlocks) {
      const int c = 64 * blk + lane;
      if (c < kNBias)
#pragma unroll 8
        for (int q = wv; q < nb; q += 4) s += a.biasP[(int64_t)q * kNBias + c];
      part[tid] = s;
      __syncthreads();
      if (wv == 0 && c < kNBias) {
        const float g = (float)(((part[lane] + part[64 + lane]) +
                                 part[128 + lane]) + part[192 + lane]);
        const int i = c < kNHid       ? kOffB1 + c
                      : c < 2 * kNHid ? kOffB2 + c - kNHid
                                      : kOffB3 + c - 2 * kNHid;
        take_grad(w, i, g);
      }
    } else {
      for (int q = tid; q < nb; q += 256) s += a.lossP[q];
      part[tid] = s;
      __syncthreads();
      for (int st = 128; st > 0; st >>= 1) {
        if (tid < st) part[tid] += part[tid + st];
        __syncthreads();
      }
      if (tid == 0) *loss = part[0];
    }
    return;
  }
  int k0, n0;
  const int mat = weight_tile(blockIdx.x * 4 + wv, k0, n0);
  const unsigned short* A =
      act_of(a, (mat == 1 ? kActF : mat == 2 ? kActH1 : kActH2) + k0 +
                    (lane & 15)) + (lane >> 4) * 8;
  const unsigned short* Bt =
      act_of(a, (mat == 1 ? kActZ1 : mat == 2 ? kActZ2 : kActD) + n0 +
                    (lane & 15)) + (lane >> 4) * 8;
  const int steps = a.Bp / kKStep;
  const int s0 = (int)((int64_t)steps * blockIdx.y / n_split);
  const int s1 = (int)((int64_t)steps * (blockIdx.y + 1) / n_split);
  typedef const bf16x8 __attribute__((address_space(1))) gbf;
  f32x4 acc{0.f, 0.f, 0.f, 0.f};
  int q = s0;
  auto chunks = [&](auto len) {  // len chunks at a time: loads, then products
    constexpr int kL = decltype(len)::value;
    for (; q + kL <= s1; q += kL) {
      bf16x8 x[kL], y[kL];
#pragma unroll
      for (int e = 0; e < kL; ++e) {
        x[e] = *(gbf*)(A + (int64_t)kKStep * (q + e));
        y[e] = *(gbf*)(Bt + (int64_t)kKStep * (q + e));
      }
#pragma unroll
      for (int e = 0; e < kL; ++e)
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x[e], y[e], acc, 0, 0,
                                                      0);
    }
  };
  chunks(std::integral_constant<int, 16>{});
  chunks(std::integral_constant<int, 4>{});
  chunks(std::integral_constant<int, 1>{});
  const int nout = mat == 3 ? kNOut : kNHid;
  const int off = mat == 1 ? kOffW1 : mat == 2 ? kOffW2 : kOffW3;
  const int n = n0 + (lane & 15);
  if (n >= nout) return;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int k = k0 + 4 * (lane >> 4) + e, i = off + k * nout + n;
    if (n_split > 1) {
      split[(int64_t)blockIdx.y * kNParams + i] = acc[e];
    } else {
      const float p = take_grad(w, i, acc[e]);
      if (!w.G) put_weight(a.WT, mat, k, n, p);
    }
  }
}

// the splits' weight gradients summed (double, in order), with their Adam step
__global__ __launch_bounds__(256) void k_train_splits(
    AdamArgs w, unsigned short* WT, const float* __restrict__ split,
    int n_split) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= kNParams) return;
  int mat, k, n;
  if (i < kOffB1) {
    mat = 1; k = i / kNHid; n = i % kNHid;
  } else if (i >= kOffW2 && i < kOffB2) {
    mat = 2; k = (i - kOffW2) / kNHid; n = (i - kOffW2) % kNHid;
  } else if (i >= kOffW3 && i < kOffB3) {
    mat = 3; k = (i - kOffW3) / kNOut; n = (i - kOffW3) % kNOut;
  } else {
    return;  // a bias
  }
  double s = 0.0;
  for (int q = 0; q < n_split; ++q) s += (double)split[(int64_t)q * kNParams + i];
  const float p = take_grad(w, i, (float)s);
  if (!w.G) put_weight(WT, mat, k, n, p);
}

// ----------------------------------------------------------------------------
// pose of a configuration: t = COM - c0, R = body frame, omega = log R,
// features = sin/cos of the conditioning torsions
// ----------------------------------------------------------------------------
struct Frame {
  float R[3][3];  // columns e1, e2, e3
};

__device__ void body_frame(const float* x, const int* fa, Frame& F) {
  float e1[3], v[3], e2[3];
  for (int a = 0; a < 3; ++a) {
    e1[a] = x[3 * fa[1] + a] - x[3 * fa[0] + a];
    v[a] = x[3 * fa[2] + a] - x[3 * fa[0] + a];
  }
  float l = rsqrtf(e1[0] * e1[0] + e1[1] * e1[1] + e1[2] * e1[2]);
  for (int a = 0; a < 3; ++a) e1[a] *= l;
  const float pr = v[0] * e1[0] + v[1] * e1[1] + v[2] * e1[2];
  for (int a = 0; a < 3; ++a) e2[a] = v[a] - pr * e1[a];
  l = rsqrtf(e2[0] * e2[0] + e2[1] * e2[1] + e2[2] * e2[2]);
  for (int a = 0; a < 3; ++a) e2[a] *= l;
  const float e3[3] = {e1[1] * e2[2] - e1[2] * e2[1],
                       e1[2] * e2[0] - e1[0] * e2[2],
                       e1[0] * e2[1] - e1[1] * e2[0]};
  for (int a = 0; a < 3; ++a) {
    F.R[a][0] = e1[a];
    F.R[a][1] = e2[a];
    F.R[a][2] = e3[a];
  }
}

// rotation vector of R (double), |omega| in [0, pi]: theta from
// atan2(|v|/2, (tr R - 1)/2) with v the axial vector of R - R^T, axis
// v/|v| (well conditioned up to theta -> pi); within ~5e-5 of pi the axis
// comes from the symmetric part (R + R^T)/4 + I/2 = n n^T
__device__ void log_rot(const double R[3][3], double w[3]) {
  const double c = (R[0][0] + R[1][1] + R[2][2] - 1.0) * 0.5;
  const double v[3] = {R[2][1] - R[1][2], R[0][2] - R[2][0], R[1][0] - R[0][1]};
  const double s2 = sqrt(v[0] * v[0] + v[1] * v[1] + v[2] * v[2]);
  const double th = atan2(0.5 * s2, c);
  if (s2 < 1e-12 && c > 0) {
    for (int a = 0; a < 3; ++a) w[a] = 0.5 * v[a];
    return;
  }
  if (s2 >= 1e-12 && (s2 > 1e-4 || c > 0)) {
    for (int a = 0; a < 3; ++a) w[a] = th * v[a] / s2;
    return;
  }
  double B[3][3];
  for (int a = 0; a < 3; ++a)
    for (int b = 0; b < 3; ++b)
      B[a][b] = 0.25 * (R[a][b] + R[b][a]) + (a == b ? 0.5 : 0.0);
  int k = 0;
  if (B[1][1] > B[k][k]) k = 1;
  if (B[2][2] > B[k][k]) k = 2;
  double n[3] = {B[0][k], B[1][k], B[2][k]};
  const double ln = sqrt(n[0] * n[0] + n[1] * n[1] + n[2] * n[2]);
  const double dn = n[0] * v[0] + n[1] * v[1] + n[2] * v[2];
  const double sgn = dn < 0 ? -1.0 : 1.0;
  for (int a = 0; a < 3; ++a) w[a] = sgn * th * n[a] / ln;
}

__device__ void rodrigues(const double w[3], double R[3][3]) {
  const double th = sqrt(w[0] * w[0] + w[1] * w[1] + w[2] * w[2]);
  const double K[3][3] = {{0, -w[2], w[1]}, {w[2], 0, -w[0]}, {-w[1], w[0], 0}};
  double a, b;
  if (th < 1e-8) {
    a = 1.0;
    b = 0.5;
  } else {
    a = sin(th) / th;
    b = (1.0 - cos(th)) / (th * th);
  }
  for (int i = 0; i < 3; ++i)
    for (int j = 0; j < 3; ++j) {
      double kk = 0.0;
      for (int q = 0; q < 3; ++q) kk += K[i][q] * K[q][j];
      R[i][j] = (i == j ? 1.0 : 0.0) + a * K[i][j] + b * kk;
    }
}

__device__ float dihedral_angle(const float* x, int4 q) {
  float b1[3], b2[3], b3[3];
  for (int a = 0; a < 3; ++a) {
    b1[a] = x[3 * q.y + a] - x[3 * q.x + a];
    b2[a] = x[3 * q.z + a] - x[3 * q.y + a];
    b3[a] = x[3 * q.w + a] - x[3 * q.z + a];
  }
  const float n1[3] = {b1[1] * b2[2] - b1[2] * b2[1], b1[2] * b2[0] - b1[0] * b2[2],
                       b1[0] * b2[1] - b1[1] * b2[0]};
  const float n2[3] = {b2[1] * b3[2] - b2[2] * b3[1], b2[2] * b3[0] - b2[0] * b3[2],
                       b2[0] * b3[1] - b2[1] * b3[0]};
  const float lb2 = sqrtf(b2[0] * b2[0] + b2[1] * b2[1] + b2[2] * b2[2]);
  const float y = lb2 * (b1[0] * n2[0] + b1[1] * n2[1] + b1[2] * n2[2]);
  const float xx = n1[0] * n2[0] + n1[1] * n2[1] + n1[2] * n2[2];
  return atan2f(y, xx);
}

// the translation of the pose of configuration x of ligand L, and the rotation
__device__ void pose_translation(const LigDev& L, const float* x, float* t) {
  double c[3] = {0, 0, 0}, M = 0;
  for (int a = 0; a < L.n; ++a) {
    const double m = L.mass[a];
    M += m;
    for (int d = 0; d < 3; ++d) c[d] += m * x[3 * a + d];
  }
  for (int d = 0; d < 3; ++d) t[d] = (float)(c[d] / M - L.site[d]);
}
__device__ void pose_rotation(const PropDev& P, const float* x, float* om) {
  Frame F;
  body_frame(x, P.frame, F);
  double R[3][3], w[3];
  for (int a = 0; a < 3; ++a)
    for (int b = 0; b < 3; ++b) R[a][b] = F.R[a][b];
  log_rot(R, w);
  for (int d = 0; d < 3; ++d) om[d] = (float)w[d];
}

// m rows of `len` floats between consecutive memory g and LDS rows `row`
// floats apart, by the whole
// workgroup; 16 bytes at a time where g is aligned
constexpr int kFeatWaves = 4;
template <bool OUT>
__device__ __forceinline__ void move_rows(float* g, int len, int m, float* l,
                                          int row) {
  const int tid = threadIdx.x, total = m * len;
  const int quads = (reinterpret_cast<uintptr_t>(g) & 15) == 0 ? total / 4 : 0;
#pragma unroll 4
  for (int q = tid; q < quads; q += kFeatWaves * 64) {
    float4* g4 = reinterpret_cast<float4*>(g) + q;
    float v[4] = {};
    if (!OUT) *reinterpret_cast<float4*>(v) = *g4;
    int c = 4 * q % len;
    float* at = l + 4 * q / len * row + c;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (OUT)
        v[e] = *at;
      else
        *at = v[e];
      ++at;
      if (++c == len) {
        c = 0;
        at += row - len;
      }
    }
    if (OUT) *g4 = make_float4(v[0], v[1], v[2], v[3]);
  }
  for (int e = 4 * quads + tid; e < total; e += kFeatWaves * 64) {
    float* at = l + e / len * row + e % len;
    if (OUT)
      g[e] = *at;
    else
      *at = g[e];
  }
}

// 64 configurations xs[i] of one ligand by four wavefronts: one takes the
// centres of mass, one the rotations, two the torsions, since 100000
// configurations are one and a half wavefronts per SIMD and the serial chain
// of a configuration (sums, atan2, a rotation's logarithm) was what bound
// this.  Positions and results pass through LDS, so that memory is read and
// written 16 bytes at a time; an odd row length spreads the rows over the
// banks.  100000 configurations of 24 atoms: 12 us; one thread for all of
// a configuration took 33 us (42 us staged like this).  64 rows of a large
// ligand would pass 64 KB: 32 then.
constexpr int kFeatOut = 6 + kNFeat;
__host__ __device__ constexpr int feat_row(int n) {
  return (3 * n > kFeatOut ? 3 * n : kFeatOut) | 1;
}
__host__ __device__ constexpr int feat_confs(int n) {
  return feat_row(n) <= 256 ? 64 : 32;
}
__global__ __launch_bounds__(kFeatWaves * 64) void k_pose_features(
    const LigDev* __restrict__ lig, const PropDev* __restrict__ prop,
    const float* __restrict__ xs, int64_t N, float* __restrict__ feats,
    float* __restrict__ poses) {
  extern __shared__ float s_conf[];
  const LigDev& L = *lig;
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int len = 3 * L.n, row = feat_row(L.n), most = feat_confs(L.n);
  const int64_t i0 = (int64_t)blockIdx.x * most;
  const int m = (int)(N - i0 < most ? N - i0 : most);
  move_rows<false>(const_cast<float*>(xs) + i0 * len, len, m, s_conf, row);
  __syncthreads();
  float* x = s_conf + lane * row;
  float v[kNFeat / 2];
  if (lane < m) {
    if (wv == 0) {
      pose_translation(L, x, v);
    } else if (wv == 1) {
      pose_rotation(*prop, x, v);
    } else {
#pragma unroll
      for (int q = 0; q < kNFeat / 4; ++q) {
        const int k = (wv - 2) + 2 * q;  // torsion
        v[2 * q] = v[2 * q + 1] = 0.f;
        if (k < prop->n_cond)
          sincosf(dihedral_angle(x, prop->cond[k]), &v[2 * q], &v[2 * q + 1]);
      }
    }
  }
  __syncthreads();
  if (lane < m) {
    if (wv < 2) {
#pragma unroll
      for (int d = 0; d < 3; ++d) x[3 * wv + d] = v[d];
    } else {
#pragma unroll
      for (int q = 0; q < kNFeat / 4; ++q) {
        const int k = (wv - 2) + 2 * q;
        x[6 + 2 * k] = v[2 * q];
        x[7 + 2 * k] = v[2 * q + 1];
      }
    }
  }
  __syncthreads();
  move_rows<true>(poses + i0 * 6, 6, m, s_conf, row);
  move_rows<true>(feats + i0 * kNFeat, kNFeat, m, s_conf + 6, row);
}

// wavefront maximum of a double (DPP tree as in wave_sum)
__device__ __forceinline__ double wave_max_d(double v) {
  v = fmax(v, dpp_d<0xB1, 0xf>(v));
  v = fmax(v, dpp_d<0x4E, 0xf>(v));
  v = fmax(v, dpp_d<0x141, 0xf>(v));
  v = fmax(v, dpp_d<0x140, 0xf>(v));
  // rows that receive no broadcast keep their value (bound_ctrl off): the
  // update_dpp "old" operand is 0 there, so take max with the lane's own
  const double b15 = dpp_d<0x142, 0xa>(v);
  if ((threadIdx.x & 63) >= 16 && ((threadIdx.x >> 4) & 1)) v = fmax(v, b15);
  const double b31 = dpp_d<0x143, 0xc>(v);
  if ((threadIdx.x & 63) >= 32) v = fmax(v, b31);
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffffll), 63);
  const int hi = __builtin_amdgcn_readlane((int)(b >> 32), 63);
  return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
}

// log q_SE3(t, omega): the mixture density of (t, omega') summed over the
// preimages omega' = omega/|omega| (|omega| + 2 pi m), m = -kFold..kFold, of
// the same rotation, each with the Haar-measure factor |omega'|^2 /
// (2 (1 - cos|omega|)); one (preimage, component) term per lane of the
// calling wavefront (all 64 lanes call; lanes past the terms add nothing)
// and a log-sum-exp across the wavefront.  |omega| < 1e-9: the identity
// rotation, one term per component.  c0[j]: the pose-free part of
// component j's log-density, its normalised log weight less 3 ln 2 pi and
// the logs of its six standard deviations.
__device__ double log_q_se3_wave(const Mix& p, const double* c0,
                                 const double t[3], const double w0[3]) {
  const int lane = threadIdx.x & 63;
  const double th = sqrt(w0[0] * w0[0] + w0[1] * w0[1] + w0[2] * w0[2]);
  const bool small = th < 1e-9;
  const int n_terms = small ? kNComp : (2 * kFold + 1) * kNComp;
  double term = -INFINITY;
  if (lane < n_terms) {
    const int j = lane % kNComp, m = lane / kNComp - kFold;
    double s = c0[j];
    for (int d = 0; d < 3; ++d) {
      const double z = (t[d] - p.mt[j][d]) / p.st[j][d];
      s += -0.5 * z * z;
    }
    if (small) {
      for (int d = 0; d < 3; ++d) {
        const double z = (0.0 - p.mw[j][d]) / p.sw[j][d];
        s += -0.5 * z * z;
      }
    } else {
      const double a = th + 2.0 * M_PI * m;
      s += 2.0 * log(fabs(a)) - log(2.0 * (1.0 - cos(th)));
      for (int d = 0; d < 3; ++d) {
        const double z = (a * w0[d] / th - p.mw[j][d]) / p.sw[j][d];
        s += -0.5 * z * z;
      }
    }
    term = s;
  }
  const double mx = wave_max_d(term);
  const double e = lane < n_terms ? exp(term - mx) : 0.0;
  return mx + log(wave_sum(e));
}

// Independence MH pose move, one workgroup of W waves per task (replica
// t.r of ligand t.lig, network outputs in row t.row).  The move is rigid, so
// the bonded energy does not change: only the grid terms and the restraint
// are evaluated at the proposed pose, and the bonded part of the energy is
// the cached one (the cached U_bond + U_angle + U_tors + U_I less the
// restraint energy of the current centre of mass).
template <int C, int W>
__global__ __launch_bounds__(W * kWave) void k_pose_move(
    GridDev g, const LigDev* __restrict__ ligs,
    const PropDev* __restrict__ props, const PoseTask* __restrict__ tasks,
    const float* __restrict__ out, uint64_t seed, int begin_next) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ float sR[9], st[3], scom[3];
  __shared__ int s_ok;
  __shared__ double s_ui0;
  const PoseTask task = tasks[blockIdx.x];
  const LigDev L = ligs[task.lig];
  const PropDev& P = props[task.lig];
  const int tid = threadIdx.x;
  const int r = task.r;
  const int n = L.n;
  const unsigned long long s = *L.counter;
  const int k = L.state_of_replica[r];
  const float* xr = L.x + (size_t)r * n * 3;
  // current pose, proposal and the proposal-density ratio (double): the
  // centre of mass by a block reduction, the mixture parsed one component
  // per lane, the two proposal densities one term per lane of wave 0, the
  // frames and the draws on thread 0
  __shared__ double s_cp[2 * W * 3];
  __shared__ Mix s_mix;
  __shared__ double s_pose[12];  // t0, w0, t1, w1p
  // per component: -3 ln 2 pi - sum_d (ln st + ln sw), then (once the
  // weights are normalised) plus its normalised log weight
  __shared__ double s_c0[kNComp];
  double lq_ratio = 0.0;
  {
    const bool own = tid < n;
    const double mi = own ? (double)L.mass[tid] : 0.0;
    const double cx = wave_sum(own ? mi * xr[3 * tid] : 0.0);
    const double cy = wave_sum(own ? mi * xr[3 * tid + 1] : 0.0);
    const double cz = wave_sum(own ? mi * xr[3 * tid + 2] : 0.0);
    const double cm = wave_sum(mi);
    if ((tid & 63) == 0) {
      const int wv = tid >> 6;
      s_cp[4 * wv] = cx;
      s_cp[4 * wv + 1] = cy;
      s_cp[4 * wv + 2] = cz;
      s_cp[4 * wv + 3] = cm;
    }
    // the mixture on the last wavefront (the one with the fewest atoms),
    // with each component's log-density constant but its weight
    const int j = tid - (W - 1) * kWave;
    if (j >= 0 && j < kNComp) {
      const float* o = out + (size_t)task.row * kNOut + 13 * j;
      s_mix.lw[j] = o[0];
      double c = -3.0 * log(2.0 * M_PI);
      for (int a = 0; a < 3; ++a) {
        s_mix.mt[j][a] = o[1 + a];
        s_mix.mw[j][a] = (float)M_PI * tanhf(o[4 + a]);
        const float sd_t = kSt0 + (kSt1 - kSt0) * sigm(o[7 + a]);
        const float sd_w = kSw0 + (kSw1 - kSw0) * sigm(o[10 + a]);
        s_mix.st[j][a] = sd_t;
        s_mix.sw[j][a] = sd_w;
        // single-precision logs: within 1e-6 of the double ones on the
        // deviations' range, far inside ln q's float error elsewhere
        c += -(double)logf(sd_t) - (double)logf(sd_w);
      }
      s_c0[j] = c;
    }
  }
  __syncthreads();
  // Two independent chains: A (thread 0) the current pose and the restraint
  // energy at the current centre of mass, B (thread 64, or thread 0 after A
  // in a one-wavefront block) the proposal; with two wavefronts they run
  // side by side.  Each computes the log-normaliser of the mixture weights
  // (log-softmax of the raw logits, float) with the same operations.
  __shared__ double s_R[2][9];  // R0, R1
  __shared__ double s_lq[2];
  const int tb = W >= 2 ? kWave : 0;
  if (tid == 0) {
    double c[3] = {0, 0, 0}, M = 0;
    for (int q = 0; q < W; ++q) {
      for (int d = 0; d < 3; ++d) c[d] += s_cp[4 * q + d];
      M += s_cp[4 * q + 3];
    }
    Frame F;
    body_frame(xr, P.frame, F);
    double R0[3][3], w0[3];
    for (int a = 0; a < 3; ++a)
      for (int b = 0; b < 3; ++b) R0[a][b] = F.R[a][b];
    log_rot(R0, w0);
    double d2 = 0.0;
    for (int d = 0; d < 3; ++d) {
      c[d] /= M;
      s_pose[d] = c[d] - L.site[d];
      s_pose[3 + d] = w0[d];
      d2 += s_pose[d] * s_pose[d];
      scom[d] = (float)c[d];
    }
    for (int a = 0; a < 3; ++a)
      for (int b = 0; b < 3; ++b) s_R[0][3 * a + b] = R0[a][b];
    // restraint energy at the current centre of mass (Eq. binding_site)
    const double ex0 = sqrt(d2) - (double)L.d0;
    s_ui0 = ex0 > 0.0 ? 0.5 * (double)L.krest * ex0 * ex0 : 0.0;
  }
  // the wavefront of lane tb: the components' weights and log-density
  // constants, one component per lane; the weights then go to every lane
  double wt[kNComp];
  if ((tid >> 6) == (tb >> 6)) {
    const float lse = mix_lse(s_mix);
    const int jj = tid - tb;
    double wj = 0.0;
    if (jj < kNComp) {
      const double lw = (double)(s_mix.lw[jj] - lse);
      wj = exp(lw);
      s_c0[jj] += lw;
    }
    for (int j = 0; j < kNComp; ++j) {
      const long long b = __double_as_longlong(wj);
      const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffffll), j);
      const int hi = __builtin_amdgcn_readlane((int)(b >> 32), j);
      wt[j] = __longlong_as_double(((long long)hi << 32) |
                                   (long long)(unsigned)lo);
    }
  }
  if (tid == tb) {
    // component by inverse CDF, then (t, omega) by Gaussian draws
    const U4 o0 = draw(seed, 0u, L.id, r, s, kPose);
    const double u = u01d(o0.x);
    double cum[kNComp], tot = 0.0;
    for (int j = 0; j < kNComp; ++j) {
      tot += wt[j];
      cum[j] = tot;
    }
    int j = 0;
    while (j < kNComp - 1 && cum[j] < u * tot) ++j;
    float z[6];
    normals3(draw(seed, 1u, L.id, r, s, kPose), z[0], z[1], z[2]);
    normals3(draw(seed, 2u, L.id, r, s, kPose), z[3], z[4], z[5]);
    double t1[3], w1[3];
    for (int d = 0; d < 3; ++d) {
      t1[d] = (double)s_mix.mt[j][d] + (double)s_mix.st[j][d] * z[d];
      w1[d] = (double)s_mix.mw[j][d] + (double)s_mix.sw[j][d] * z[3 + d];
    }
    double R1[3][3];
    rodrigues(w1, R1);
    double w1p[3];
    log_rot(R1, w1p);  // principal rotation vector of the proposal
    for (int d = 0; d < 3; ++d) {
      s_pose[6 + d] = t1[d];
      s_pose[9 + d] = w1p[d];
      st[d] = (float)(L.site[d] + t1[d]);
    }
    for (int a = 0; a < 3; ++a)
      for (int b = 0; b < 3; ++b) s_R[1][3 * a + b] = R1[a][b];
  }
  __syncthreads();
  // the two proposal densities, one term per lane: wave 0 at the current
  // pose, wave 1 (or wave 0 after that) at the proposal
  {
    const int wv = tid >> 6;
    if (W >= 2) {
      if (wv < 2) {
        const double lq = log_q_se3_wave(s_mix, s_c0, s_pose + 6 * wv,
                                         s_pose + 6 * wv + 3);
        if ((tid & 63) == 0) s_lq[wv] = lq;
      }
    } else {
      const double lq0 = log_q_se3_wave(s_mix, s_c0, s_pose, s_pose + 3);
      const double lq1 = log_q_se3_wave(s_mix, s_c0, s_pose + 6, s_pose + 9);
      if (tid == 0) {
        s_lq[0] = lq0;
        s_lq[1] = lq1;
      }
    }
  }
  if (tid == 0) {
    // x'_i = c0 + t' + R' R0^T (x_i - c): the rotation applied is R' R0^T
    for (int a = 0; a < 3; ++a)
      for (int b = 0; b < 3; ++b) {
        double v = 0.0;
        for (int q = 0; q < 3; ++q) v += s_R[1][3 * a + q] * s_R[0][3 * b + q];
        sR[3 * a + b] = (float)v;
      }
  }
  __syncthreads();
  lq_ratio = s_lq[0] - s_lq[1];
  if (tid == 0) s_ok = isfinite(lq_ratio) ? 1 : 0;
  Shared sh{};
  sh.pos = reinterpret_cast<float4*>(smem);
  sh.red = reinterpret_cast<double*>(smem + 16 * kWave * W);
  sh.com = reinterpret_cast<float*>(smem + 16 * kWave * W + 8 * W * kRedMax);
  const bool owner = tid < n;
  float x2[3] = {0.f, 0.f, 0.f}, f[3];
  if (owner) {
    float y[3];
    for (int d = 0; d < 3; ++d) y[d] = xr[3 * tid + d] - scom[d];
    for (int a = 0; a < 3; ++a)
      x2[a] = st[a] + sR[3 * a] * y[0] + sR[3 * a + 1] * y[1] + sR[3 * a + 2] * y[2];
  }
  const float m = owner ? L.mass[tid] : 0.f;
  float sc[C];
#pragma unroll
  for (int c = 0; c < C; ++c) sc[c] = owner ? L.scale[tid * C + c] : 0.f;
  float w[C];
  for (int c = 0; c < C; ++c) w[c] = L.wf[k * C + c];
  double t1e[6 + C];
  eval_block<C, W, false, true, true, false>(g, L, w, x2, m, sc, f, t1e, 0.f,
                                             0.f, sh, tid);
  const double* cp = L.comps + (size_t)r * (1 + C);
  const double ub = cp[0] - s_ui0;  // bonded energy, unchanged by the move
  double E1 = ub + t1e[3], E0 = cp[0];
  for (int c = 0; c < C; ++c) {
    E1 += L.wd[k * C + c] * t1e[4 + c];
    E0 += L.wd[k * C + c] * cp[1 + c];
  }
  __shared__ int s_acc;
  if (tid == 0) {
    const double ln_a = -L.beta[k] * (E1 - E0) + lq_ratio;
    const U4 ou = draw(seed, 3u, L.id, r, s, kPose);
    s_acc = (s_ok && isfinite(ln_a) && ln_u_below(ou.x, ln_a)) ? 1 : 0;
    P.last_ln_alpha[r] = ln_a;
    atomicAdd(&P.pose_try[k], 1ull);
    if (s_acc) atomicAdd(&P.pose_acc[k], 1ull);
  }
  __syncthreads();
  if (s_acc) {
    if (owner)
      for (int d = 0; d < 3; ++d) L.x[(size_t)r * n * 3 + 3 * tid + d] = x2[d];
    if (tid == 0) {
      double* cw = L.comps + (size_t)r * (1 + C);
      cw[0] = ub + t1e[3];
      for (int c = 0; c < C; ++c) cw[1 + c] = t1e[4 + c];
      L.fvalid[r] = 0;  // the stored start-of-trajectory forces are stale
    }
  }
  // the next run of neighbour-scheme sweeps starts from this replica's
  // state and (new or kept) components
  if (begin_next && tid == 0)
    begin_replica(L, r, k, s, *L.n_rec, L.comps + (size_t)r * (1 + C));
}

}  // namespace

// ----------------------------------------------------------------------------
// launchers
// ----------------------------------------------------------------------------
hipError_t launch_mlp_forward(const float* P, const unsigned short* WT,
                              const float* X, int B, float* out,
                              hipStream_t st) {
  if (B <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_mlp_forward, dim3((B + kFRows - 1) / kFRows),
                     dim3(kFWaves * 64), 0, st, P, WT, X, B, out);
  return hipGetLastError();
}

// one split per 4096 rows (64 at most): up to there a wavefront per tile
// takes all rows, 128 chunks, in order
int train_splits(int Bp) { return std::min(64, (Bp + 4095) / 4096); }

hipError_t launch_train_step(const TrainArgs& a, const AdamArgs& w,
                             float* split, double* loss, hipStream_t st) {
  if (a.B <= 0 || a.Bp % kKStep != 0 || a.Bp < a.B) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_train_rows, dim3(a.Bp / kFRows), dim3(kFWaves * 64), 0,
                     st, a);
  const int ns = train_splits(a.Bp);
  hipLaunchKernelGGL(k_train_weights,
                     dim3(kTileBlocks + kBiasBlocks + 1, ns), dim3(256), 0, st,
                     a, w, ns, split, loss);
  if (ns > 1)
    hipLaunchKernelGGL(k_train_splits, dim3((kNParams + 255) / 256), dim3(256),
                       0, st, w, a.WT, split, ns);
  return hipGetLastError();
}

hipError_t launch_pose_network(const MlpGroup* groups, int n_groups,
                               const LigDev* ligs, const PropDev* props,
                               const PoseTask* tasks, float* out,
                               const LigDev* fin, int n_fin,
                               int exchange_every, int sample_every,
                               uint64_t seed, hipStream_t st) {
  if (n_groups + n_fin <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_pose_network, dim3(n_groups + n_fin),
                     dim3(kFWaves * 64), 0, st, groups, n_groups, ligs, props,
                     tasks, out, fin, exchange_every, sample_every, seed);
  return hipGetLastError();
}

hipError_t launch_weights_bf16(const float* P, unsigned short* WT,
                               hipStream_t st) {
  hipLaunchKernelGGL(k_weights_bf16, dim3((kTSize + 255) / 256), dim3(256), 0,
                     st, P, WT);
  return hipGetLastError();
}

hipError_t launch_pose_features(const LigDev* lig, const PropDev* prop, int n,
                                const float* xs, int64_t N, float* feats,
                                float* poses, hipStream_t st) {
  if (N <= 0) return hipSuccess;
  const int m = feat_confs(n);
  // a launch's share: a grid of 2^32 threads or more is cut short silently
  const int64_t most = ((1ll << 24) - 1) * m;
  for (int64_t c = 0; c < N; c += most) {
    const int64_t now = N - c < most ? N - c : most;
    hipLaunchKernelGGL(k_pose_features, dim3((unsigned)((now + m - 1) / m)),
                       dim3(kFeatWaves * 64), m * feat_row(n) * 4, st, lig,
                       prop, xs + c * n * 3, now, feats + c * kNFeat,
                       poses + c * 6);
  }
  return hipGetLastError();
}

hipError_t launch_pose_move(const GridDev& g, const LigDev* ligs,
                            const PropDev* props, const PoseTask* tasks,
                            int n, const float* out, int waves, int lds,
                            uint64_t seed, bool begin_next, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  switch (g.C) {
    case 3:
      if (waves == 1)
        hipLaunchKernelGGL((k_pose_move<3, 1>), dim3(n), dim3(64), lds, st, g,
                           ligs, props, tasks, out, seed, begin_next ? 1 : 0);
      else
        hipLaunchKernelGGL((k_pose_move<3, 2>), dim3(n), dim3(128), lds, st, g,
                           ligs, props, tasks, out, seed, begin_next ? 1 : 0);
      break;
    case 5:
      if (waves == 1)
        hipLaunchKernelGGL((k_pose_move<5, 1>), dim3(n), dim3(64), lds, st, g,
                           ligs, props, tasks, out, seed, begin_next ? 1 : 0);
      else
        hipLaunchKernelGGL((k_pose_move<5, 2>), dim3(n), dim3(128), lds, st, g,
                           ligs, props, tasks, out, seed, begin_next ? 1 : 0);
      break;
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace bpmf
