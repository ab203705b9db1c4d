// MBAR on the device in double precision (Shirts & Chodera 2008; the paper
// estimates f_BC,L and f_CD' with it, Methodology "Estimation").
//
// The free energies minimise the convex function
//   F(f) = sum_n ln sum_k N_k exp(f_k - u_kn) - sum_i N_i f_i,   f_0 = 0,
// whose gradient is g_i = N_i (sum_n W_ni - 1) and Hessian
//   H_ij = N_i delta_ij sum_n W_ni - N_i N_j sum_n W_ni W_nj,
// W_ni = exp(f_i - u_in) / sum_k N_k exp(f_k - u_kn).  Newton steps solve the
// gauge-fixed system; var(f_k - f_0) = (H~^-1)_kk - 1/N_k - 1/N_0.
//
// Every kernel serves a list of independent problems (one per ligand):
// blockIdx.y picks the problem, and each problem keeps its own block count
// for every grid-wide loop, so a problem's arithmetic -- and its result --
// is the same whether it is solved alone or in a batch.  All reductions run
// over a fixed block grid in a fixed order, so results do not depend on
// scheduling either.
//
// The iteration's decisions are taken on the device (MbarState), and one pass
// over u_kn gives both the objective at a point and the sums of the Newton
// step from it, so a round is four launches -- sums, their reduction, the
// decision with the next step, the rare fixed-point values -- which the host
// enqueues without waiting for their outcome (86 states x 64500 samples, 18
// Newton steps and 43 objectives: 11.6 ms with separate passes and a host
// decision after every step, 1.9 ms so; 32 problems of 32 x 6400: 6.9 and
// 2.1 ms).
#include <hip/hip_runtime.h>
#include <math.h>

#include <algorithm>

#include "device.h"
#include "internal.h"

namespace bpmf {

namespace {

constexpr int kT = 256;
typedef double f64x4 __attribute__((ext_vector_type(4)));
// two doubles of a matrix row: rows start at any multiple of 8 bytes
typedef double f64x2u __attribute__((ext_vector_type(2), aligned(8)));

template <int T>
__device__ __forceinline__ double block_sum(double v, double* red) {
  red[threadIdx.x] = v;
  __syncthreads();
#pragma unroll
  for (int s = T / 2; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
    __syncthreads();
  }
  const double r = red[0];
  __syncthreads();
  return r;
}

template <int T>
__device__ __forceinline__ double block_max(double v, double* red) {
  red[threadIdx.x] = v;
  __syncthreads();
#pragma unroll
  for (int s = T / 2; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s)
      red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + s]);
    __syncthreads();
  }
  const double r = red[0];
  __syncthreads();
  return r;
}

// wavefront maximum of non-negative values (lanes a step does not reach
// receive 0; the result is in lane 63), and sums and maxima over the 16 lanes
// of a row: every lane of the row gets the result
__device__ __forceinline__ double wave_max0(double v) {
  v = fmax(v, dpp_d<0xB1, 0xf>(v));
  v = fmax(v, dpp_d<0x4E, 0xf>(v));
  v = fmax(v, dpp_d<0x141, 0xf>(v));
  v = fmax(v, dpp_d<0x140, 0xf>(v));
  v = fmax(v, dpp_d<0x142, 0xa>(v));
  v = fmax(v, dpp_d<0x143, 0xc>(v));
  return v;
}
__device__ __forceinline__ double row_max(double v) {
  v = fmax(v, dpp_d<0xB1, 0xf>(v));
  v = fmax(v, dpp_d<0x4E, 0xf>(v));
  v = fmax(v, dpp_d<0x141, 0xf>(v));
  return fmax(v, dpp_d<0x140, 0xf>(v));
}
__device__ __forceinline__ double row_sum(double v) {
  v += dpp_d<0xB1, 0xf>(v);
  v += dpp_d<0x4E, 0xf>(v);
  v += dpp_d<0x141, 0xf>(v);
  return v + dpp_d<0x140, 0xf>(v);
}

// 1 / x by the hardware's estimate and two Newton steps (x neither denormal
// nor infinite, or of no use anyway)
__device__ __forceinline__ double near_rcp(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = fma(r, fma(-x, r, 1.0), r);
  return fma(r, fma(-x, r, 1.0), r);
}

// the point the phase asks the objective at, state k of K: the trial, the
// fixed-point update (less its first value), or f at the start
__device__ __forceinline__ double point(const MbarProb& p, int phase, int k) {
  const double* src = phase == kMbarSearch  ? p.ftry
                      : phase == kMbarFixed ? p.step
                                            : p.f;
  return src[k] - (phase == kMbarFixed ? src[0] : 0.0);
}

// One pass over u_kn at the phase's point f: logD_n = ln sum_k exp(logN_k +
// f_k - u_kn), and over the block's samples partial[b] = [sum logD, 15 x 0 |
// colsum_i (16 NT) | tiles of M = E E^T], E_in = N_i W_in = exp(logN_i + f_i
// - u_in - logD_n), K <= 16 NT (rows past K zero).  M is symmetric: its 16 x
// 16 tiles (R, C), C <= R, in the order R (R + 1) / 2 + C.  A wavefront takes
// 4 S samples at a time, the next ones' energies loading meanwhile: lane l
// holds row l % 16 of every 16-row fragment for the samples S (l / 16) ..
// + S - 1.  A sample's states are then one row of 16 lanes (DPP maxima and
// sums), every exponential serves both logD and E, and the fragments are the
// operands of S 16x16x4 double MFMAs for both factors as they are; u_kn is
// read once.

// energies of a chunk: samples n0 .. n0 + S - 1 of row 16 R + i (clamped to
// the last state and sample)
template <int NT, int S>
__device__ __forceinline__ void load_energies(const double* __restrict__ ukn,
                                              int K, int64_t N, int64_t ld,
                                              int i, int64_t n0, bool whole,
                                              double (&w)[NT][S]) {
#pragma unroll
  for (int R = 0; R < NT; ++R) {
    const int k = 16 * R + i < K ? 16 * R + i : K - 1;
    const double* u = ukn + (size_t)k * ld;
    if (whole) {
#pragma unroll
      for (int s = 0; s < S; s += 2) {
        const f64x2u uv = *(const f64x2u*)(u + n0 + s);
        w[R][s] = uv.x;
        w[R][s + 1] = uv.y;
      }
    } else {
#pragma unroll
      for (int s = 0; s < S; ++s) w[R][s] = u[n0 + s < N ? n0 + s : N - 1];
    }
  }
}

// E of a chunk from its energies `u`, samples n0 + s: logD stored, col and obj
// added to
template <int NT, int S>
__device__ __forceinline__ void weights(const double (&u)[NT][S],
                                        const double (&ak)[NT], int K,
                                        int64_t N, int64_t n0, int i,
                                        double* __restrict__ logD,
                                        double (&w)[NT][S], double (&col)[NT],
                                        double& obj) {
  double m[S], t[S];
#pragma unroll
  for (int s = 0; s < S; ++s) {
    // past K a lane repeats state K - 1's energy: kept out of every sum
    m[s] = -INFINITY;
#pragma unroll
    for (int R = 0; R < NT; ++R) {
      w[R][s] = ak[R] - u[R][s];
      if (16 * (R + 1) <= K || 16 * R + i < K) m[s] = fmax(m[s], w[R][s]);
    }
    m[s] = row_max(m[s]);
  }
#pragma unroll
  for (int s = 0; s < S; ++s) {
    t[s] = 0.0;
#pragma unroll
    for (int R = 0; R < NT; ++R) {
      const double e = exp(w[R][s] - m[s]);
      w[R][s] = 16 * (R + 1) <= K || 16 * R + i < K ? e : 0.0;
      t[s] += w[R][s];
    }
    t[s] = row_sum(t[s]);
  }
  // lane s of a row takes sample s's logarithm
  {
    double ms = m[0], ts = t[0];
#pragma unroll
    for (int s = 1; s < S; ++s)
      if (i == s) {
        ms = m[s];
        ts = t[s];
      }
    const double l = ms + log(ts);
    if (i < S && n0 + i < N) {
      logD[n0 + i] = l;
      obj += l;
    }
  }
#pragma unroll
  for (int s = 0; s < S; ++s) {
    // correctly rounded: an error with a bias would enter every sample's sum
    // of weights alike, which the Hessian's smallest eigenvalue magnifies
    // about a thousand times in the variances
    const double rt = n0 + s < N ? 1.0 / t[s] : 0.0;
#pragma unroll
    for (int R = 0; R < NT; ++R) {
      w[R][s] *= rt;
      col[R] += w[R][s];
    }
  }
}

// column sums and objective of a block of kW wavefronts, in order
template <int NT, int kW>
__device__ __forceinline__ void put_sums(double* out, double (&col)[NT],
                                         double obj,
                                         double (&csum)[kW][16 * NT],
                                         double (&osum)[kW]) {
  const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x >> 6;
  obj = wave_sum(obj);
  if (lane == 0) osum[wv] = obj;
#pragma unroll
  for (int R = 0; R < NT; ++R) {
    double c = col[R];
    c += __shfl_xor(c, 16);
    c += __shfl_xor(c, 32);
    if (lane < 16) csum[wv][16 * R + lane] = c;
  }
  __syncthreads();
  for (int k = threadIdx.x; k < 16 * NT; k += kW * kWave) {
    double v = 0.0;
#pragma unroll
    for (int x = 0; x < kW; ++x) v += csum[x][k];
    out[kMbarHead + k] = v;
  }
  if (threadIdx.x < kMbarHead) {
    double v = 0.0;
    if (threadIdx.x == 0)
#pragma unroll
      for (int x = 0; x < kW; ++x) v += osum[x];
    out[threadIdx.x] = v;
  }
}

// Up to 48 states: a wavefront keeps all of its tiles and multiplies its own
// fragments straight from registers (S = 4: whole 128-byte lines of u_kn).
// Bound by latency -- the table, u_kn, the sums' chain -- with two to four
// wavefronts a SIMD; 32 problems of 32 x 6400: 13.4 us for the objective and
// 16.6 us for the sums (W staged in LDS, FP64 FMAs on all of M) as two passes,
// 21 us so.
template <int NT>
__global__ __launch_bounds__(kT) void k_sums(const MbarProb* __restrict__ P) {
  constexpr int kTiles = NT * (NT + 1) / 2, S = 4;
  const MbarProb& p = P[blockIdx.y];
  const int phase = p.state.phase;
  if ((int)blockIdx.x >= p.nb || phase == kMbarDone) return;
  constexpr int kW = kT / kWave;       // wavefronts
  constexpr int kG = 4;                // tiles summed at a time at the end
  __shared__ double sum[kW][kG][256];
  __shared__ double csum[kW][16 * NT], osum[kW];
  const int K = p.K;
  const int64_t N = p.N, ld = p.ld;
  const double* __restrict__ ukn = p.ukn;
  const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x >> 6;
  const int i = lane & 15, kk = lane >> 4;
  f64x4 acc[kTiles];
  double col[NT], ak[NT], obj = 0.0;  // a_k = logN_k + f_k
#pragma unroll
  for (int q = 0; q < kTiles; ++q) acc[q] = f64x4{0.0, 0.0, 0.0, 0.0};
  const int64_t n_chunks = (N + 4 * S - 1) / (4 * S);
  const int64_t step = (int64_t)p.nb * kW;
  int64_t ch = (int64_t)blockIdx.x * kW + wv;
  double next[NT][S];
  if (ch < n_chunks)
    load_energies<NT, S>(ukn, K, N, ld, i, 4 * S * ch + S * kk,
                         4 * S * (ch + 1) <= N, next);
#pragma unroll
  for (int R = 0; R < NT; ++R) {
    const int k = 16 * R + i;
    col[R] = 0.0;
    ak[R] = k < K ? p.logN[k] + point(p, phase, k) : 0.0;
  }
  for (; ch < n_chunks; ch += step) {
    double u[NT][S], w[NT][S];
#pragma unroll
    for (int R = 0; R < NT; ++R)
#pragma unroll
      for (int s = 0; s < S; ++s) u[R][s] = next[R][s];
    if (ch + step < n_chunks)
      load_energies<NT, S>(ukn, K, N, ld, i, 4 * S * (ch + step) + S * kk,
                           4 * S * (ch + step + 1) <= N, next);
    weights<NT, S>(u, ak, K, N, 4 * S * ch + S * kk, i, p.logD, w, col, obj);
#pragma unroll
    for (int s = 0; s < S; ++s)
#pragma unroll
      for (int R = 0; R < NT; ++R)
#pragma unroll
        for (int C = 0; C <= R; ++C)
          acc[R * (R + 1) / 2 + C] = __builtin_amdgcn_mfma_f64_16x16x4f64(
              w[R][s], w[C][s], acc[R * (R + 1) / 2 + C], 0, 0, 0);
  }
  // the wavefronts' sums, in order; a lane holds rows 4 q + l / 16 of column
  // l % 16 of a tile
  double* out = p.partial + (size_t)blockIdx.x * mbar_width(K);
  put_sums<NT, kW>(out, col, obj, csum, osum);
  double* tiles = out + kMbarHead + 16 * NT;
#pragma unroll
  for (int t0 = 0; t0 < kTiles; t0 += kG) {
    if (t0 > 0) __syncthreads();
#pragma unroll
    for (int q = 0; q < kG; ++q)
      if (t0 + q < kTiles)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          sum[wv][q][(4 * r + kk) * 16 + i] = acc[t0 + q][r];
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kG; ++q)
      if (t0 + q < kTiles) {
        double v = 0.0;
#pragma unroll
        for (int x = 0; x < kW; ++x) v += sum[x][q][threadIdx.x];
        tiles[256 * (t0 + q) + threadIdx.x] = v;
      }
  }
}

// 49 states and more: all tiles of a wavefront would fill its registers and
// leave one wavefront a SIMD, whose exponentials and products could not
// overlap.  Eight wavefronts share their fragments through LDS instead (lane
// by lane as the MFMA wants them, two buffers) and each multiplies an eighth
// of the tiles over all of them; of the two wavefronts on a SIMD one forms
// the next fragments while the other multiplies the last.  Bound by the
// exponentials and the FP64 matrix rate side by side; 86 x 64500 (21 tiles):
// 31 us for the objective and 105 us for the sums as two passes, 41 us in one
// with the tiles in registers, 37 us so (12 us of it the launch, the table's
// latency and the partial sums' 11 MB).
constexpr int kWideT = 512;
template <int NT>
__global__ __launch_bounds__(kWideT) void k_sums_wide(
    const MbarProb* __restrict__ P) {
  constexpr int kTiles = NT * (NT + 1) / 2, S = 2, kW = kWideT / kWave;
  constexpr int kMine = (kTiles + kW - 1) / kW;
  const MbarProb& p = P[blockIdx.y];
  const int phase = p.state.phase;
  if ((int)blockIdx.x >= p.nb || phase == kMbarDone) return;
  __shared__ double E[2][kW][S][NT][kWave];
  __shared__ double csum[kW][16 * NT], osum[kW];
  const int K = p.K;
  const int64_t N = p.N, ld = p.ld;
  const double* __restrict__ ukn = p.ukn;
  const int lane = threadIdx.x & (kWave - 1);
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int i = lane & 15, kk = lane >> 4;
  f64x4 acc[kMine];
  double col[NT], ak[NT], obj = 0.0;  // a_k = logN_k + f_k
  int tr[kMine], tc[kMine];           // rows and columns of the tiles
#pragma unroll
  for (int q = 0; q < kMine; ++q) {
    acc[q] = f64x4{0.0, 0.0, 0.0, 0.0};
    // a wavefront without a last tile repeats tile 0 (not written): its
    // product has no branches, so the LDS reads run ahead of the MFMAs
    const int t = wv + kW * q < kTiles ? wv + kW * q : 0;
    int R = 0;
    while ((R + 1) * (R + 2) / 2 <= t) ++R;
    tr[q] = R;
    tc[q] = t - R * (R + 1) / 2;
  }
  // iteration j of the block: chunk 8 (j nb + block) + wavefront
  const int64_t n_iter = (N + 4 * S * kW - 1) / (4 * S * kW);
  int64_t it = blockIdx.x;
  auto first = [&](int64_t j) { return 4 * S * (kW * j + wv) + S * kk; };
  auto whole = [&](int64_t j) { return 4 * S * (kW * j + wv + 1) <= N; };
  double next[NT][S];
  load_energies<NT, S>(ukn, K, N, ld, i, first(it), whole(it), next);
#pragma unroll
  for (int R = 0; R < NT; ++R) {
    const int k = 16 * R + i;
    col[R] = 0.0;
    ak[R] = k < K ? p.logN[k] + point(p, phase, k) : 0.0;
  }
  // fragments of iteration j into buffer b; the energies of the one after it
  auto form = [&](int64_t j, int b) {
    double u[NT][S], w[NT][S];
#pragma unroll
    for (int R = 0; R < NT; ++R)
#pragma unroll
      for (int s = 0; s < S; ++s) u[R][s] = next[R][s];
    if (j + p.nb < n_iter)
      load_energies<NT, S>(ukn, K, N, ld, i, first(j + p.nb), whole(j + p.nb),
                           next);
    weights<NT, S>(u, ak, K, N, first(j), i, p.logD, w, col, obj);
#pragma unroll
    for (int s = 0; s < S; ++s)
#pragma unroll
      for (int R = 0; R < NT; ++R) E[b][wv][s][R][lane] = w[R][s];
  };
  auto multiply = [&](int b) {
#pragma unroll 4
    for (int v = 0; v < kW; ++v)
#pragma unroll
      for (int s = 0; s < S; ++s)
#pragma unroll
        for (int q = 0; q < kMine; ++q)
          acc[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(
              E[b][v][s][tr[q]][lane], E[b][v][s][tc[q]][lane], acc[q], 0, 0,
              0);
  };
  form(it, 0);
  __syncthreads();
  for (int b = 0; it < n_iter; it += p.nb, b ^= 1) {
    const bool more = it + p.nb < n_iter;
    if (wv < kW / 2) {
      if (more) form(it + p.nb, b ^ 1);
      multiply(b);
    } else {
      multiply(b);
      if (more) form(it + p.nb, b ^ 1);
    }
    __syncthreads();
  }
  double* out = p.partial + (size_t)blockIdx.x * mbar_width(K);
  put_sums<NT, kW>(out, col, obj, csum, osum);
  double* tiles = out + kMbarHead + 16 * NT;
#pragma unroll
  for (int q = 0; q < kMine; ++q)
    if (wv + kW * q < kTiles)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        tiles[256 * (wv + kW * q) + (4 * r + kk) * 16 + i] = acc[q][r];
}

// red[e] = sum over blocks of partial[b][e]: kRedG interleaved runs of blocks,
// each in order, then the runs in order (many short runs keep enough loads in
// flight)
constexpr int kRedE = 64, kRedG = 16;
__global__ __launch_bounds__(kRedE * kRedG) void k_reduce_partials(
    const MbarProb* __restrict__ P) {
  const MbarProb& p = P[blockIdx.y];
  const int width = mbar_width(p.K);
  const int x = threadIdx.x & (kRedE - 1), g = threadIdx.x / kRedE;
  const int e = blockIdx.x * kRedE + x;
  if ((int)blockIdx.x * kRedE >= width || p.state.phase == kMbarDone) return;
  __shared__ double part[kRedG][kRedE];
  const double* __restrict__ src = p.partial;
  const int nb = p.nb;
  double s = 0.0;
  if (e < width) {
#pragma unroll 8
    for (int b = g; b < nb; b += kRedG) s += src[(size_t)b * width + e];
  }
  part[g][x] = s;
  __syncthreads();
  if (g == 0 && e < width) {
#pragma unroll
    for (int q = 1; q < kRedG; ++q) s += part[q][x];
    p.red[e] = s;
  }
}

// iteration bookkeeping after a move of size `change`: true when it was the
// last one
__device__ __forceinline__ bool finish_move(MbarState& s, double change,
                                            double tol, int max_iter) {
  if (!(change >= tol)) {
    s.n_iter = s.it;
    return true;
  }
  if (s.it >= max_iter) {
    s.n_iter = max_iter;
    return true;
  }
  ++s.it;
  return false;
}

// What follows from the sums at the phase's point (one block per problem): a
// trial is accepted or halved, a fixed-point update taken; then, at an
// accepted point, the Newton step and the next trial, or, after the last
// move, the variances.
// The gauge-fixed system H~ x = -g~ has m = K - 1 unknowns.  [H~ | -g~] sits
// in registers: thread (y, x) of a 16 x 16 block holds the rows y + 16 a and
// columns x + 16 b, a, b < NB, 16 NB >= K.  Step q subtracts multiples of row
// q from the rows below it; column q of those rows, then zero, takes the
// multiplier instead, so the rows end as the unit lower triangle's inverse Li
// (left of the diagonal), the pivots D (on it) and y = Li (-g~): x = Li^T
// D^-1 y and diag(H~^-1)_c = sum_r Li_rc^2 / D_r need no back substitution.
// Row and column q reach the block through LDS, one barrier a step.  Bound by
// the steps' chain (LDS write, barrier, read, reciprocal, FMA); 85 unknowns:
// 385 us by Gauss-Jordan elimination in LDS (1179 us with the inverse, in
// global memory), 52 us so; 31 unknowns: 36 us and 12 us.
template <int NB>
__global__ __launch_bounds__(kT) void k_step(
    MbarProb* P, double tol,
    int max_iter, int* n_done, int n_all, volatile int* host_done) {
  const MbarProb& p = P[blockIdx.y];
  if (p.state.phase == kMbarDone) return;
  constexpr int kC = 16 * NB;
  __shared__ double rowq[2][kC], colq[2][kC], gsh[kC];
  __shared__ double ys[kC], ds[kC], xs[16][kC], is[16][kC];
  __shared__ double wred[2][kT / kWave];
  const int K = p.K, m = K - 1;
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid >> 6;
  const int tx = tid & 15, ty = tid >> 4;
  const double* __restrict__ red = p.red;
  const double* __restrict__ Nk = p.Nk;
  // every thread follows the decision on its own copy of the state (the
  // barrier after the sums stands between these reads and the last writes)
  MbarState s = p.state;
  const int was = s.phase;
  const double* cs = red + kMbarHead;  // column sums N_i sum_n W_ni
  // objective sum_n logD_n - sum_k N_k f_k; change of a fixed-point update
  {
    double s2 = 0.0, ch = 0.0;
    const double fk = tid < K ? point(p, was, tid) : 0.0;
    if (tid < K) {
      s2 = Nk[tid] * fk;
      ch = fabs(fk - p.f[tid]);
    }
    const double w2 = wave_sum(s2), wc = wave_max0(ch);
    if (lane == kWave - 1) {
      wred[0][wv] = w2;
      wred[1][wv] = wc;
    }
    if (tid < K) gsh[tid] = cs[tid] - Nk[tid];
    __syncthreads();
    const double sf = wred[0][0] + wred[0][1];  // K <= 128: two wavefronts
    const double change = fmax(wred[1][0], wred[1][1]);
    const double F = red[0] - sf;
    bool last = false;
    if (was == kMbarStart) {
      s.Fcur = F;
    } else if (was == kMbarFixed) {
      s.Fcur = F;
      last = finish_move(s, change, tol, max_iter);
    } else {
      bool take = F <= s.Fcur + 1e-4 * s.t * s.gs + 1e-13 * fabs(s.Fcur) ||
                  s.t * s.maxstep < tol;
      if (!take) {
        s.t *= 0.5;
        // after 60 trials the last one is taken anyway
        take = ++s.ls >= 60;
      }
      if (!take) {
        if (tid < K) p.ftry[tid] = p.f[tid] + s.t * p.step[tid];
        if (tid == 0) P[blockIdx.y].state = s;
        return;
      }
      s.Fcur = F;
      s.trust = s.t * s.maxstep;
      last = finish_move(s, s.trust, tol, max_iter);
    }
    if (tid < K && was != kMbarStart) p.f[tid] = fk;
    s.phase = last ? kMbarDone : kMbarSearch;
  }
  double A[NB][NB], dm = 0.0;
  const double* tiles = cs + 16 * mbar_tiles(K);
#pragma unroll
  for (int a = 0; a < NB; ++a)
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const int r = ty + 16 * a, c = tx + 16 * b;
      double v = 0.0;
      if (r < m && c < m) {
        const int i = r + 1, j = c + 1, hi = i > j ? i : j, lo = i > j ? j : i;
        const int R = hi >> 4, C = lo >> 4;
        v = -tiles[256 * (R * (R + 1) / 2 + C) + (hi & 15) * 16 + (lo & 15)];
        if (i == j) {
          v += cs[i];
          dm = fmax(dm, v);
        }
      } else if (r < m && c == m) {
        v = -gsh[r + 1];
      }
      A[a][b] = v;
    }
  dm = wave_max0(dm);
  __syncthreads();  // wred's readers are done
  if (lane == kWave - 1) wred[0][wv] = dm;
  __syncthreads();
  dm = fmax(fmax(wred[0][0], wred[0][1]), fmax(wred[0][2], wred[0][3]));
  // a pivot below 1e-13 of the largest diagonal entry marks the system as
  // not numerically positive definite (a fixed-point step follows instead)
  const double pmin = 1e-13 * dm;
  bool bad = false;
  int buf = 0;
#pragma unroll
  for (int aq = 0; aq < NB; ++aq)
    for (int tq = 0; tq < 16; ++tq, buf ^= 1) {
      const int q = 16 * aq + tq;
      if (q >= m) break;
      if (ty == tq)
#pragma unroll
        for (int b = 0; b < NB; ++b) rowq[buf][tx + 16 * b] = A[aq][b];
      if (tx == tq)
#pragma unroll
        for (int a = aq; a < NB; ++a) colq[buf][ty + 16 * a] = A[a][aq];
      __syncthreads();
      const double piv = rowq[buf][q];
      bad = bad || !(piv > pmin);
      const double ip = near_rcp(piv);
      double rc[NB];
#pragma unroll
      for (int b = 0; b < NB; ++b) rc[b] = rowq[buf][tx + 16 * b];
#pragma unroll
      for (int a = aq; a < NB; ++a) {
        // rows up to q in its own 16 stay as they are
        const bool below = a > aq || ty > tq;
        const double f = below ? colq[buf][ty + 16 * a] * ip : 0.0;
#pragma unroll
        for (int b = 0; b < NB; ++b) A[a][b] = fma(-f, rc[b], A[a][b]);
        if (below && tx == tq) A[a][aq] = -f;
      }
    }
  // x and the inverse's diagonal: a thread's rows, then the 16 threads of a
  // column, in order
#pragma unroll
  for (int a = 0; a < NB; ++a)
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const int r = ty + 16 * a, c = tx + 16 * b;
      if (c == m) ys[r] = A[a][b];
      if (c == r) ds[r] = A[a][b];
    }
  __syncthreads();
  {
    double x[NB], iv[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) x[b] = iv[b] = 0.0;
#pragma unroll
    for (int a = 0; a < NB; ++a) {
      const int r = ty + 16 * a;
      if (r < m) {
        const double iD = 1.0 / ds[r], y = ys[r];
#pragma unroll
        for (int b = 0; b < NB; ++b) {
          const int c = tx + 16 * b;
          const double li = c < r ? A[a][b] : c == r ? 1.0 : 0.0;
          x[b] = fma(li * iD, y, x[b]);
          iv[b] = fma(li * iD, li, iv[b]);
        }
      }
    }
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      xs[ty][tx + 16 * b] = x[b];
      is[ty][tx + 16 * b] = iv[b];
    }
  }
  __syncthreads();
  double xv = 0.0, vv = 0.0;  // one unknown a thread
  const bool act = tid < m;
  if (act)
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      xv += xs[q][tid];
      vv += is[q][tid];
    }
  if (s.phase == kMbarDone) {
    if (act)
      p.var[tid + 1] =
          bad ? INFINITY : vv - 1.0 / Nk[tid + 1] - 1.0 / Nk[0];
    if (tid == 0) {
      p.var[0] = 0.0;
      *p.iter = (double)s.n_iter;
      P[blockIdx.y].state = s;
      // the last problem of the call tells the host
      if (atomicAdd(n_done, 1) + 1 == n_all) {
        __threadfence_system();
        *host_done = 1;
      }
    }
    return;
  }
  if (bad) {
    s.phase = kMbarFixed;
    if (tid == 0) P[blockIdx.y].state = s;
    return;
  }
  // largest step and slope
  const double wm = wave_max0(act ? fabs(xv) : 0.0);
  const double wg = wave_sum(act ? gsh[tid + 1] * xv : 0.0);
  if (lane == kWave - 1) {
    wred[0][wv] = wm;
    wred[1][wv] = wg;
  }
  __syncthreads();
  s.maxstep = fmax(wred[0][0], wred[0][1]);
  s.gs = wred[1][0] + wred[1][1];
  // while accepted moves are large the first trial moves no component by
  // more than twice the last one
  s.t = s.trust >= 1.0 ? fmin(1.0, 2.0 * s.trust / s.maxstep) : 1.0;
  s.ls = 0;
  if (act) {
    p.step[tid + 1] = xv;
    p.ftry[tid + 1] = p.f[tid + 1] + s.t * xv;
  }
  if (tid == 0) {
    p.step[0] = 0.0;
    p.ftry[0] = p.f[0];
    P[blockIdx.y].state = s;
  }
}

// self-consistent update step_i = -ln sum_n exp(-u_in - logD_n), one block
// per state (logD current for f), for the problems whose Newton step failed
constexpr int kSelfT = 1024;
__global__ __launch_bounds__(kSelfT) void k_self_consistent(
    const MbarProb* __restrict__ P) {
  const MbarProb& p = P[blockIdx.y];
  const int i = blockIdx.x;
  if (i >= p.K || p.state.phase != kMbarFixed) return;
  __shared__ double red[kSelfT];
  const int64_t N = p.N;
  const double* __restrict__ row = p.ukn + (size_t)i * p.ld;
  const double* __restrict__ logD = p.logD;
  double m = -INFINITY;
#pragma unroll 4
  for (int64_t n = threadIdx.x; n < N; n += kSelfT)
    m = fmax(m, -row[n] - logD[n]);
  const double M = block_max<kSelfT>(m, red);
  double acc = 0.0;
#pragma unroll 4
  for (int64_t n = threadIdx.x; n < N; n += kSelfT)
    acc += exp(-row[n] - logD[n] - M);
  const double s = block_sum<kSelfT>(acc, red);
  if (threadIdx.x == 0) p.step[i] = -(M + log(s));
}

}  // namespace

// Few states: two 16-sample chunks per wavefront where that leaves at most
// 256 blocks, since a block's partial sums are as large as its share of a
// small problem's u_kn (32 problems of 32 x 6400: 1, 2, 3, 4, 6 and 8 chunks
// give 21.6, 21.0, 21.5, 23.3, 25.1 and 25.5 us).  Many: a block a CU, each
// iteration 64 samples.  With these, calls of 1 to 32 problems of 2 to 128
// states and 1 to 800 samples a state take 1/2.3 to 1/23 of the time of the
// separate passes with a host decision each, the fewest where 32 problems of 17
// states have 800.
int mbar_blocks(int K, int64_t N) {
  const int64_t per = mbar_tiles(K) <= kMbarNarrow ? 128 : 64;
  return (int)std::min<int64_t>(256, (N + per - 1) / per);
}

hipError_t mbar_sums(MbarProb* P, int n, int nt, int max_blocks,
                     hipStream_t st) {
  if (n == 0) return hipSuccess;
  const dim3 grid(max_blocks, n);
#define BPMF_SUMS(NT_)                                               \
  case NT_:                                                          \
    hipLaunchKernelGGL(k_sums<NT_>, grid, dim3(kT), 0, st, P);       \
    break
#define BPMF_SUMS_WIDE(NT_)                                            \
  case NT_:                                                            \
    hipLaunchKernelGGL(k_sums_wide<NT_>, grid, dim3(kWideT), 0, st, P); \
    break
  switch (nt) {
    BPMF_SUMS(1);
    BPMF_SUMS(2);
    BPMF_SUMS(3);
    BPMF_SUMS_WIDE(4);
    BPMF_SUMS_WIDE(5);
    BPMF_SUMS_WIDE(6);
    BPMF_SUMS_WIDE(7);
    BPMF_SUMS_WIDE(8);
    default: return hipErrorInvalidValue;
  }
#undef BPMF_SUMS
#undef BPMF_SUMS_WIDE
  return hipGetLastError();
}

hipError_t mbar_reduce(MbarProb* P, int n, int max_K,
                       hipStream_t st) {
  const int width = mbar_width(max_K);
  hipLaunchKernelGGL(k_reduce_partials, dim3((width + kRedE - 1) / kRedE, n),
                     dim3(kRedE * kRedG), 0, st, P);
  return hipGetLastError();
}

hipError_t mbar_step(MbarProb* P, int n, int nt,
                     double tol, int max_iter, int* n_done, int n_all,
                     volatile int* host_done, hipStream_t st) {
  if (n == 0) return hipSuccess;
#define BPMF_STEP(NB_)                                                     \
  hipLaunchKernelGGL(k_step<NB_>, dim3(1, n), dim3(kT), 0, st, P, tol, \
                     max_iter, n_done, n_all, host_done)
  if (nt <= 2)
    BPMF_STEP(2);
  else if (nt <= 4)
    BPMF_STEP(4);
  else if (nt <= 6)
    BPMF_STEP(6);
  else
    BPMF_STEP(8);
#undef BPMF_STEP
  return hipGetLastError();
}

hipError_t mbar_self_consistent(MbarProb* P, int n,
                                int max_K, hipStream_t st) {
  hipLaunchKernelGGL(k_self_consistent, dim3(max_K, n), dim3(kSelfT), 0, st, P);
  return hipGetLastError();
}

}  // namespace bpmf
