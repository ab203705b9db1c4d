// gfx950 kernels of the BPMF sampling hot path: HMC sweep, replica exchange,
// sample recording, per-sample energy components, u_kn expansion, and the
// exposed energy/force and grid evaluators.
#include <hip/hip_runtime.h>
#include <math.h>

#include "deferred.h"
#include "device.h"
#include "internal.h"

namespace bpmf {

namespace {

// Dynamic LDS of a W-wave block: positions (64 W float4), per-wave partial
// sums, centre-of-mass partials, n_acc x 3 fixed-point force accumulators,
// then the ligand's topology (staged once per launch).
template <int W, bool SYNC = true>
__device__ __forceinline__ Shared carve(unsigned char* raw, const LigDev& L,
                                        int n_acc, int tid) {
  Shared sh;
  sh.pos = reinterpret_cast<float4*>(raw);
  sh.red = reinterpret_cast<double*>(raw + 16 * kWave * W);
  sh.com = reinterpret_cast<float*>(raw + 16 * kWave * W +
                                    8 * W * kRedMax);
  // offset arithmetic on the LDS base keeps the pointers in LDS space;
  // force accumulators exist when n_acc > 0 (force-evaluating kernels)
  const int acc0 = 16 * kWave * W + 8 * W * kRedMax + 16 * W;
  sh.sl = Slots{(lds_u32*)(raw + acc0), 3 * n_acc};
  for (int i = tid; i < kAccCopies * 3 * n_acc; i += W * kWave)
    sh.sl.acc[i] = 0u;
  stage_topology(L, raw + acc0 + acc_lds_bytes(n_acc), sh, tid, W * kWave);
  // SYNC false: the caller issues more work before its own barrier
  if (SYNC) __syncthreads();
  return sh;
}

// block-wide double sums of two per-thread floats (fixed order); W0: the
// sums are needed (and formed) in wavefront 0 only, 0 elsewhere
template <int W, bool W0 = false>
__device__ __forceinline__ void block_sum2(float a, float b, double* buf,
                                           int tid, double& sa, double& sb) {
  const double wa = wave_sum((double)a), wb = wave_sum((double)b);
  if ((tid & (kWave - 1)) == 0) {
    buf[2 * (tid >> 6)] = wa;
    buf[2 * (tid >> 6) + 1] = wb;
  }
  block_sync();
  sa = 0.0;
  sb = 0.0;
  if (W0 && tid >= kWave) return;
#pragma unroll
  for (int q = 0; q < W; ++q) {
    sa += buf[2 * q];
    sb += buf[2 * q + 1];
  }
}

// ----------------------------------------------------------------------------
// replica exchange (Eq. repXacc), state labels swapped
// ----------------------------------------------------------------------------
#pragma clang fp contract(off)
__device__ double state_energy(const LigDev& L, int k, int rep) {
  const double* cp = L.comps + (size_t)rep * (1 + L.C);
  double E = cp[0];
  for (int c = 0; c < L.C; ++c) E += L.wd[k * L.C + c] * cp[1 + c];
  return E;
}

__device__ bool attempt_pair(const LigDev& L, int a, int b, int sep,
                             uint64_t sweep, int sub, uint64_t seed) {
  const int ra = L.replica_of_state[a], rb = L.replica_of_state[b];
  const double ba = L.beta[a], bb = L.beta[b];
  const double delta =
      ba * (state_energy(L, a, rb) - state_energy(L, a, ra)) +
      bb * (state_energy(L, b, ra) - state_energy(L, b, rb));
  const uint32_t purpose = (uint32_t)kExchange | ((uint32_t)sep << 8);
  const U4 o = draw(seed, (uint32_t)a, L.id, sub, sweep, purpose);
  const double lnu = log(u01d(o.x));
  const bool ok = isfinite(delta) && (lnu < -delta);
  if (sep == 1) atomicAdd(&L.ex_try[a], 1ull);
  if (ok) {
    L.replica_of_state[a] = rb;
    L.replica_of_state[b] = ra;
    L.state_of_replica[ra] = b;
    L.state_of_replica[rb] = a;
    if (sep == 1) atomicAdd(&L.ex_acc[a], 1ull);
  }
  return ok;
}

// The all-separations sweep with the state data staged in LDS.  Within one
// separation d, pair (a, a + d) only touches states of residue a mod d, so
// the d residue classes are independent chains, each taken in ascending a by
// a wavefront of its own (position t of class rho = state rho + t d, one per
// lane, in blocks of 64).  A chain is a sequence of runs: the replica of the
// run's first position q is carried up the chain while its swaps are accepted
// and stays at the position where one is rejected (or where the chain ends);
// the next run starts one position further up with that position's own
// replica.  When pair (t, t + 1) is attempted, position t + 1 still holds its
// replica from the start of the pass, so whether the replica of q would pass
// from t to t + 1 depends only on (q, t) and the labels at the start of the
// pass: the attempts of a run are independent of each other.
//   1. every state's energy with its own replica and with the next one's, and
//      its own replica's at the kXAhead states above it (two threads a state);
//   2. with those, the first kXAhead steps of the run that would start at
//      each state, all at once;
//   3. the class's wavefront walks the runs that happen (scalar, one lane
//      read per run); a run still open after those steps is finished by one
//      attempt per lane, the replica's at every later position of the block,
//      and the first rejection found by a ballot; then a bit per run start
//      gives every position its new replica.
// The cost is latency: three barriers and about twenty dependent LDS round
// trips a pass (1.1k + 0.8k cycles for steps 1 and 2; 2k for step 3 where a
// class fits one block, 4-7k over two or three), not the longest run's
// length in steps, as when one lane per first position follows its run step
// by step (170 states, 25 sweeps of 5 separations, neighbours swapping at
// 0.87: 926 us a call so, 334 us this way).  kXAhead: 4, 6 and 8 steps give
// 372, 355 and 354 us; with the walk's doublings as well, 334.  Separations of
// many short classes are walked by a lane per class instead
// (exchange_wave_separations).  The energies are the same double sums as
// state_energy and each attempt sees the replicas the one-thread order gives
// it, so every decision is that order's.
constexpr int kXStates = 256, kXChannels = 5;
constexpr int kXAhead = 8;      // steps decided ahead of the walk
constexpr int kXHalf = kXAhead / 2;
constexpr int kXJump = 3;       // doublings of the walk's step
constexpr int kXShort = 8;      // positions up to which a walk does without
constexpr int kXThreads = 512;  // block of the exchange kernels
struct alignas(16) XStage {
  double cp[kXStates * (1 + kXChannels)];  // components per replica
  double sw[kXStates * (1 + kXChannels)];  // weights and beta per state
  // by lower state of a pair: energy of the replica in a + d at state a, and
  // ln u of the pass (two buffers, by pass)
  double2 el[2][kXStates];
  double ecur[kXStates];  // energy of the replica in state k at state k
  int ros[2][kXStates];   // replica of each state (two buffers)
  int len[2][kXStates];   // swaps ahead of a run from the state, by halves
  int nacc[kXStates];     // accepted swaps of separation 1, by lower state
};

// 1 + C doubles of a staged array's entry, as 16-byte reads
template <int C>
__device__ __forceinline__ void staged_load(const double* p,
                                            double (&v)[1 + C]) {
  static_assert((1 + C) % 2 == 0, "entries are read as double2");
  const double2* q = reinterpret_cast<const double2*>(p);
#pragma unroll
  for (int e = 0; e < (1 + C) / 2; ++e) {
    const double2 t = q[e];
    v[2 * e] = t.x;
    v[2 * e + 1] = t.y;
  }
}
// energy of components v at a state of weights u (u[C]: its beta), in the
// order of state_energy
template <int C>
__device__ __forceinline__ double staged_sum(const double (&v)[1 + C],
                                             const double (&u)[1 + C]) {
  double E = v[0];
#pragma unroll
  for (int c = 0; c < C; ++c) E += u[c] * v[1 + c];
  return E;
}

// ladders of up to kXTable states also keep the whole table E(k, r) of
// every replica's energy at every state, computed once per call: an attempt
// then reads its energies instead of summing components
constexpr int kXTable = 64;

// the Metropolis test of attempt_pair
__device__ __forceinline__ bool staged_accepts(double ba, double bb,
                                               double2 el, double e,
                                               double eba, double ebb) {
  const double delta = ba * (el.x - e) + bb * (eba - ebb);
  return (bool)(isfinite(delta) & (el.y < -delta));
}

constexpr unsigned kXOpen = 1u << 16;  // mark of an open run in the walk

// Step 3 for one class by one wavefront: X.ros[cur] read, the other buffer
// written.  count: add the accepted swaps of every pair to X.nacc.
template <int C, bool TABLE, int WALK>
__device__ __forceinline__ void exchange_class(XStage& X, const double* em,
                                               int K, int d, int rho, int cur,
                                               int lb, bool count) {
  const int lane = threadIdx.x & (kWave - 1);
  const int T = (K - rho + d - 1) / d;  // positions of the class
  const int* ros = X.ros[cur];
  const double2* el = X.el[lb];
  // the lane's operands of block `held` (positions past the last pair: unused)
  int held = -1;
  double hw0[1 + C], hw1[1 + C], hec = 0.0;
  double2 hel = make_double2(0.0, 0.0);
  int q = 0, before = 0;  // next run's start, last start below the block
  for (int b0 = 0; b0 < T; b0 += kWave) {
    const int t = b0 + lane, ac = rho + (t < T ? t : T - 1) * d;
    const int rep = ros[ac];
    int ln = X.len[0][ac];
    if (ln == kXHalf) ln += X.len[1][ac];
    // the next run's start, relative to the block, or an open run's position
    // (a pair above it is left to attempt) with a mark
    unsigned next =
        ln == kXAhead && t + kXAhead < T - 1
            ? (unsigned)(t + kXAhead) | kXOpen : (unsigned)(lane + ln + 1);
    const unsigned lim = T - b0 < kWave ? T - b0 : kWave;
    // up to 2^kXJump runs in a row as one: the starts met and what follows
    unsigned mlo = lane < 32 ? 1u << lane : 0u;
    unsigned mhi = lane < 32 ? 0u : 1u << (lane - 32);
    if (WALK == kWalkNear || T > kXShort) {
#pragma unroll
      for (int i = 0; i < kXJump; ++i) {
        const int src = 4 * (int)(next < lim ? next : (unsigned)lane);
        mlo |= (unsigned)__builtin_amdgcn_ds_bpermute(src, (int)mlo);
        mhi |= (unsigned)__builtin_amdgcn_ds_bpermute(src, (int)mhi);
        next = (unsigned)__builtin_amdgcn_ds_bpermute(src, (int)next);
      }
    }
    unsigned long long start = 0ull;
    unsigned qr = q - b0;
    while (qr < lim) {
      do {
        const unsigned lo = __builtin_amdgcn_readlane(mlo, qr);
        const unsigned hi = __builtin_amdgcn_readlane(mhi, qr);
        start |= (unsigned long long)hi << 32 | lo;
        qr = __builtin_amdgcn_readlane(next, qr);
      } while (qr < lim);
      if (qr & kXOpen) {
        // the open run is the last one met
        const int rq = __builtin_amdgcn_readlane(
            rep, 63 - __builtin_clzll(start));
        double cv[1 + C];
        if (!TABLE) staged_load<C>(X.cp + rq * (1 + C), cv);
        // attempts of the carried replica at positions p, p + 1, ...
        for (int p = qr & (kXOpen - 1);;) {
          const int blk = (unsigned)p / kWave;
          const int ta = kWave * blk + lane;
          const bool live = ta >= p && ta + 1 < T;
          const int s0 = rho + (ta + 1 < T ? ta : T - 2) * d, s1 = s0 + d;
          if (blk != held) {
            held = blk;
            hel = el[s0];
            hec = X.ecur[s1];
            staged_load<C>(X.sw + s0 * (1 + C), hw0);
            staged_load<C>(X.sw + s1 * (1 + C), hw1);
          }
          const double e0 =
              TABLE ? em[s0 * kXTable + rq] : staged_sum<C>(cv, hw0);
          const double e1 =
              TABLE ? em[s1 * kXTable + rq] : staged_sum<C>(cv, hw1);
          const bool ok = staged_accepts(hw0[C], hw1[C], hel, e0, e1, hec);
          const unsigned long long no = __ballot(live && !ok);
          if (no) {
            qr = kWave * blk + __builtin_ctzll(no) + 1 - b0;
            break;
          }
          p = kWave * (blk + 1);
          if (p >= T - 1) {
            qr = T - b0;
            break;
          }
        }
      }
    }
    q = b0 + qr;
    // a position where a run ends takes the run's replica; any other one had
    // its swap with the position above accepted
    const unsigned long long at = start & (~0ull >> (63 - lane));
    const int qs = at ? b0 + 63 - __builtin_clzll(at) : before;
    const unsigned long long up =
        (start >> 1) | (q == b0 + kWave ? 1ull << 63 : 0ull);
    if (t < T) {
      const int a = rho + t * d;
      const bool ends = t == T - 1 || ((up >> lane) & 1ull);
      X.ros[cur ^ 1][a] = ros[ends ? rho + qs * d : a + d];
      if (count && !ends) X.nacc[a] += 1;
    }
    if (start) before = b0 + 63 - __builtin_clzll(start);
  }
}

// Step 3 for a class by one lane, for separations of many short classes: the
// positions in order, each either passing its replica on to the next one or
// keeping the run's.  The states' replicas and run lengths load kXLane
// positions at a time, ahead of the chain; a run still open after its kXAhead
// steps goes on attempt by attempt.
constexpr int kXLane = 4;
template <int C, bool TABLE>
__device__ __forceinline__ void exchange_lane(XStage& X, const double* em,
                                              int K, int d, int rho, int cur,
                                              int lb) {
  const int* ros = X.ros[cur];
  const double2* el = X.el[lb];
  int rq = 0, left = 0;  // the run's replica, its known swaps still to come
  bool start = true, open = false;
  for (int a0 = rho; a0 < K; a0 += kXLane * d) {
    int rep[kXLane + 1], ln[kXLane];
#pragma unroll
    for (int m = 0; m <= kXLane; ++m) {
      const int a = a0 + m * d < K ? a0 + m * d : a0;
      rep[m] = ros[a];
      if (m < kXLane) {
        const int l0 = X.len[0][a], l1 = X.len[1][a];
        ln[m] = l0 == kXHalf ? l0 + l1 : l0;
      }
    }
#pragma unroll
    for (int m = 0; m < kXLane; ++m) {
      const int a = a0 + m * d, b = a + d;
      if (a >= K) break;
      if (start) {
        rq = rep[m];
        left = ln[m];
        open = left == kXAhead;
      }
      bool swap = left > 0;
      if (!swap && open && b < K) {
        double ua[1 + C], ub[1 + C], cv[1 + C];
        staged_load<C>(X.sw + a * (1 + C), ua);
        staged_load<C>(X.sw + b * (1 + C), ub);
        if (!TABLE) staged_load<C>(X.cp + rq * (1 + C), cv);
        const double e0 = TABLE ? em[a * kXTable + rq] : staged_sum<C>(cv, ua);
        const double e1 = TABLE ? em[b * kXTable + rq] : staged_sum<C>(cv, ub);
        swap = staged_accepts(ua[C], ub[C], el[a], e0, e1, X.ecur[b]);
        open = swap;
      } else {
        --left;
      }
      X.ros[cur ^ 1][a] = swap ? rep[m + 1] : rq;
      start = !swap;
    }
  }
}

// WALK: the launch's ladders (ExchangeWalk).  kWalkFar has kernels of its own:
// with both walks in one, the loop's scalars spill and a pass of the nearest
// separations takes 5 % longer; steps past the end of every class, whose
// energies no run asks for, are then left out.
template <int C, bool TABLE, int WALK>
__device__ __forceinline__ void exchange_all_staged(
    const LigDev& L, uint64_t sweep, int max_sep, int n_sub, uint64_t seed,
    XStage& X, double* em) {
  constexpr int C1 = 1 + C;
  constexpr bool kFar = WALK == kWalkFar;
  const int K = L.K;
  const int tid = threadIdx.x, nt = blockDim.x;
  const int nw = nt / kWave;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  for (int i = tid; i < K * C1; i += nt) {
    const int k = i / C1, c = i - k * C1;
    X.cp[i] = L.comps[i];
    X.sw[i] = c < C ? L.wd[k * C + c] : L.beta[k];
  }
  for (int k = tid; k < K; k += nt) {
    X.ros[0][k] = L.replica_of_state[k];
    X.nacc[k] = 0;
  }
  __syncthreads();
  if (TABLE) {
    for (int i = tid; i < K * K; i += nt) {
      const int k = i / K, r = i - k * K;
      double v[C1], u[C1];
      staged_load<C>(X.cp + r * C1, v);
      staged_load<C>(X.sw + k * C1, u);
      em[k * kXTable + r] = staged_sum<C>(v, u);
    }
  }
  int cur = 0, lb = 0;
  const int dmax = max_sep < K - 1 ? max_sep : K - 1;
  // ln u of the pass (j, d) into buffer b, by threads t0, t0 + stride, ...
  auto draw_pass = [&](int j, int d, int b, int t0, int stride) {
    const uint32_t purpose = (uint32_t)kExchange | ((uint32_t)d << 8);
    for (int a = t0; a + d < K; a += stride)
      X.el[b][a].y =
          log(u01d(draw(seed, (uint32_t)a, L.id, j, sweep, purpose).x));
  };
  if (n_sub > 0 && dmax > 0) draw_pass(0, 1, 0, tid, nt);
  if (TABLE) __syncthreads();
  // steps 1 and 2: threads 0..255 and 256..511 (half h) each take the state
  // tid mod 256, whose weights they keep in registers
  static_assert(kXThreads == 2 * kXStates, "two threads a state");
  const int h = tid / kXStates, a = tid - h * kXStates;
  const int hu = wv / (kXStates / kWave);  // h, known to be uniform
  const bool act = a < K;
  double ua[C1];
  staged_load<C>(X.sw + (act ? a : 0) * C1, ua);
  const int dw = exchange_wave_separations(K);
  for (int j = 0; j < n_sub; ++j) {
    for (int d = 1; d <= dmax; ++d) {
      const bool lanes = kFar && d > dw;
      const int* ros = X.ros[cur];
      double2* el = X.el[lb];
      // energies of the state's replica at the half's states, the energy at
      // the state of its own (h = 0) or the next state's replica (h = 1)
      double e[kXHalf + 1], be[kXHalf + 1];
      int st[kXHalf + 1];
      if (act) {
        const int r = ros[a], r1 = ros[a + d < K ? a + d : a];
        double v[C1], v1[C1];
        if (!TABLE) {
          staged_load<C>(X.cp + r * C1, v);
          if (h == 1) staged_load<C>(X.cp + r1 * C1, v1);
        }
#pragma unroll
        for (int m = 0; m <= kXHalf; ++m) {
          // steps past every class's end
          if (kFar && (kXHalf * hu + m) * d >= K) break;
          const int s = a + (kXHalf * h + m) * d;
          st[m] = s < K ? s : a;  // past the end: any state (not counted)
          double u[C1];
          staged_load<C>(X.sw + st[m] * C1, u);
          e[m] = TABLE ? em[st[m] * kXTable + r] : staged_sum<C>(v, u);
          be[m] = u[C];
        }
        if (h == 0) {
          X.ecur[a] = e[0];
        } else {
          el[a].x = TABLE ? em[a * kXTable + r1] : staged_sum<C>(v1, ua);
        }
      }
      __syncthreads();
      if (act) {
        int len = 0;
        bool go = true;
#pragma unroll
        for (int m = 0; m < kXHalf; ++m) {
          if (kFar && (kXHalf * hu + m + 1) * d >= K) break;
          const bool ok = staged_accepts(be[m], be[m + 1], el[st[m]], e[m],
                                         e[m + 1], X.ecur[st[m + 1]]);
          go = (bool)(go & ok & (a + (kXHalf * h + m + 1) * d < K));
          len += go ? 1 : 0;
        }
        X.len[h][a] = len;
      }
      __syncthreads();
      // (3) the walk, a wavefront or a lane per class; the next pass's
      // uniforms by the wavefronts without a class meanwhile (by every one,
      // first, when all have classes)
      const int dn = d < dmax ? d + 1 : 1, jn = d < dmax ? j : j + 1;
      const int w0 = lanes ? (d + kWave - 1) / kWave : d < nw ? d : 0;
      if (jn < n_sub && wv >= w0)
        draw_pass(jn, dn, lb ^ 1, tid - w0 * kWave, nt - w0 * kWave);
      if (!lanes) {
        for (int rho = wv; rho < d; rho += nw)
          exchange_class<C, TABLE, WALK>(X, em, K, d, rho, cur, lb, d == 1);
      } else if (tid < d) {
        exchange_lane<C, TABLE>(X, em, K, d, tid, cur, lb);
      }
      cur ^= 1;
      lb ^= 1;
      __syncthreads();
    }
  }
  for (int k = tid; k < K; k += nt) {
    const int r = X.ros[cur][k];
    L.replica_of_state[k] = r;
    L.state_of_replica[r] = k;
    if (k + 1 < K && dmax > 0) {
      atomicAdd(&L.ex_try[k], (unsigned long long)n_sub);
      if (X.nacc[k]) atomicAdd(&L.ex_acc[k], (unsigned long long)X.nacc[k]);
    }
  }
}
#pragma clang fp contract(fast)

// block-wide exchange for one ligand (called by all threads): n_sub
// exchange sweeps in a row, sweep j drawing its uniforms with replica field j
// Inlined into its kernels, with everything below it: in a called function
// the staged data's pointers are generic and every access a flat one.
template <int WALK>
__device__ __forceinline__ void exchange_block(const LigDev& L, uint64_t sweep,
                                               int scheme, int max_sep,
                                               int n_sub, uint64_t seed) {
  __shared__ XStage X;
  __shared__ double em[kXTable * kXTable];
  const int K = L.K;
  if (K < 2) return;
  if (scheme == 0) {
    // disjoint neighbour pairs: independent, one thread each
    const int a0 = (int)(sweep & 1ull);
    for (int j = 0; j < n_sub; ++j) {
      if (j > 0) __syncthreads();
      for (int a = a0 + 2 * (int)threadIdx.x; a + 1 < K; a += 2 * blockDim.x)
        attempt_pair(L, a, a + 1, 1, sweep, j, seed);
    }
  } else if (K <= kXTable && L.C == 3) {
    exchange_all_staged<3, true, WALK>(L, sweep, max_sep, n_sub, seed, X,
                                       em);
  } else if (K <= kXTable && L.C == 5) {
    exchange_all_staged<5, true, WALK>(L, sweep, max_sep, n_sub, seed, X,
                                       em);
  } else if (K <= kXStates && L.C == 3) {
    exchange_all_staged<3, false, WALK>(L, sweep, max_sep, n_sub, seed, X,
                                       em);
  } else if (K <= kXStates && L.C == 5) {
    exchange_all_staged<5, false, WALK>(L, sweep, max_sep, n_sub, seed, X,
                                       em);
  } else if (threadIdx.x == 0) {
    const int dmax = max_sep < K - 1 ? max_sep : K - 1;
    for (int j = 0; j < n_sub; ++j)
      for (int d = 1; d <= dmax; ++d)
        for (int a = 0; a + d < K; ++a)
          attempt_pair(L, a, a + d, d, sweep, j, seed);
  }
  // every replica's state after the exchange (round-trip bookkeeping)
  __syncthreads();
  for (int r = threadIdx.x; r < K; r += blockDim.x)
    note_state(L, r, L.state_of_replica[r]);
}

// Tail of one ligand's sweep, run by one whole block: exchange (if due),
// record one sample per state (if due), counter += 1.
template <int WALK>
__device__ __forceinline__ void sweep_tail(const LigDev& L, int exchange_every,
                                           int scheme, int max_sep, int n_sub,
                                           int sample_every, uint64_t seed) {
  const unsigned long long s = *L.counter;
  if (exchange_every > 0 && s % (unsigned long long)exchange_every == 0ull)
    exchange_block<WALK>(L, s, scheme, max_sep, n_sub, seed);
  __syncthreads();
  const unsigned long long rec = *L.n_rec;
  const bool record = sample_every > 0 &&
                      (s + 1ull) % (unsigned long long)sample_every == 0ull &&
                      rec < (unsigned long long)L.cap;
  if (record) {
    const int n3 = L.n * 3, C1 = 1 + L.C;
    float* dx = L.samp_x + (size_t)rec * L.K * n3;
    double* dc = L.samp_c + (size_t)rec * L.K * C1;
    for (int q = threadIdx.x; q < L.K * n3; q += blockDim.x) {
      const int k = q / n3, e = q - k * n3;
      dx[q] = L.x[(size_t)L.replica_of_state[k] * n3 + e];
    }
    for (int q = threadIdx.x; q < L.K * C1; q += blockDim.x) {
      const int k = q / C1, e = q - k * C1;
      dc[q] = L.comps[(size_t)L.replica_of_state[k] * C1 + e];
    }
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    *L.counter = s + 1ull;
    if (record) *L.n_rec = rec + 1ull;
  }
}

// One block per ligand: the tail as a kernel of its own.
template <int WALK>
__global__ __launch_bounds__(kXThreads) void k_sweep_tail(
    const LigDev* __restrict__ ligs, int exchange_every, int scheme,
    int max_sep, int n_sub, int sample_every, uint64_t seed) {
  sweep_tail<WALK>(ligs[blockIdx.x], exchange_every, scheme, max_sep, n_sub,
             sample_every, seed);
}

// Start of a run of neighbour-scheme sweeps: buffer (s-1)&1 from the
// canonical state, nothing pending.  One block per ligand.
__global__ __launch_bounds__(256) void k_sweep_begin(
    const LigDev* __restrict__ ligs) {
  begin_ligand(ligs[blockIdx.x]);
}

// End of a run: the pending exchange and record of the last sweep, the
// canonical state written back.  One block per ligand.
__global__ __launch_bounds__(256) void k_sweep_finish(
    const LigDev* __restrict__ ligs, int exchange_every, int sample_every,
    uint64_t seed) {
  finish_ligand(ligs[blockIdx.x], exchange_every, sample_every, seed);
}

// ----------------------------------------------------------------------------
// HMC: one trial move per replica, one workgroup of W wavefronts per replica.
// (Sampling: HMC trial moves from velocity-Verlet molecular dynamics.)
// ----------------------------------------------------------------------------
// ONE: the launch covers the replicas of a single ligand, whose table entry
// comes in the kernel arguments (block b = replica b) instead of through the
// task list.
// PAIRS (partners at once, or 0): ligands whose pair terms are in the energy
// (L.pairs_on) evaluate them too.
template <int C, int W, bool ONE, int PAIRS>
__global__ __launch_bounds__(W * kWave) void k_hmc_sweep(
    GridDev g, const LigDev* __restrict__ ligs, const int2* __restrict__ tasks,
    LigDev one, int nleap, uint64_t seed, TailArgs tail) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int tid = threadIdx.x;
  const int2 task = ONE ? make_int2(0, (int)blockIdx.x) : tasks[blockIdx.x];
  const LigDev L = ONE ? one : ligs[task.x];  // kernel-lifetime copy
  const int r = task.y;
  const int n = L.n;
  const bool deferred = tail.scheme == 0;

  // per-replica state and per-atom data: issued before the topology is
  // staged so that both latencies overlap
  unsigned long long s;
  int a = 0, pin = 0, ain = 0;
  bool pend = false;
  if (deferred) {
    s = BPMF_GMEM(const unsigned long long, L.rcnt)[r];
    auto rsor = BPMF_GMEM(const int, L.rsor);
    auto rpend = BPMF_GMEM(const int, L.rpend);
    const int a0 = rsor[r], a1 = rsor[L.K + r];
    const int p0 = rpend[r], p1 = rpend[L.K + r];
    pin = (int)((s - 1ull) & 1ull);
    ain = pin ? a1 : a0;
    a = rsor_state(ain);
    pend = (pin ? p1 : p0) != 0;
  } else {
    s = *BPMF_GMEM(const unsigned long long, L.counter);
    a = BPMF_GMEM(const int, L.state_of_replica)[r];
  }
  const int fv = BPMF_GMEM(const int, L.fvalid)[r];
  const bool owner = tid < n;
  float x[3], v[3], f[3];
  const float m = owner ? BPMF_GMEM(const float, L.mass)[tid] : 0.f;
  float sc[C];
#pragma unroll
  for (int c = 0; c < C; ++c)
    sc[c] = owner ? BPMF_GMEM(const float, L.scale)[tid * C + c] : 0.f;
  const float im = owner ? BPMF_GMEM(const float, L.inv_mass)[tid] : 0.f;
  auto xr = BPMF_GMEM(const float, L.x) + (size_t)r * n * 3;
#pragma unroll
  for (int d = 0; d < 3; ++d) x[d] = owner ? xr[tid * 3 + d] : 0.f;

  // the ligand's topology goes to LDS now: its loads need only the table
  // entry, so they overlap the replica's; the barrier comes after the
  // loads below have been issued as well
  const Shared sh = carve<W, false>(smem, L, L.n, tid);

  // scheme 0 first applies the exchange (and record) that ended the previous
  // sweep, from the double buffer; the parameters of both states of the
  // replica's pair are loaded with the pair's components
  const Pair pr = (deferred && pend) ? own_pair(L.K, a, s, tail.exchange_every)
                                     : Pair{a, a, false};
  const int kb = pr.active ? (a == pr.lo ? pr.hi : pr.lo) : a;
  float wa[C], wb[C];
  double wda[C], wdb[C];
  auto wf = BPMF_GMEM(const float, L.wf);
  auto wdp = BPMF_GMEM(const double, L.wd);
#pragma unroll
  for (int c = 0; c < C; ++c) {
    wa[c] = wf[a * C + c];
    wb[c] = wf[kb * C + c];
    wda[c] = wdp[a * C + c];
    wdb[c] = wdp[kb * C + c];
  }
  auto Tf = BPMF_GMEM(const float, L.Tf);
  auto dtf = BPMF_GMEM(const float, L.dtf);
  auto bt = BPMF_GMEM(const double, L.beta);
  const float Ta = Tf[a], Tb = Tf[kb];
  const float dta = dtf[a], dtb = dtf[kb];
  const double ba = bt[a], bb = bt[kb];
  // the start of the trajectory's stored parts (state-independent force of
  // the current positions, restraint factor, components), loaded beside
  // the exchange's operands
  constexpr int kFC = 3 + 3 * C;
  const int C1 = 1 + C;
  const int cur = fv > 0 ? fv - 1 : 0, nxt = 1 - cur;
  float* const fc_cur = L.fcache + ((size_t)cur * L.K + r) * n * kFC;
  float* const fc_nxt = L.fcache + ((size_t)nxt * L.K + r) * n * kFC;
  float ca[kFC], cr[4];
  double cp[1 + C];
  if (fv > 0) {
    if (owner) {
      auto cap = BPMF_GMEM(const float, fc_cur + (size_t)tid * kFC);
#pragma unroll
      for (int q = 0; q < kFC; ++q) ca[q] = cap[q];
    } else {
#pragma unroll
      for (int q = 0; q < kFC; ++q) ca[q] = 0.f;
    }
    auto crp = BPMF_GMEM(const float, L.frc + ((size_t)cur * L.K + r) * 4);
#pragma unroll
    for (int q = 0; q < 4; ++q) cr[q] = crp[q];
    auto cpp = BPMF_GMEM(const double,
                         deferred ? L.scomp + ((size_t)pin * L.K + a) * C1
                                  : L.comps + (size_t)r * C1);
#pragma unroll
    for (int q = 0; q < 1 + C; ++q) cp[q] = cpp[q];
  }
  // the decision is the block's: the last wavefront (the one with the
  // fewest atoms) takes it and publishes it with the barrier that ends the
  // staging
  // The replica's next state-map entry (its state after this decision and
  // its round-trip mark) is written here: only this block reads it, in the
  // next sweep.
  __shared__ int s_swap;
  int* const rsor_out = L.rsor + (1 - pin) * L.K + r;
  if (pr.active && (tid >> 6) == W - 1) {
    const bool sw = pair_accepts<C>(L, pr, pin, s, seed);
    if (tid == (W - 1) * kWave) {
      s_swap = sw ? 1 : 0;
      if (a == pr.lo) {
        atomicAdd(&L.ex_try[pr.lo], 1ull);
        if (sw) atomicAdd(&L.ex_acc[pr.lo], 1ull);
      }
      *rsor_out = sw ? rsor_pack(kb, rt_step(L, rsor_mark(ain), kb)) : ain;
    }
  }
  if (deferred && !pr.active && tid == 0) *rsor_out = ain;
  // the momenta's standard normals do not depend on the state: drawn
  // beside the decision
  float z[3] = {0.f, 0.f, 0.f};
  if (owner) {
    const U4 o = draw(seed, (uint32_t)tid, L.id, r, s, kMomenta);
    normals3(o, z[0], z[1], z[2]);
  }
  __syncthreads();  // the staged topology and the decision
  const bool swap = pr.active && s_swap != 0;
  const int k = swap ? kb : a;
  float w[C];
  double wdk[C];
#pragma unroll
  for (int c = 0; c < C; ++c) {
    w[c] = swap ? wb[c] : wa[c];
    wdk[c] = swap ? wdb[c] : wda[c];
  }
  const float T = swap ? Tb : Ta;
  const float dt = swap ? dtb : dta;
  const double beta = swap ? bb : ba;

  __shared__ double fin[2 * W];
  // the previous sweep's round: this replica's configuration and components
  // go to the slot of its state after that exchange.  The replica's record
  // counter is advanced at the end of the kernel, after the barriers, so that
  // every wavefront has read it first.
  bool recorded = false;
  unsigned long long rec = 0ull;
  if (deferred && pend && record_due(s, tail.sample_every)) {
    rec = BPMF_GMEM(const unsigned long long, L.rnrec)[r];
    if (rec < (unsigned long long)L.cap) {
      recorded = true;
      if (owner)
#pragma unroll
        for (int d = 0; d < 3; ++d)
          BPMF_GMEM(float, L.samp_x)[((size_t)rec * L.K + k) * n * 3 +
                                     tid * 3 + d] = x[d];
      if (tid < C1)
        BPMF_GMEM(double, L.samp_c)[((size_t)rec * L.K + k) * C1 + tid] =
            BPMF_GMEM(const double, L.scomp)[((size_t)pin * L.K + a) * C1 +
                                             tid];
    }
  }
  {
    const float sd = owner ? sqrtf((float)kRGas * T * im * 1e-4f) : 0.f;
    v[0] = sd * z[0];
    v[1] = sd * z[1];
    v[2] = sd * z[2];
  }
  const float ke0 = 0.5f * m * (v[0] * v[0] + v[1] * v[1] + v[2] * v[2]);

  // start of the trajectory: force and energy at the current positions,
  // rebuilt from the state-independent parts stored when these positions
  // were last evaluated (same arithmetic, same bits), or evaluated
  double U0, KE0;
  if (fv > 0) {
    U0 = cp[0];
#pragma unroll
    for (int c = 0; c < C; ++c) U0 += wdk[c] * cp[1 + c];
    if (owner) {
      float de[C][3], ge[3] = {0.f, 0.f, 0.f};
#pragma unroll
      for (int c = 0; c < C; ++c)
#pragma unroll
        for (int d = 0; d < 3; ++d) de[c][d] = ca[3 + 3 * c + d];
      grid_force<C>(w, de, ge);
      restraint_force(cr[0], m, cr[1], cr[2], cr[3], ge);
      f[0] = ca[0] + ge[0];
      f[1] = ca[1] + ge[1];
      f[2] = ca[2] + ge[2];
    } else {
      f[0] = f[1] = f[2] = 0.f;
    }
    double ke, unused;
    block_sum2<W, true>(ke0, 0.f, fin, tid, ke, unused);
    KE0 = ke * 1e4;
  } else {
    double t0[6 + C];
    eval_block<C, W, true, true, false, true, PAIRS>(
        g, L, w, x, m, sc, f, t0, ke0, 0.f, sh, tid,
        owner ? fc_cur + (size_t)tid * kFC : nullptr,
        L.frc + ((size_t)cur * L.K + r) * 4);
    U0 = t0[0] + t0[1] + t0[2] + t0[3];
#pragma unroll
    for (int c = 0; c < C; ++c) U0 += wdk[c] * t0[4 + c];
    KE0 = t0[4 + C] * 1e4;
  }

  // nleap velocity-Verlet steps; the last one also evaluates the energy
  const float hk = 0.5f * dt * 1e-4f * im;
  double t1[6 + C];
  for (int step = 0; step < nleap - 1; ++step) {
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      v[d] = fmaf(hk, f[d], v[d]);
      x[d] = fmaf(dt, v[d], x[d]);
    }
    eval_block<C, W, true, false, false, true, PAIRS>(g, L, w, x, m, sc, f,
                                                      t1, 0.f, 0.f, sh, tid);
#pragma unroll
    for (int d = 0; d < 3; ++d) v[d] = fmaf(hk, f[d], v[d]);
  }
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    v[d] = fmaf(hk, f[d], v[d]);
    x[d] = fmaf(dt, v[d], x[d]);
  }
  // lean sums: the bonded total (the sweep needs no single bonded term),
  // formed in wavefront 0 only (its lanes take the decision and write the
  // components)
  eval_block<C, W, true, true, true, true, PAIRS, true>(
      g, L, w, x, m, sc, f, t1, 0.f, 0.f, sh, tid,
      owner ? fc_nxt + (size_t)tid * kFC : nullptr,
      L.frc + ((size_t)nxt * L.K + r) * 4);
#pragma unroll
  for (int d = 0; d < 3; ++d) v[d] = fmaf(hk, f[d], v[d]);
  double U1 = t1[0] + t1[1] + t1[2] + t1[3];
#pragma unroll
  for (int c = 0; c < C; ++c) U1 += wdk[c] * t1[4 + c];
  const float ke1 = 0.5f * m * (v[0] * v[0] + v[1] * v[1] + v[2] * v[2]);
  const float bad =
      (!isfinite(x[0]) || !isfinite(x[1]) || !isfinite(x[2])) ? 1.f : 0.f;
  double KE1, nbad;
  block_sum2<W, true>(ke1, bad, fin, tid, KE1, nbad);
  // the Metropolis decision in wavefront 0, published through LDS
  __shared__ int s_acc;
  bool finite = true;
  if (tid < kWave) {
    KE1 *= 1e4;
    const double dH = (U1 + KE1) - (U0 + KE0);
    const U4 o = draw(seed, 0u, L.id, r, s, kAccept);
    finite = isfinite(dH) && nbad == 0.0;
    const bool acc0 = finite && ln_u_below(o.x, -beta * dH);
    if (tid == 0) s_acc = acc0 ? 1 : 0;
  }
  block_sync();
  const bool accept = s_acc != 0;
  if (accept) {
    auto xw = BPMF_GMEM(float, L.x) + (size_t)r * n * 3;
    if (owner)
#pragma unroll
      for (int d = 0; d < 3; ++d) xw[tid * 3 + d] = x[d];
  }
  // components of the replica after the move (scheme 0: into the output
  // buffer, indexed by state)
  if (tid < C1 && (accept || deferred)) {
    double cv;
    if (accept) {
      // select without a register-array index
      cv = t1[0] + t1[1] + t1[2] + t1[3];
#pragma unroll
      for (int c = 0; c < C; ++c)
        if (tid == 1 + c) cv = t1[4 + c];
    } else {
      cv = BPMF_GMEM(const double, L.scomp)[((size_t)pin * L.K + a) * C1 +
                                            tid];
    }
    if (deferred)
      BPMF_GMEM(double, L.scomp)[((size_t)(s & 1ull) * L.K + k) * C1 + tid] =
          cv;
    else
      BPMF_GMEM(double, L.comps)[(size_t)r * C1 + tid] = cv;
  }
  if (tid == 0) {
    // the stored parts of the replica's (new or kept) positions
    BPMF_GMEM(int, L.fvalid)[r] = 1 + (accept ? nxt : cur);
    atomicAdd(&L.hmc_try[k], 1ull);
    if (accept) atomicAdd(&L.hmc_acc[k], 1ull);
    if (!finite) atomicAdd(L.nonfinite, 1ull);
    if (deferred) {
      const int pout = (int)(s & 1ull);
      BPMF_GMEM(int, L.rpend)[pout * L.K + r] = 1;
      BPMF_GMEM(unsigned long long, L.rcnt)[r] = s + 1ull;
      if (recorded) BPMF_GMEM(unsigned long long, L.rnrec)[r] = rec + 1ull;
    }
  }
}

template <int WALK>
__global__ __launch_bounds__(kXThreads) void k_exchange(
    const LigDev* __restrict__ ligs, int scheme, int max_sep, int n_sub,
    uint64_t seed) {
  const LigDev& L = ligs[blockIdx.x];
  exchange_block<WALK>(L, *L.counter, scheme, max_sep, n_sub, seed);
}

// ----------------------------------------------------------------------------
// reduced-energy matrix u_kn = beta_k (U0_n + sum_c w_kc Psi_cn) of samples
// of one or many ligands (Estimation), energy only
// ----------------------------------------------------------------------------
// First sample of block b's share of a launch (b = nblocks: the end): the
// shares are contiguous runs of the flat sample index of equal estimated
// cost, so a block holding a large ligand's samples takes fewer of them.
// Position P = b * total_cost / nblocks falls in job j (jobs[j].cfirst <= P
// < jobs[j + 1].cfirst; the sentinel ends the list) and the share starts at
// the first of its samples whose cost starts at or after P.  j: that job.
__device__ __forceinline__ int64_t ukn_share_start(
    const UknJob* __restrict__ jobs, int n_jobs, int b, int nblocks, int& j) {
  const int64_t P = (int64_t)b * jobs[n_jobs].cfirst / nblocks;
  int lo = 0, hi = n_jobs;
  while (hi - lo > 1) {
    const int mid = (lo + hi) / 2;
    if (jobs[mid].cfirst <= P) lo = mid; else hi = mid;
  }
  const int64_t c = jobs[lo].cost;
  int64_t k = (P - jobs[lo].cfirst + c - 1) / c;
  if (k > jobs[lo].n) k = jobs[lo].n;
  // block-uniform results, held in scalar registers (the 64-bit division
  // is vector code)
  j = __builtin_amdgcn_readfirstlane(lo);
  const int64_t r = jobs[lo].first + k;
  const uint32_t rlo = __builtin_amdgcn_readfirstlane((uint32_t)r);
  const uint32_t rhi = __builtin_amdgcn_readfirstlane((uint32_t)(r >> 32));
  return (int64_t)(((uint64_t)rhi << 32) | rlo);
}

// One W-wave block evaluates one sample at a time, persistent over the
// launch: block b takes the b-th contiguous share (by cost) of the flat
// sample index over all jobs (job j's samples are [jobs[j].first, jobs[j+1].first); a
// sentinel ends the list), so it stages a ligand's topology once per
// segment.  Each sample's column (K entries) goes to LDS; every `group`
// samples (at most 16: a 128-byte line of each row) the columns are written
// out row by row by consecutive lanes.
template <int C, int W, bool PAIRS>
__global__ __launch_bounds__(W * kWave) void k_energy_matrix(
    GridDev g, const LigDev* __restrict__ ligs,
    const UknJob* __restrict__ jobs, int n_jobs, int64_t total,
    int group) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int tid = threadIdx.x;
  const float w0[C] = {};
  // ligands and jobs come from restrict arguments: the u_kn stores cannot
  // clobber them, so they load into scalar registers
  int j, j_end;
  const int64_t b0 = ukn_share_start(jobs, n_jobs, blockIdx.x, gridDim.x, j);
  const int64_t b1 =
      ukn_share_start(jobs, n_jobs, blockIdx.x + 1, gridDim.x, j_end);
  if (b0 >= b1) return;
  typedef const float __attribute__((address_space(1))) gfloat;
  typedef const double __attribute__((address_space(1))) gcdouble;
  for (int64_t s = b0; s < b1; ++j) {
    const UknJob J = jobs[j];
    const int64_t e = jobs[j + 1].first < b1 ? jobs[j + 1].first : b1;
    if (s >= e) continue;  // empty job
    const LigDev L = ligs[J.lig];
    // topology staged for the segment; the barrier in carve also keeps the
    // previous segment's readers ahead of the copy
    const Shared sh = carve<W>(smem, L, 0, tid);
    // state weights and beta_k after the topology, for the expansion, then
    // the group's columns (the evaluation's first barrier orders these
    // writes before their reads)
    const int K = L.K;
    double* ew = reinterpret_cast<double*>(
        smem + block_lds_bytes(W, false, L.n, L.nb, L.na, L.nt,
                               PAIRS && L.pairs_on));
    double* col = ew + K * (C + 1);
    for (int i = tid; i < K * (C + 1); i += W * kWave)
      ew[i] = i < K * C ? ((gcdouble*)L.wd)[i]
                        : ((gcdouble*)L.beta)[i - K * C];
    // per-lane data through global (not flat) loads, so that the waits of
    // the evaluation's LDS reads do not wait on them
    const int n = L.n;
    const bool owner = tid < n;
    const float m = owner ? ((gfloat*)L.mass)[tid] : 0.f;
    float sc[C];
#pragma unroll
    for (int c = 0; c < C; ++c)
      sc[c] = owner ? ((gfloat*)L.scale)[tid * C + c] : 0.f;
    const gfloat* xb = (const gfloat*)J.xs + (size_t)tid * 3;
    // positions of the next sample load during the current evaluation
    float xn[3];
#pragma unroll
    for (int d = 0; d < 3; ++d)
      xn[d] = owner ? xb[(size_t)(s - J.first) * n * 3 + d] : 0.f;
    for (; s < e;) {
      const int64_t g1 = s + group < e ? s + group : e;
      for (int64_t q = s; q < g1; ++q) {
        float x[3] = {xn[0], xn[1], xn[2]}, f[3];
        if (q + 1 < e) {
#pragma unroll
          for (int d = 0; d < 3; ++d)
            xn[d] = owner ? xb[(size_t)(q + 1 - J.first) * n * 3 + d] : 0.f;
        }
        double t[6 + C];
        eval_block<C, W, false, true, true, true, PAIRS ? kPairAhead : 0>(
            g, L, w0, x, m, sc, f, t, 0.f, 0.f, sh, tid);
        const double U0 = t[0] + t[1] + t[2] + t[3];
        double* cs = col + (q - s) * K;
        for (int k = tid; k < K; k += W * kWave) {
          double E = U0;
#pragma unroll
          for (int c = 0; c < C; ++c) E = fma(ew[k * C + c], t[4 + c], E);
          cs[k] = ew[K * C + k] * E;
        }
      }
      // the group's columns: each row's run of consecutive samples written
      // by consecutive lanes (global stores: no wait of the next LDS access
      // depends on them)
      block_sync();
      const int cnt = (int)(g1 - s);
      const int64_t n0 = s - J.first;
      auto out = BPMF_GMEM(double, J.ukn);
      for (int i = tid; i < cnt * K; i += W * kWave) {
        const int k = i / cnt, qq = i - k * cnt;
        out[(size_t)k * J.ld + n0 + qq] = col[qq * K + k];
      }
      s = g1;
    }
  }
}

// The same u_kn with one wavefront per sample, or one for two samples at
// once (H = 2), and no workgroup barrier inside a sample: for ligands whose
// pair terms are not in the energy.  A block of kUknWaves wavefronts stages
// the topology of its current job once (shared by its wavefronts); the job's
// samples are dealt to the wavefronts in runs, worked through in groups of
// up to kUknWaveGroup.  A wavefront evaluates a sample alone: lane l owns
// atoms l and l + 64 (AP = 2) or l; the grid terms of its atoms, every bonded
// chunk of the ligand (energies only), the mass-weighted position sums of the
// restraint, then double sums over the wavefront, as the lean block evaluation
// forms them: U0 = (bonded total) + U_I, and the C channel sums.  Its LDS (positions, the
// group's columns) is its own; LDS operations of one wavefront complete in
// order, so its lanes see each other's stores after a wavefront-scope fence.
//
// Bound by instruction issue (some 600 vector instructions a sample whatever
// part of the lanes owns an atom), so up to 32 atoms the wavefront's halves
// take a sample each: 225000 poses of 24 atoms, 50 states and 5 channels take
// 212 us, one at a time 289 us.  A wavefront's share is a run of whole pairs:
// dealt in groups of 8, 133 samples to four wavefronts left one with 40 (32
// ligands of 10 to 80 atoms, 3200 samples each: 165 -> 135 us, with the
// halves).  Registers: four wavefronts a SIMD with 3 channels, three with 5
// (four spill: 230 us instead of 212); both forms in one kernel spill as well,
// so a launch whose ligands all take the same one has a kernel of that form
// (one ligand of 48 atoms, 12000 samples of 4 states, a call with its wait:
// 50.2 us with both in the kernel, 48.2 us).
// The float sums of a half are those of a whole wavefront with the sample in
// its lower half: a lane's bonded items 64 apart in one accumulator, the
// position sums over two rows of 16.

// sum over each half of the wavefront, to all its lanes
__device__ __forceinline__ double half_sum(double v) {
  v += dpp_d<0xB1, 0xf>(v);
  v += dpp_d<0x4E, 0xf>(v);
  v += dpp_d<0x141, 0xf>(v);
  v += dpp_d<0x140, 0xf>(v);
  const long long b = __double_as_longlong(v);
  const auto lo = __builtin_amdgcn_permlane16_swap((int)(b & 0xffffffffll),
                                                   (int)(b & 0xffffffffll),
                                                   false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap((int)(b >> 32),
                                                   (int)(b >> 32), false,
                                                   false);
  return __longlong_as_double(((long long)hi[0] << 32) |
                              (long long)(unsigned)lo[0]) +
         __longlong_as_double(((long long)hi[1] << 32) |
                              (long long)(unsigned)lo[1]);
}
__device__ __forceinline__ float half_sumf(float v) {
  v += dpp_f<0xB1, 0xf>(v);
  v += dpp_f<0x4E, 0xf>(v);
  v += dpp_f<0x141, 0xf>(v);
  v += dpp_f<0x140, 0xf>(v);
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_int(v),
                                                  __float_as_int(v), false,
                                                  false);
  return __int_as_float(r[0]) + __int_as_float(r[1]);
}

// The columns of samples q0 .. q1 - 1 (at most kUknWaveGroup) of job J, by one
// wavefront.
template <int C, int AP, int H>
__device__ __forceinline__ void ukn_group(const GridDev& g, const LigDev& L,
                                          const UknJob& J, const Shared& sh,
                                          const double* ew, float4* pos,
                                          double* col, const float (&m)[AP],
                                          const float (&sc)[AP][C],
                                          const bool (&own)[AP], int64_t q0,
                                          int64_t q1, int lane) {
  static_assert(H == 1 || AP == 1, "two samples at once: up to 32 atoms");
  typedef const float __attribute__((address_space(1))) gfloat;
  constexpr int kSpan = kWave / H;
  auto wave_fence = []() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
  const Slots no_forces{nullptr, 0};
  const int n = L.n, K = L.K;
  const int hl = lane & (kSpan - 1), half = H == 2 ? lane >> 5 : 0;
  if (H == 2) pos += kSpan * half;
  const int ntc = (L.nt + kSpan - 1) / kSpan;
  const int nac = (L.na + kSpan - 1) / kSpan;
  const int nbc = (L.nb + kSpan - 1) / kSpan;
  for (int64_t q = q0; q < q1; q += H) {
    // the last sample again where the second half has none
    const int64_t qs = H == 2 && q + half >= q1 ? q : q + half;
    const gfloat* xq = (const gfloat*)J.xs + (size_t)(qs - J.first) * n * 3;
    float x[AP][3];
#pragma unroll
    for (int a = 0; a < AP; ++a)
#pragma unroll
      for (int d = 0; d < 3; ++d)
        x[a][d] = own[a] ? xq[(hl + kWave * a) * 3 + d] : 0.f;
#pragma unroll
    for (int a = 0; a < AP; ++a)
      if (own[a])
        pos[hl + kWave * a] = make_float4(x[a][0], x[a][1], x[a][2], m[a]);
    // the first atom's cell records load during the torsions, the second's
    // (AP = 2) during the angles and bonds: one record set in registers at a
    // time
    float psi[C];
#pragma unroll
    for (int c = 0; c < C; ++c) psi[c] = 0.f;
    Corners<C> cn;
    if (own[0]) grid_fetch<C>(g, x[0][0], x[0][1], x[0][2], cn);
    wave_fence();
    // bonded terms, energies only, every chunk of the ligand
    float eb[H] = {}, ea[H] = {}, et[H] = {};
    // (the two accumulators of H = 2 change places from chunk to chunk)
    auto chunks = [&](int nch, int items, float (&e)[H], auto term) {
#pragma unroll 1
      for (int ch = 0; ch < nch; ++ch) {
        const int t = ch * kSpan + hl;
        if (t < items) e[0] += term(t);
        if (H == 2) {
          const float first = e[0];
          e[0] = e[H - 1];
          e[H - 1] = first;
        }
      }
    };
    chunks(ntc, L.nt, et, [&](int t) {
      return torsion_term<false>(pos, sh.tijkl[t], sh.tpar[t], no_forces);
    });
    auto angles_bonds = [&]() {
      chunks(nac, L.na, ea, [&](int t) {
        return angle_term<false>(pos, sh.aijk[t], sh.apar[t], no_forces);
      });
      chunks(nbc, L.nb, eb, [&](int t) {
        return bond_term<false>(pos, sh.bij[t], sh.bpar[t], no_forces);
      });
    };
#pragma unroll
    for (int a = 0; a < AP; ++a) {
      if (own[a]) {
        float ev[C], dv[C][3];
        grid_finish<C, false>(g, cn, sc[a], ev, dv);
#pragma unroll
        for (int c = 0; c < C; ++c) psi[c] += ev[c];
      }
      if (a + 1 < AP && own[a + 1])
        grid_fetch<C>(g, x[a + 1][0], x[a + 1][1], x[a + 1][2], cn);
      if (a + 1 < AP) angles_bonds();
    }
    if (AP == 1) angles_bonds();
    // the centre of mass
    float px = 0.f, py = 0.f, pz = 0.f;
#pragma unroll
    for (int a = 0; a < AP; ++a) {
      px += m[a] * x[a][0];
      py += m[a] * x[a][1];
      pz += m[a] * x[a][2];
    }
    double U0b = (double)eb[0] + (double)ea[0] + (double)et[0];
    if (H == 2) U0b += (double)eb[H - 1] + (double)ea[H - 1] + (double)et[H - 1];
    double ps[C];
    if (H == 2) {
      px = half_sumf(px);
      py = half_sumf(py);
      pz = half_sumf(pz);
      U0b = half_sum(U0b);
#pragma unroll
      for (int c = 0; c < C; ++c) ps[c] = half_sum((double)psi[c]);
    } else {
      wave_sumf3(px, py, pz);
      U0b = wave_sum(U0b);
#pragma unroll
      for (int c = 0; c < C; ++c) ps[c] = wave_sum((double)psi[c]);
    }
    const float cx = px * L.inv_total_mass - L.site[0];
    const float cy = py * L.inv_total_mass - L.site[1];
    const float cz = pz * L.inv_total_mass - L.site[2];
    // fused as the block evaluation fuses it, whatever is inlined here
    const float d = sqrtf(fmaf(cz, cz, fmaf(cx, cx, cy * cy)));
    const float excess = d - L.d0;
    const double ui = excess > 0.f
                          ? 0.5 * (double)L.krest * (double)excess *
                                (double)excess
                          : 0.0;
    const double U0 = U0b + 0.0 + 0.0 + ui;
    // (a second half without a sample writes the first's column again)
    double* cs = col + (qs - q0) * K;
#pragma unroll 1
    for (int k = hl; k < K; k += kSpan) {
      double E = U0;
#pragma unroll
      for (int c = 0; c < C; ++c) E = fma(ew[k * C + c], ps[c], E);
      cs[k] = ew[K * C + k] * E;
    }
    // the next sample's position stores come after every lane's reads of
    // this one
    wave_fence();
  }
  // the group's columns, row by row: a run of consecutive samples of each row
  // by consecutive lanes
  wave_fence();
  const int cnt = (int)(q1 - q0);
  const int64_t n0 = q0 - J.first;
  auto out = BPMF_GMEM(double, J.ukn);
  if (cnt == kUknWaveGroup) {
#pragma unroll 2
    for (int i = lane; i < kUknWaveGroup * K; i += kWave) {
      const int k = i / kUknWaveGroup, qq = i % kUknWaveGroup;
      out[(size_t)k * J.ld + n0 + qq] = col[qq * K + k];
    }
  } else {
#pragma unroll 1
    for (int i = lane; i < cnt * K; i += kWave) {
      const int k = i / cnt, qq = i - k * cnt;
      out[(size_t)k * J.ld + n0 + qq] = col[qq * K + k];
    }
  }
  wave_fence();
}

// H: samples a wavefront takes at once, 0 by the ligand (launches with ligands
// on both sides of 32 atoms).
template <int C, int AP, int H>
__global__ __launch_bounds__(kUknWaves * kWave, C == 3 ? 4 : 3)
void k_energy_matrix_wave(
    GridDev g, const LigDev* __restrict__ ligs,
    const UknJob* __restrict__ jobs, int n_jobs, int64_t total) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid >> 6;
  int j, j_end;
  const int64_t b0 = ukn_share_start(jobs, n_jobs, blockIdx.x, gridDim.x, j);
  const int64_t b1 =
      ukn_share_start(jobs, n_jobs, blockIdx.x + 1, gridDim.x, j_end);
  if (b0 >= b1) return;
  typedef const float __attribute__((address_space(1))) gfloat;
  typedef const double __attribute__((address_space(1))) gcdouble;
  for (int64_t s = b0; s < b1; ++j) {
    const UknJob J = jobs[j];
    const int64_t e = jobs[j + 1].first < b1 ? jobs[j + 1].first : b1;
    if (s >= e) continue;  // empty job
    const LigDev L = ligs[J.lig];
    const int K = L.K, n = L.n;
    double* ew = reinterpret_cast<double*>(smem);
    unsigned char* slot =
        smem + ukn_wave_head_bytes(K, C) + wv * ukn_wave_slot_bytes(K, AP);
    float4* pos = reinterpret_cast<float4*>(slot);
    double* col = reinterpret_cast<double*>(slot + 16 * kWave * AP);
    unsigned char* topo = smem + ukn_wave_head_bytes(K, C) +
                          kUknWaves * ukn_wave_slot_bytes(K, AP);
    __syncthreads();  // the previous job's readers are done
    Shared sh{};
    stage_topology(L, topo, sh, tid, kUknWaves * kWave);
    for (int i = tid; i < K * (C + 1); i += kUknWaves * kWave)
      ew[i] = i < K * C ? ((gcdouble*)L.wd)[i]
                        : ((gcdouble*)L.beta)[i - K * C];
    __syncthreads();
    const bool two = H == 2 || (H == 0 && ukn_two_samples(n));
    float m[AP], sc[AP][C];
    bool own[AP];
#pragma unroll
    for (int a = 0; a < AP; ++a) {
      const int at = (two ? lane & (kWave / 2 - 1) : lane) + kWave * a;
      own[a] = at < n;
      m[a] = own[a] ? ((gfloat*)L.mass)[at] : 0.f;
#pragma unroll
      for (int c = 0; c < C; ++c)
        sc[a][c] = own[a] ? ((gfloat*)L.scale)[at * C + c] : 0.f;
    }
    // the wavefront's share: pairs of samples, in order
    const int64_t pairs = (e - s + 1) / 2;
    const int64_t s0 = s + 2 * (pairs * wv / kUknWaves);
    const int64_t s1 = wv + 1 < kUknWaves
                           ? s + 2 * (pairs * (wv + 1) / kUknWaves) : e;
    for (int64_t q0 = s0; q0 < s1; q0 += kUknWaveGroup) {
      const int64_t q1 = q0 + kUknWaveGroup < s1 ? q0 + kUknWaveGroup : s1;
      if constexpr (H != 1) {
        if (two) {
          ukn_group<C, AP, 2>(g, L, J, sh, ew, pos, col, m, sc, own, q0, q1,
                              lane);
          continue;
        }
      }
      if constexpr (H != 2)
        ukn_group<C, AP, 1>(g, L, J, sh, ew, pos, col, m, sc, own, q0, q1,
                            lane);
    }
    s = e;
  }
}

// ----------------------------------------------------------------------------
// exposed evaluator: terms and forces for arbitrary configurations/weights
// ----------------------------------------------------------------------------
template <int C, int W>
__global__ __launch_bounds__(W * kWave) void k_evaluate(
    GridDev g, const LigDev* __restrict__ lig, const float* __restrict__ xs,
    int64_t N, const double* __restrict__ wconf, double* __restrict__ terms,
    float* __restrict__ forces) {
  extern __shared__ __align__(16) unsigned char smem[];
  const LigDev L = *lig;
  const int tid = threadIdx.x;
  const int n = L.n;
  const Shared sh = carve<W>(smem, L, L.n, tid);
  const bool owner = tid < n;
  const float m = owner ? L.mass[tid] : 0.f;
  float sc[C];
#pragma unroll
  for (int c = 0; c < C; ++c) sc[c] = owner ? L.scale[tid * C + c] : 0.f;
  for (int64_t cf = blockIdx.x; cf < N; cf += gridDim.x) {
    float w[C];
#pragma unroll
    for (int c = 0; c < C; ++c) w[c] = (float)wconf[cf * C + c];
    float x[3], f[3];
    const float* xr = xs + (size_t)cf * n * 3;
#pragma unroll
    for (int d = 0; d < 3; ++d) x[d] = owner ? xr[tid * 3 + d] : 0.f;
    double t[6 + C];
    eval_block<C, W, true, true>(g, L, w, x, m, sc, f, t, 0.f, 0.f, sh, tid);
    if (tid == 0)
      for (int q = 0; q < 4 + C; ++q) terms[(size_t)cf * (4 + C) + q] = t[q];
    if (forces && owner) {
      float* fo = forces + (size_t)cf * n * 3;
#pragma unroll
      for (int d = 0; d < 3; ++d) fo[tid * 3 + d] = f[d];
    }
  }
}

// recompute cached components of every replica from its positions
template <int C, int W, bool PAIRS>
__global__ __launch_bounds__(W * kWave) void k_recompute(
    GridDev g, const LigDev* __restrict__ lig) {
  extern __shared__ __align__(16) unsigned char smem[];
  const LigDev L = *lig;
  const int tid = threadIdx.x;
  const int n = L.n;
  const Shared sh = carve<W>(smem, L, 0, tid);
  const int r = blockIdx.x;
  const bool owner = tid < n;
  const float m = owner ? L.mass[tid] : 0.f;
  float sc[C];
#pragma unroll
  for (int c = 0; c < C; ++c) sc[c] = owner ? L.scale[tid * C + c] : 0.f;
  float x[3], f[3];
  const float w0[C] = {};
#pragma unroll
  for (int d = 0; d < 3; ++d)
    x[d] = owner ? L.x[((size_t)r * n + tid) * 3 + d] : 0.f;
  double t[6 + C];
  eval_block<C, W, false, true, false, true, PAIRS ? kPairAhead : 0>(
      g, L, w0, x, m, sc, f, t, 0.f, 0.f, sh, tid);
  if (tid == 0) {
    double* cp = L.comps + (size_t)r * (1 + C);
    cp[0] = t[0] + t[1] + t[2] + t[3];
#pragma unroll
    for (int c = 0; c < C; ++c) cp[1 + c] = t[4 + c];
  }
}

// ----------------------------------------------------------------------------
// grid term alone, one thread per point
// ----------------------------------------------------------------------------
template <int C>
struct WeightsC {
  float w[C];
};

template <int C>
__global__ __launch_bounds__(256) void k_grid_eval(
    GridDev g, const float* __restrict__ pos, const float* __restrict__ scale,
    int64_t n, WeightsC<C> wc, float* __restrict__ energy,
    float* __restrict__ force) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    Corners<C> cn;
    grid_fetch<C>(g, pos[3 * i], pos[3 * i + 1], pos[3 * i + 2], cn);
    float s[C], e[C], de[C][3];
#pragma unroll
    for (int c = 0; c < C; ++c) s[c] = scale[i * C + c];
    grid_finish<C, true>(g, cn, s, e, de);
    if (energy)
#pragma unroll
      for (int c = 0; c < C; ++c) energy[i * C + c] = e[c];
    if (force) {
      float fx = 0.f, fy = 0.f, fz = 0.f;
#pragma unroll
      for (int c = 0; c < C; ++c) {
        fx -= wc.w[c] * de[c][0];
        fy -= wc.w[c] * de[c][1];
        fz -= wc.w[c] * de[c][2];
      }
      force[3 * i] = fx;
      force[3 * i + 1] = fy;
      force[3 * i + 2] = fz;
    }
  }
}

// cell-major records from the node-major grid (one thread per record float,
// pads zero)
__global__ __launch_bounds__(256) void k_expand_cells(
    const float* __restrict__ nodes, int nx, int ny, int nz, int C,
    float* __restrict__ cells) {
  const int stride = cell_stride(C);
  const size_t cx = nx - 1, cy = ny - 1;
  const size_t total = cx * cy * (size_t)(nz - 1) * stride;
  for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < total;
       e += (size_t)gridDim.x * blockDim.x) {
    const size_t cell = e / stride;
    const int o = (int)(e - cell * stride);
    float v = 0.f;
    if (o < 8 * C) {
      const int q = o / C, c = o - q * C;
      const size_t i = cell % cx + (q & 1);
      const size_t j = (cell / cx) % cy + ((q >> 1) & 1);
      const size_t k = cell / (cx * cy) + (q >> 2);
      v = nodes[((k * ny + j) * nx + i) * C + c];
    }
    cells[e] = v;
  }
}

int grid_blocks(int64_t work, int per_block, int cap) {
  int64_t b = (work + per_block - 1) / per_block;
  if (b < 1) b = 1;
  if (b > cap) b = cap;
  return (int)b;
}

}  // namespace

// ----------------------------------------------------------------------------
// launchers
// ----------------------------------------------------------------------------
#define BPMF_DISPATCH_C(C_, ...)                                   \
  switch (C_) {                                                    \
    case 3: {                                                      \
      constexpr int C = 3;                                         \
      __VA_ARGS__;                                                 \
    } break;                                                       \
    case 5: {                                                      \
      constexpr int C = 5;                                         \
      __VA_ARGS__;                                                 \
    } break;                                                       \
    default:                                                       \
      return hipErrorInvalidValue;                                 \
  }

#define BPMF_DISPATCH_W(W_, ...)                                   \
  switch (W_) {                                                    \
    case 1: {                                                      \
      constexpr int W = 1;                                         \
      __VA_ARGS__;                                                 \
    } break;                                                       \
    case 2: {                                                      \
      constexpr int W = 2;                                         \
      __VA_ARGS__;                                                 \
    } break;                                                       \
    case 4: {                                                      \
      constexpr int W = 4;                                         \
      __VA_ARGS__;                                                 \
    } break;                                                       \
    case 8: {                                                      \
      constexpr int W = 8;                                         \
      __VA_ARGS__;                                                 \
    } break;                                                       \
    default:                                                       \
      return hipErrorInvalidValue;                                 \
  }

hipError_t launch_hmc_sweep(const GridDev& g, const LigDev* d_ligs,
                            const int2* d_tasks, int n_tasks, int waves,
                            int lds_bytes, int nleap, uint64_t seed,
                            TailArgs tail, const LigDev* one, int pairs,
                            hipStream_t st) {
  if (n_tasks <= 0) return hipSuccess;
  const LigDev none{};
  const LigDev& arg = one ? *one : none;
#define BPMF_SWEEP(ONE_, PAIRS_)                                            \
  BPMF_DISPATCH_C(g.C, BPMF_DISPATCH_W(waves, {                             \
    hipLaunchKernelGGL((k_hmc_sweep<C, W, ONE_, PAIRS_>), dim3(n_tasks),    \
                       dim3(W * kWave), lds_bytes, st, g, d_ligs, d_tasks,  \
                       arg, nleap, seed, tail);                             \
  }))
  if (one && pairs == kPairShort) {  // on two wavefronts or more
    BPMF_SWEEP(true, (W > 1 ? kPairShort : kPairAhead));
  } else if (one && pairs) {
    BPMF_SWEEP(true, kPairAhead);
  } else if (one) {
    BPMF_SWEEP(true, 0);
  } else if (pairs == kPairShort) {
    BPMF_SWEEP(false, (W > 1 ? kPairShort : kPairAhead));
  } else if (pairs) {
    BPMF_SWEEP(false, kPairAhead);
  } else {
    BPMF_SWEEP(false, 0);
  }
#undef BPMF_SWEEP
  return hipGetLastError();
}

hipError_t launch_sweep_tail(const LigDev* d_ligs, int n_ligs,
                             int exchange_every, int scheme, int max_sep,
                             int n_sub, int sample_every, int walk,
                             uint64_t seed, hipStream_t st) {
  if (n_ligs <= 0) return hipSuccess;
  hipLaunchKernelGGL(walk == kWalkFar     ? k_sweep_tail<kWalkFar>
                     : walk == kWalkShort ? k_sweep_tail<kWalkShort>
                                          : k_sweep_tail<kWalkNear>,
                     dim3(n_ligs), dim3(kXThreads), 0, st, d_ligs,
                     exchange_every, scheme, max_sep, n_sub, sample_every,
                     seed);
  return hipGetLastError();
}

hipError_t launch_sweep_begin(const LigDev* d_ligs, int n_ligs,
                              hipStream_t st) {
  if (n_ligs <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_sweep_begin, dim3(n_ligs), dim3(256), 0, st, d_ligs);
  return hipGetLastError();
}

hipError_t launch_sweep_finish(const LigDev* d_ligs, int n_ligs,
                               int exchange_every, int sample_every,
                               uint64_t seed, hipStream_t st) {
  if (n_ligs <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_sweep_finish, dim3(n_ligs), dim3(256), 0, st, d_ligs,
                     exchange_every, sample_every, seed);
  return hipGetLastError();
}

hipError_t launch_exchange(const LigDev* d_lig, int n_ligs, int scheme,
                           int max_sep, int n_sub, int walk, uint64_t seed,
                           hipStream_t st) {
  if (n_ligs <= 0) return hipSuccess;
  hipLaunchKernelGGL(walk == kWalkFar     ? k_exchange<kWalkFar>
                     : walk == kWalkShort ? k_exchange<kWalkShort>
                                          : k_exchange<kWalkNear>,
                     dim3(n_ligs), dim3(kXThreads), 0, st, d_lig, scheme,
                     max_sep, n_sub, seed);
  return hipGetLastError();
}

namespace {
constexpr int kJobChunk = 32;
struct JobChunk {
  UknJob j[kJobChunk];
  int n;
};
__global__ __launch_bounds__(kJobChunk) void k_put_jobs(UknJob* dst,
                                                        JobChunk ch) {
  if ((int)threadIdx.x < ch.n) dst[threadIdx.x] = ch.j[threadIdx.x];
}
}  // namespace

hipError_t launch_put_jobs(UknJob* dst, const UknJob* jobs, int n,
                           hipStream_t st) {
  for (int first = 0; first < n; first += kJobChunk) {
    JobChunk ch;
    ch.n = n - first < kJobChunk ? n - first : kJobChunk;
    for (int i = 0; i < ch.n; ++i) ch.j[i] = jobs[first + i];
    hipLaunchKernelGGL(k_put_jobs, dim3(1), dim3(kJobChunk), 0, st,
                       dst + first, ch);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_energy_matrix(const GridDev& g, const LigDev* d_ligs,
                                int waves, const UknJob* d_jobs, int n_jobs,
                                int64_t total, int group, int lds_bytes,
                                int n_cu, bool pairs, bool per_wave,
                                int at_once, hipStream_t st) {
  if (total <= 0) return hipSuccess;
  if (per_wave) {
    if (waves != 1 && waves != 2) return hipErrorInvalidValue;
    if (waves == 2) at_once = 1;
    BPMF_DISPATCH_C(g.C, {
      auto kern = waves == 2     ? k_energy_matrix_wave<C, 2, 1>
                  : at_once == 2 ? k_energy_matrix_wave<C, 1, 2>
                  : at_once == 1 ? k_energy_matrix_wave<C, 1, 1>
                                 : k_energy_matrix_wave<C, 1, 0>;
      int per_cu = 0;
      hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
          &per_cu, kern, kUknWaves * kWave, lds_bytes);
      if (e != hipSuccess) return e;
      int64_t blocks = (int64_t)(per_cu > 0 ? per_cu : 1) * n_cu;
      // at least a group per wavefront
      const int64_t most =
          (total + kUknWaves * kUknWaveGroup - 1) / (kUknWaves * kUknWaveGroup);
      if (blocks > most) blocks = most;
      hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(kUknWaves * kWave),
                         lds_bytes, st, g, d_ligs, d_jobs, n_jobs, total);
    });
    return hipGetLastError();
  }
  BPMF_DISPATCH_C(g.C, BPMF_DISPATCH_W(waves, {
    auto kern = pairs ? k_energy_matrix<C, W, true>
                      : k_energy_matrix<C, W, false>;
    int per_cu = 0;
    hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
        &per_cu, kern, W * kWave, lds_bytes);
    if (e != hipSuccess) return e;
    int64_t blocks = (int64_t)(per_cu > 0 ? per_cu : 1) * n_cu;
    if (blocks > total) blocks = total;
    hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(W * kWave),
                       lds_bytes, st, g, d_ligs, d_jobs, n_jobs, total,
                       group);
  }));
  return hipGetLastError();
}

hipError_t launch_evaluate(const GridDev& g, const LigDev* d_lig,
                           int waves, const float* xs, int64_t N,
                           const double* w, double* terms, float* forces,
                           int lds_bytes, hipStream_t st) {
  if (N <= 0) return hipSuccess;
  const int blocks = grid_blocks(N, 1, 1 << 20);
  BPMF_DISPATCH_C(g.C, BPMF_DISPATCH_W(waves, {
    hipLaunchKernelGGL((k_evaluate<C, W>), dim3(blocks), dim3(W * kWave),
                       lds_bytes, st, g, d_lig, xs, N, w, terms, forces);
  }));
  return hipGetLastError();
}

hipError_t launch_recompute_comps(const GridDev& g, const LigDev* d_lig,
                                  int waves, int K, int lds_bytes, bool pairs,
                                  hipStream_t st) {
  if (pairs) {
    BPMF_DISPATCH_C(g.C, BPMF_DISPATCH_W(waves, {
      hipLaunchKernelGGL((k_recompute<C, W, true>), dim3(K), dim3(W * kWave),
                         lds_bytes, st, g, d_lig);
    }));
  } else {
    BPMF_DISPATCH_C(g.C, BPMF_DISPATCH_W(waves, {
      hipLaunchKernelGGL((k_recompute<C, W, false>), dim3(K), dim3(W * kWave),
                         lds_bytes, st, g, d_lig);
    }));
  }
  return hipGetLastError();
}

hipError_t launch_expand_cells(const float* nodes, int nx, int ny, int nz,
                               int C, float* cells, hipStream_t st) {
  const int64_t total =
      (int64_t)(nx - 1) * (ny - 1) * (nz - 1) * cell_stride(C);
  hipLaunchKernelGGL(k_expand_cells, dim3(grid_blocks(total, 256, 1 << 16)),
                     dim3(256), 0, st, nodes, nx, ny, nz, C, cells);
  return hipGetLastError();
}

hipError_t launch_grid_eval(const GridDev& g, const float* pos,
                            const float* scale, int64_t n, const double* w,
                            float* energy, float* force, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  const int blocks = grid_blocks(n, 256, 1 << 20);
  BPMF_DISPATCH_C(g.C, {
    WeightsC<C> wc;
    for (int c = 0; c < C; ++c) wc.w[c] = (float)w[c];
    hipLaunchKernelGGL((k_grid_eval<C>), dim3(blocks), dim3(256), 0, st, g,
                       pos, scale, n, wc, energy, force);
  });
  return hipGetLastError();
}

}  // namespace bpmf
