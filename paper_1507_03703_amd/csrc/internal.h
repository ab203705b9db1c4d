// Structures shared by the host side of libbpmf and its gfx950 kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "pairs.h"

namespace bpmf {

constexpr int kWave = 64;
constexpr double kRGas = 8.314462618e-3;  // kJ/(mol K)
#define BPMF_MAX_MBAR_STATES_DEV 128
constexpr int kRedSlots = 4 + 8 + 2;  // per-wave partial sums (see Shared)

// copies of the fixed-point force accumulators: a bonded-term lane adds
// into copy (lane mod kAccCopies), which divides the lanes of one LDS
// atomic instruction that meet the same atom among that many addresses
constexpr int kAccCopies = 4;

// LDS bytes of the fixed-point force accumulators (kAccCopies x n x 3
// int32), rounded up to 16 so that the topology staged after them stays
// 16-byte aligned
__host__ __device__ inline int acc_lds_bytes(int n) {
  return (kAccCopies * 12 * n + 15) & ~15;
}

// Bonded terms are taken in chunks of 64 terms of one kind (a wavefront
// takes a chunk in one pass): torsion chunks, then angle chunks, then bond
// chunks.  The schedule of a ligand gives, for each launch width (1, 2, 4,
// 8 wavefronts), the chunks of each wavefront: a row of 9 offsets
// (wavefront w takes entries off[w] .. off[w+1]-1) followed by the chunk
// ids, stored as 16-bit values.
__host__ __device__ inline int bonded_chunks(int nb, int na, int nt) {
  return (nt + kWave - 1) / kWave + (na + kWave - 1) / kWave +
         (nb + kWave - 1) / kWave;
}
__host__ __device__ inline int sched_row(int nb, int na, int nt) {
  return 9 + bonded_chunks(nb, na, nt);
}

// dynamic LDS bytes of a W-wave evaluation block: per-evaluation areas,
// force accumulators (forces only), the staged topology (with the schedule
// row of this width) and, with pair terms in the energy, the pair
// parameters and scratch
__host__ __device__ inline int block_lds_bytes(int waves, bool forces, int n,
                                                int nb, int na, int nt,
                                                bool pairs = false) {
  const int head = 16 * kWave * waves + 8 * waves * kRedSlots + 16 * waves +
                   (forces ? acc_lds_bytes(n) : 0);
  const int topo = 32 * nt + 24 * na + 16 * nb +
                   ((2 * sched_row(nb, na, nt) + 15) & ~15);
  return head + topo + (pairs ? pair_lds_bytes(n, waves) : 0);
}

// LDS of a k_energy_matrix_wave block: the states' weights and beta_k, then
// per wavefront its positions (64 AP float4) and the columns of a group of
// kUknWaveGroup samples, then the ligand's topology (as stage_topology lays
// it out)
constexpr int kUknWaves = 4, kUknWaveGroup = 8;
// a wavefront takes two samples at once
__host__ __device__ constexpr bool ukn_two_samples(int n) { return n <= 32; }
__host__ __device__ inline int ukn_wave_head_bytes(int K, int C) {
  return (K * (C + 1) * 8 + 15) & ~15;
}
__host__ __device__ inline int ukn_wave_slot_bytes(int K, int ap) {
  return 16 * kWave * ap + kUknWaveGroup * K * 8;
}
__host__ __device__ inline int ukn_wave_lds_bytes(int K, int C, int ap,
                                                  int nb, int na, int nt) {
  return ukn_wave_head_bytes(K, C) + kUknWaves * ukn_wave_slot_bytes(K, ap) +
         32 * nt + 24 * na + 16 * nb +
         ((2 * sched_row(nb, na, nt) + 15) & ~15);
}

enum Purpose : uint32_t { kMomenta = 1, kAccept = 2, kExchange = 3 };

// Floats per cell record of the cell-major grid: the 8 corners x C channels
// rounded up to a power of two, so that a record of up to 4 channels is one
// aligned 128-byte cache line.
constexpr int cell_stride(int C) {
  return 8 * C <= 8 ? 8 : 8 * C <= 16 ? 16 : 8 * C <= 32 ? 32 : 64;
}

// Receptor grid as the kernels see it, cell-major: cell (i, j, k) (i < nx-1,
// j < ny-1, k < nz-1) owns the record at cells + ((k*(ny-1) + j)*(nx-1) + i)
// * cell_stride(C) holding the values of its corners, corner q = (i + (q&1),
// j + ((q>>1)&1), k + (q>>2)) at [q*C + c] for channel c.  Each node value
// appears in up to 8 records: one interpolation reads one record instead of
// 8 scattered corners.  Channel c holds a quartic root when bit c of
// quartic_mask is set.
struct GridDev {
  const float* cells;
  int nx, ny, nz, C;
  float ox, oy, oz, inv_h;
  int quartic_mask;
};

// One ligand: force field, state ladder, replica state, statistics and the
// sample store, all resident in device memory.  Replica r of a ligand with
// K states owns x[r*n*3 .. (r+1)*n*3).
struct LigDev {
  int n, K, C;
  int nb, na, nt, n_slots;
  int id;     // ligand id (enters the random-number counter)
  int cap;    // recorded samples per state
  float site[3];
  float d0, krest, inv_total_mass;
  const float* mass;      // n
  const float* inv_mass;  // n
  const float* scale;     // n*C
  const int2* bij;        // nb
  const float2* bpar;     // nb: K_r, r0
  const int4* aijk;       // na: i, j(vertex), k, -
  const float2* apar;     // na: K_theta, theta0
  const int4* tijkl;      // nt
  const float4* tpar;     // nt: V/2, n (integer 1..6), cos gamma, sin gamma
  const unsigned short* bsched;  // 4 x sched_row: bonded chunks per wavefront
  const double* beta;     // K: 1/(R T_k)
  const float* Tf;        // K
  const float* dtf;       // K
  const float* wf;        // K*C
  const double* wd;       // K*C
  float* x;               // K*n*3
  double* comps;          // K*(1+C)
  int* state_of_replica;  // K
  int* replica_of_state;  // K
  unsigned long long* counter;    // sweeps done
  unsigned long long* n_rec;      // recorded rounds
  unsigned long long* hmc_acc;    // K
  unsigned long long* hmc_try;    // K
  unsigned long long* ex_acc;     // max(K-1,1)
  unsigned long long* ex_try;     // max(K-1,1)
  unsigned long long* nonfinite;  // 1
  unsigned long long* ext_acc;    // K: external moves accepted per state
  unsigned long long* ext_try;    // K: external moves tried per state
  // Neighbour-scheme sweeps apply the exchange (and record) that ends sweep
  // s-1 at the start of sweep s, in every replica's own block: sweep s
  // reads buffer (s-1)&1 and writes buffer s&1 (k_sweep_begin fills the
  // first from the canonical arrays above, k_sweep_finish applies the last
  // pending exchange and writes them back).
  unsigned long long* rcnt;   // K: sweep counter of each replica
  unsigned long long* rnrec;  // K: recorded rounds seen by each replica
  int* rpend;                 // 2K: exchange/record of the previous sweep due
  int* rsor;                  // 2K: state of each replica
  double* scomp;              // 2K(1+C): components of the replica in each state
  // start-of-trajectory force reuse: per replica two slots of the parts of
  // the force at its current positions that do not depend on the state
  // (per atom: bonded force, grid gradients of every channel; per replica:
  // restraint factor and centre-of-mass offset); fvalid[r] = 0 (none) or
  // 1 + the slot holding the current positions' parts
  float* fcache;              // 2K x n x (3 + 3C)
  float* frc;                 // 2K x 4
  int* fvalid;                // K
  float* samp_x;                  // cap*K*n*3
  double* samp_c;                 // cap*K*(1+C)
  // intramolecular nonbonded and OBC GB/SA terms in the sampled energy
  // (bpmf_pair_sample): on when pairs_on, parameters in `pair`
  int pairs_on;
  PairDev pair;
};

// Every region of a ligand's device arena starts on a 256-byte boundary.
constexpr size_t kArenaAlign = 256;

// Round-trip bookkeeping (kept out of the table, whose every field the
// sweep kernel holds in scalar registers), in the arena region right after
// fvalid: per replica the extreme state it last visited on its way (0 =
// state 0, 1 = state K-1, -1 = neither yet), then, 8-byte aligned, the
// ligand's trip count.
__host__ __device__ inline int* rt_end_of(const LigDev& L) {
  const size_t b = ((size_t)L.K * 4 + kArenaAlign - 1) & ~(kArenaAlign - 1);
  return (int*)((char*)L.fvalid + b);
}
__host__ __device__ inline unsigned long long* round_trips_of(
    const LigDev& L) {
  return (unsigned long long*)(rt_end_of(L) + ((L.K + 1) & ~1));
}
__host__ __device__ inline size_t rt_region_bytes(int K) {
  return (size_t)((K + 1) & ~1) * 4 + 8;
}

// Launch wrappers (kernels.hip).  All return hipError_t of the launch.
// waves = wavefronts per replica (1, 2 or 4); n_atoms <= 64 * waves
// exchange/record schedule of a sweep (scheme 0: deferred into the next
// sweep's blocks; scheme 1: a tail kernel after every sweep, running
// exchange_sweeps exchange sweeps when an exchange is due)
struct TailArgs {
  int exchange_every, scheme, max_sep, sample_every, exchange_sweeps;
};
// one: the host copy of the table entry when the launch covers a single
// ligand (its replicas 0..n_tasks-1 in order), else null
// pairs: partners at once (the most pair_at_once of the launch's ligands with
// their pair terms in the energy; 0: none has)
hipError_t launch_hmc_sweep(const GridDev& g, const LigDev* d_ligs,
                            const int2* d_tasks, int n_tasks, int waves,
                            int lds_bytes, int nleap, uint64_t seed,
                            TailArgs tail, const LigDev* one, int pairs,
                            hipStream_t st);
hipError_t launch_sweep_tail(const LigDev* d_ligs, int n_ligs,
                             int exchange_every, int scheme, int max_sep,
                             int n_sub, int sample_every, int walk,
                             uint64_t seed, hipStream_t st);
hipError_t launch_sweep_begin(const LigDev* d_ligs, int n_ligs,
                              hipStream_t st);
hipError_t launch_sweep_finish(const LigDev* d_ligs, int n_ligs,
                               int exchange_every, int sample_every,
                               uint64_t seed, hipStream_t st);
// n_sub exchange sweeps in a row (sweep j draws with replica field j)
hipError_t launch_exchange(const LigDev* d_lig, int n_ligs, int scheme,
                           int max_sep, int n_sub, int walk, uint64_t seed,
                           hipStream_t st);
// All-separations exchange of K states: up to this separation the residue
// classes are walked by a wavefront each, eight at a time; past it, where there
// are many classes of few states, by a lane each.  The line is where
// both cost the same: a wavefront's walk of a class costs 0.7 us however short
// the class, all lanes' walks together 0.3 to 1 us by its length.  One sweep
// over every separation, a wavefront for each class and this way: 64 states
// 244 and 87 us, 170 states 1433 and 250 us, 256 states 3096 and 418 us (549 us
// with one lane per first state following its run); up to 12 separations of
// 16 states, five sweeps: 110 and 89 us; of 256 states: 173 us by wavefronts,
// 248 us by lanes.
__host__ __device__ constexpr int exchange_wave_separations(int K) {
  return K <= 64 ? 8 : K <= 192 ? 16 : 24;
}
// The kernels of the exchange (`walk` above), by the ladders of a launch: with
// some ladder past its line, with short ladders only, and the others.  A
// wavefront doubles its steps along a class three times before it takes them;
// up to eight positions the steps themselves cost less (up to 5 separations, 25
// sweeps, doublings always and not there: 4 states 101 and 95 us, 16 states 175
// and 165 us, 32 states 186 and 184 us), but the test costs the longer ladders
// more than they gain (64 states 194 and 199 us).
enum ExchangeWalk : int { kWalkNear = 0, kWalkFar = 1, kWalkShort = 2 };
inline int exchange_walk(int K, int max_sep) {
  if ((max_sep < K - 1 ? max_sep : K - 1) > exchange_wave_separations(K))
    return kWalkFar;
  return K <= 32 ? kWalkShort : kWalkNear;
}
// one ligand's share of an energy-matrix launch: samples xs (n x n_atoms x
// 3), output u_kn (K x ld); its samples are [first, first + n) of the
// launch's flat sample index
struct UknJob {
  int lig;   // index into the ligand table
  int cost;  // estimated cost of one sample (instruction-issue units)
  const float* xs;
  double* ukn;
  int64_t n, ld;
  int64_t first;   // flat index of the job's first sample
  int64_t cfirst;  // cost of the launch's samples before the job's first
};
// d_jobs: n_jobs jobs in flat order, every ligand needing `waves`
// wavefronts, then a sentinel with first = total and cfirst = the launch's
// total cost (each block takes a contiguous share of equal cost); group = samples whose
// columns are staged in LDS before they are written.  per_wave: one
// wavefront per sample (k_energy_matrix_wave, for ligands whose pair terms
// are not in the energy; `waves` is then the atoms per lane, 1 or 2, and
// lds_bytes comes from ukn_wave_lds_bytes); at_once: samples a wavefront takes
// at once at one atom per lane, ukn_two_samples of every ligand of the launch
// (2, 1) or 0 where they differ
hipError_t launch_energy_matrix(const GridDev& g, const LigDev* d_ligs,
                                int waves, const UknJob* d_jobs, int n_jobs,
                                int64_t total, int group, int lds_bytes,
                                int n_cu, bool pairs, bool per_wave,
                                int at_once, hipStream_t st);
// copy n jobs from host memory into the device table dst by kernels that
// take the jobs as arguments (no host staging buffer, no copy engine)
hipError_t launch_put_jobs(UknJob* dst, const UknJob* jobs, int n,
                           hipStream_t st);
hipError_t launch_evaluate(const GridDev& g, const LigDev* d_lig,
                           int waves, const float* xs, int64_t N,
                           const double* w, double* terms, float* forces,
                           int lds_bytes, hipStream_t st);
// cell-major records (GridDev) from a node-major grid nodes[((k*ny + j)*nx +
// i)*C + c]
hipError_t launch_expand_cells(const float* nodes, int nx, int ny, int nz,
                               int C, float* cells, hipStream_t st);
hipError_t launch_grid_eval(const GridDev& g, const float* pos,
                            const float* scale, int64_t n, const double* w,
                            float* energy, float* force, hipStream_t st);
hipError_t launch_recompute_comps(const GridDev& g, const LigDev* d_lig,
                                  int waves, int K, int lds_bytes, bool pairs,
                                  hipStream_t st);

// MBAR kernels (mbar.hip).  One entry per problem of a batch, in device
// memory, ordered by tile count; a launch covers a run of them, blockIdx.y
// each.
// What a problem waits for: the sums at its start, at a trial, at a
// fixed-point update (whose values k_self_consistent forms first), nothing.
enum MbarPhase : int {
  kMbarStart = 0,
  kMbarSearch = 1,
  kMbarFixed = 2,
  kMbarDone = 3
};
struct MbarState {
  int phase;
  int it;      // current iteration (1-based)
  int ls;      // line-search trials made in this iteration
  int n_iter;  // iterations taken, once done
  double trust, Fcur, t, maxstep, gs;
};
// 16-row tiles of the weights' product, and the doubles of one block's
// partial sums: the objective's sum (padded), column sums, then the lower
// triangle's tiles
constexpr int kMbarHead = 16;
__host__ __device__ inline int mbar_tiles(int K) { return (K + 15) / 16; }
__host__ __device__ inline int mbar_width(int K) {
  const int nt = mbar_tiles(K);
  return kMbarHead + 16 * nt + 256 * (nt * (nt + 1) / 2);
}
struct MbarProb {
  const double* ukn;  // K x N, leading dimension ld
  int64_t N, ld;
  int K;
  int nb;             // blocks of the pass over u_kn
  double* f;          // K current point (f_0 = 0)
  double* ftry;       // K line-search trial
  double* logN;       // K
  double* Nk;         // K
  double* logD;       // N
  double* partial;    // nb x mbar_width(K)
  double* red;        // mbar_width(K) reduced sums
  double* step;       // K Newton step / fixed-point values
  double* var;        // K variances
  double* iter;       // iterations taken (result)
  MbarState state;
};
constexpr int kMbarNarrow = 3;  // tiles a wavefront keeps to itself
int mbar_blocks(int K, int64_t N);
// One round: every problem's sums at the point its phase asks for (every
// problem of the run has nt = mbar_tiles(K)) ...
hipError_t mbar_sums(MbarProb* P, int n, int nt, int max_blocks,
                     hipStream_t st);
// ... their reduction ...
hipError_t mbar_reduce(MbarProb* P, int n, int max_K, hipStream_t st);
// ... the decision and the next step (every problem of the run has nt or
// nt - 1 tiles, nt even); the last of the call's n_all problems to be done
// (*n_done counts them) sets *host_done ...
hipError_t mbar_step(MbarProb* P, int n, int nt, double tol, int max_iter,
                     int* n_done, int n_all, volatile int* host_done,
                     hipStream_t st);
// ... and the fixed-point values of those whose Hessian was singular.
hipError_t mbar_self_consistent(MbarProb* P, int n, int max_K,
                                hipStream_t st);

}  // namespace bpmf
