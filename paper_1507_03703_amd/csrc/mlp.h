// Learned pose proposal: network shape, parameter layout, device state and
// launchers (mlp.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "internal.h"

namespace bpmf {

constexpr int kNFeat = 16, kNHid = 256, kNComp = 8, kNOut = kNComp * 13;
constexpr int kFold = 3;  // preimages (theta + 2 pi m) n, m = -3..3
constexpr float kSt0 = 0.02f, kSt1 = 3.0f;  // translation sigma range (A)
constexpr float kSw0 = 0.02f, kSw1 = 1.5f;  // rotation sigma range (rad)

// flat fp32 parameter vector: W1 (16x256) b1 W2 (256x256) b2 W3 (256x104) b3,
// weights row-major [in][out]
constexpr int kOffW1 = 0;
constexpr int kOffB1 = kOffW1 + kNFeat * kNHid;
constexpr int kOffW2 = kOffB1 + kNHid;
constexpr int kOffB2 = kOffW2 + kNHid * kNHid;
constexpr int kOffW3 = kOffB2 + kNHid;
constexpr int kOffB3 = kOffW3 + kNHid * kNOut;
constexpr int kNParams = kOffB3 + kNOut;

// bf16 copy of the weights for the forward pass, each matrix
// transposed ([out][in]) with rows padded so that a lane's eight
// consecutive k values are one 16-byte load and every 16-column output tile
// is in range: W1^T 256 x 32, W2^T 256 x 256, W3^T 112 x 256 (padding 0)
constexpr int kT1Ld = 32, kT2Ld = kNHid, kT3Ld = kNHid, kT3Rows = 112;
constexpr int kTOff1 = 0;
constexpr int kTOff2 = kTOff1 + kNHid * kT1Ld;
constexpr int kTOff3 = kTOff2 + kNHid * kT2Ld;
// the same of W2 and W3 row by row, for the backward pass: W2 256 x 256, W3
// 256 x 128 (padding 0)
constexpr int kR3Ld = 128;
constexpr int kTOffR2 = kTOff3 + kT3Rows * kT3Ld;
constexpr int kTOffR3 = kTOffR2 + kNHid * kNHid;
constexpr int kTSize = kTOffR3 + kNHid * kR3Ld;

// rows of a minibatch's transposed bf16 activations (Bp elements each):
// features, H1, H2, dout, dZ2, dZ1; and the biases (b1, b2, b3)
constexpr int kActF = 0, kActH1 = kNFeat, kActH2 = kActH1 + kNHid,
              kActD = kActH2 + kNHid, kActZ2 = kActD + kT3Rows,
              kActZ1 = kActZ2 + kNHid, kActRows = kActZ1 + kNHid;
constexpr int kNBias = 2 * kNHid + kNOut;

enum Purpose2 : uint32_t { kPose = 4, kBatch = 5 };

// Device state of one ligand's proposal.
struct PropDev {
  int frame[3];
  int n_cond;
  int4 cond[8];
  unsigned long long* pose_acc;  // K
  unsigned long long* pose_try;  // K
  double* last_ln_alpha;         // K, ln alpha of each replica's last move
};

// One replica of a batch of pose moves over several ligands: its ligand's
// table index, the replica, and its row in the batch's features, poses and
// network outputs.
struct PoseTask {
  int lig, r, row, pad;
};

// One workgroup of a batched forward pass: rows [row0, row0 + rows) (at
// most 16) through the network whose parameters start at P.
struct MlpGroup {
  const float* P;             // fp32 parameters (the biases are read here)
  const unsigned short* WT;   // bf16 weights (kTSize)
  int row0, rows;
};

// One gradient of the mean negative log-likelihood over B rows (Bp: rounded
// up to 32).  gather: row i is training row philox(step, i) mod N of feats
// and poses; else row i.
struct TrainArgs {
  const float* P;          // fp32 parameters (the biases are read here)
  unsigned short* WT;      // bf16 copies of the weights (kTSize)
  const float* feats;      // N x kNFeat
  const float* poses;      // N x 6
  int64_t N;
  int B, Bp;
  bool gather;
  uint64_t seed, step;
  float inv_b;             // 1 / B
  unsigned short* act;     // kActRows x Bp transposed activations
  double* biasP;           // Bp / 16 x kNBias column sums per row block
  double* lossP;           // Bp / 16 loss sums per row block
};
// Where a gradient goes: into G, or (G null) into an Adam step of P with
// moments m and v (c1, c2: the bias corrections)
struct AdamArgs {
  float* G;
  float *P, *m, *v;
  float lr, b1, b2, eps, c1, c2;
};
// out = network(X) for B rows (features B x kNFeat, outputs B x kNOut)
hipError_t launch_mlp_forward(const float* P, const unsigned short* WT,
                              const float* X, int B, float* out,
                              hipStream_t st);
// one gradient or Adam step; *loss (device) = the rows' summed loss; split:
// train_splits(Bp) x kNParams floats when that is more than one
int train_splits(int Bp);
hipError_t launch_train_step(const TrainArgs& a, const AdamArgs& w,
                             float* split, double* loss, hipStream_t st);
// n: the ligand's atoms
hipError_t launch_pose_features(const LigDev* lig, const PropDev* prop, int n,
                                const float* xs, int64_t N, float* feats,
                                float* poses, hipStream_t st);
// the network on the current configurations of tasks [row0, row0 + rows)
// of every group (features computed in place), outputs only; n_fin further
// blocks close the neighbour-scheme run of ligands fin[0..n_fin) as
// launch_sweep_finish does
hipError_t launch_pose_network(const MlpGroup* groups, int n_groups,
                               const LigDev* ligs, const PropDev* props,
                               const PoseTask* tasks, float* out,
                               const LigDev* fin, int n_fin,
                               int exchange_every, int sample_every,
                               uint64_t seed, hipStream_t st);
// the bf16 copies of the weights of parameter vector P
hipError_t launch_weights_bf16(const float* P, unsigned short* WT,
                               hipStream_t st);
// one pose move of each of the n tasks (all of `waves` wavefronts; props
// indexed by ligand table index, out by task row); begin_next: each task's
// replica then starts the next run of neighbour-scheme sweeps
// (begin_replica), in place of launch_sweep_begin
hipError_t launch_pose_move(const GridDev& g, const LigDev* ligs,
                            const PropDev* props, const PoseTask* tasks,
                            int n, const float* out, int waves, int lds,
                            uint64_t seed, bool begin_next, hipStream_t st);

}  // namespace bpmf
