// Internal launch interfaces between the C-ABI host layer and the kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "rehyat_device.h"

namespace rehyat {

// ---- chunk-state kernel: partial sums of phi_k(K)^T V and phi_k(K) ----------
// Segment s of a window is the token range that enters the linear set between
// chunk (chunk0 + s) and the next one, [s_lo(chunk0+s), s_lo(chunk0+s+1))
// (Eq. 13, Eq. 17-18); each segment is cut into `nsplit` pieces, one workgroup
// per (batch*head, segment, piece).
struct StateArgs {
  const bf16_t* k;      // [BH, N, d]
  const bf16_t* v;      // [BH, N, d]
  const bf16_t* w1_k;   // [H, hidden, d]
  const float* b1_k;    // [H, hidden]
  const bf16_t* w2_k;   // [H, dprime, hidden]
  const float* b2_k;    // [H, dprime]
  float* partial;       // [BH, partial_slots, d*dprime + dprime] (S^T [d][dprime], then z)
  int H, T, HW, chunk, overlap;
  int chunk0;           // first chunk of the window
  int n_seg;            // segments computed in this launch
  int nsplit;           // pieces per segment
  int partial_slots;    // slot stride per (b, h)
  int n_items;          // BH * n_seg * nsplit
  int items_per_xcd;
  int64_t kv_bh_stride; // elements between the k (and v) rows of consecutive (b, h)
  int step_n;           // > 0: one segment, rows [0, step_n) of k / v (streaming step); the
                        // frame geometry above is then unused
  // Gradient of the chunk state (k = q, v = G): segment s is the query range [q_lo, q_hi) of chunk chunk0 + s, and the
  // sums are those of (tok_scale phi_q(q)) G^T and tok_weight phi_q(q).
  const float* tok_scale;    // [BH, N] 1 / den
  const float* tok_weight;   // [BH, N] w
};

// pieces in flight per thread of the prefix and suffix passes
constexpr int kScanDepth = 8;

// ---- prefix kernel: states S_t, z_t of the window's chunks ---------------------
struct PrefixArgs {
  const float* partial;  // as written by the state kernel
  float* carry;          // [BH, d*dprime + dprime] fp32, state at the window's first chunk
  bf16_t* state_s;       // [BH, state_slots, d, dprime] bf16 (S_t transposed)
  float* state_z;        // [BH, state_slots, dprime]
  int BH;
  int n_chunks;          // chunks in the window (states written)
  int n_seg;             // segments available (n_chunks or n_chunks - 1)
  int nsplit;
  int partial_slots, state_slots;
  int first_window;      // 1: state at the window's first chunk is zero (Eq. 14-15)
  int elems;             // d*dprime + dprime
  int s_elems;           // d*dprime
};

// ---- fused softmax + read-out + merge kernel -----------------------------------
struct AttnArgs {
  const bf16_t *q, *k, *v;
  bf16_t* out;
  const bf16_t* w1_q;
  const float* b1_q;
  const bf16_t* w2_q;
  const float* b2_q;
  const bf16_t* state_s;  // [BH, state_slots, d, dprime]
  const float* state_z;   // [BH, state_slots, dprime]
  float *dbg_m, *dbg_nS, *dbg_aS, *dbg_nL, *dbg_aL;
  float scale_log2e;      // log2(e) / sqrt(d)
  int H, T, HW, chunk, overlap;
  int chunk0;            // first chunk of the window
  int qtiles;            // query tiles per (full) chunk
  int bh_items;          // query tiles of the window's chunks; only the last one can have fewer than
                         // qtiles (counted as a full one, its missing tiles left some XCDs with
                         // less work: 3 heads of 61 frames in chunks of five 4,270 us, now 3,994)
  int state_slots;
  int stab_mode;
  int n_items, items_per_xcd;
  int n_short;           // > 0: the window's first chunk is chunk 0 (no linear part); its n_short
                         // = BH * qtiles items run last on every XCD (items_per_xcd then counts
                         // ceil(long / 8) + ceil(short / 8))
  int64_t q_bh_stride;   // elements between the q (and out) rows of consecutive (b, h)
  int64_t kv_bh_stride;  // same for k and v
  int step_nq, step_nwin;  // step_nq > 0 (streaming step): queries are rows [0, step_nq) of q,
                           // the softmax window is rows [0, step_nwin) of k / v, the linear
                           // state is slot 0; the frame geometry above is then unused
  const float *step_S, *step_z;   // streaming step with the split kernel: the caller's S [BH, dprime, d]
                                  // and z [BH, dprime] (then no slot is read); otherwise null
  int all_linear;          // 1: every chunk reads a state (bidirectional sets of Eq. 11-12)
  unsigned xcd_mask;       // measurement hook: workgroups on XCD x (index % 8) run only if bit x is set
};

// ---- transposes the carry into the [dprime][d] layout of the public state hook ----
struct StateOutArgs {
  const float* carry;  // [BH, d*dprime + dprime], S^T [d][dprime] then z
  float* S_out;        // [BH, dprime, d]
  float* z_out;        // [BH, dprime]
  int BH, d, dprime;
};

// ---- bidirectional states: everything outside each chunk's softmax window -----------
// state(c) = total - sum of the per-frame sums of the frames inside window c (Eq. 11-12);
// the per-frame sums of frames [frame0, frame0 + n_frames) are in `partial`
// (frame-major, nsplit pieces each), the total over all frames is in `total`, or (sum_total) is formed
// here first, when all T frames are in `partial`, and left there.
struct BidirArgs {
  const float* partial;
  float* total;          // [BH, d*dprime + dprime]
  int sum_total;
  bf16_t* state_s;       // [BH, state_slots, d, dprime]
  float* state_z;        // [BH, state_slots, dprime]
  int BH, T, chunk, overlap;
  int chunk0, n_chunks;  // chunks of this window -> state slots 0 .. n_chunks-1
  int frame0;            // first frame held in `partial`
  int nsplit, partial_slots, state_slots;
  int elems, s_elems;
};

// ---- streaming step: the caller's state feeds the read-out and absorbs the step's pieces ----
// state slot 0 <- the caller's S, z as they are on entry (bf16 S^T [d][dprime] and fp32 z: what
// Eq. 16 reads for this chunk); then S, z += the pieces the chunk-state kernel wrote (Eq. 17-18),
// in place, in the caller's layout.
struct StepStateArgs {
  float* S;              // [BH, dprime, d]   read and written
  float* z;              // [BH, dprime]      read and written
  const float* partial;  // [BH, partial_slots, d*dprime + dprime]: S^T [d][dprime], then z
  bf16_t* state_s;       // [BH, state_slots, d, dprime]
  float* state_z;        // [BH, state_slots, dprime]
  int BH, d, dprime;
  int nsplit;            // pieces to add (0: the state is only copied into slot 0)
  int partial_slots, state_slots;
  int write_slot;        // 1: slot 0 <- the state as it is before the pieces are added
};

// =================================================================================
// Gradient of the output with respect to the feature-map parameters: one step of the
// attention distillation of section 3.4 (Eq. 19) trains only phi_q and phi_k.
// With G = dL/dy_hat, den_i = n^S_i + n^L_i, u_i = G_i / den_i, w_i = -(G_i . y_i) / den_i:
//   dL/dPhi_q,i = S_t u_i + w_i z_t                 (queries of chunk t)
//   dL/dS_t = sum_i Phi_q,i u_i^T ,  dL/dz_t = sum_i w_i Phi_q,i
// (u is never written: the kernels read G, and scale Phi and S_t G by 1 / den)
//   dL/dPhi_k,j = R_tau v_j + r_tau ,  R_tau = sum_{t > tau} dL/dS_t ,  r_tau likewise,
// for keys j of segment tau = [s_lo(tau), s_lo(tau+1)) (Eq. 13: they belong to the linear
// set of every later chunk), followed by the backward pass of the two-layer map.
// =================================================================================

// 1 / den and w = -(G . y) / den per token
struct PrepArgs {
  const bf16_t* g;    // [tokens, d] upstream gradient
  const bf16_t* y;    // [tokens, d] forward output
  const float* nS;    // [tokens]
  const float* nL;    // [tokens]
  float* inv;         // [tokens]
  float* tokw;        // [tokens]
  const bf16_t* w2_q; // [H, 2d, 2d]
  const bf16_t* w2_k;
  bf16_t* w2t;        // [2, H, 2d, 2d]  each matrix of w2_q, then of w2_k, transposed
  int64_t tokens;
  int H, d;
};

// R_tau, r_tau: sums over the later chunks of the chunk-state gradients
struct SuffixArgs {
  const float* part;    // [BH, part_slots, elems]: segment s, piece p at slot s*nsplit + p
  bf16_t* Rt;           // [BH, slots, d, dp]  (transposed, as the forward chunk states)
  float* r;             // [BH, slots, dp]
  int BH, n_seg, nsplit, part_slots, slots;
  int elems, s_elems, dp;
};

// Activation gradients of one side (queries or keys): recomputes U = relu(W1 x + b1) and
// psi = relu(W2 U + b2), forms dPhi = inv * M vec + tokw * zv for the token's segment, and writes
// dpsi = dPhi * dphi/dpsi token-major for the weight-gradient kernels.
struct ActGradArgs {
  const bf16_t* x;      // [BH, N, d]  q or k
  const bf16_t* vec;    // [BH, N, d]  G (query side) or v (key side)
  const float* tokw;    // [BH, N] per-token weight of zv and scale of M vec (query side); unused on the key side (1)
  const float* inv;
  const bf16_t* w1;
  const float* b1;
  const bf16_t* w2;
  const float* b2;
  const bf16_t* M;      // [BH, slots, d, dp]  S_t (query side) or R_tau (key side), transposed
  const float* zv;      // [BH, slots, dp]     z_t or r_tau
  bf16_t* dpsi;         // [BH, N, dp]
  uint32_t* signs;      // [BH, 2d/32, N]  which hidden units of a token are positive, 32 to a word
  float* db2_part;      // [n_items, dp]  sum over the item's tokens of dpsi
  int H, T, HW, chunk, overlap;
                        // query side: segment s = queries of chunk s+1, slot s+1; else key segment s, slot s
  int n_seg, nsplit, slots, n_items, items_per_xcd;
};

// Weight gradients of both sides.  dW2 partial sums: part_w2[f][hid] = sum over a token range of
// dpsi[tok][f] * U[tok][hid], with U = relu(W1 x + b1) recomputed from x (cheaper than moving it through
// HBM).  First layer: dU = (dpsi W2) * [U > 0] (signs from act_grad_kernel); part_w1 = x^T dU ([d][hidden]), then the column sums of
// dU ([hidden]).
struct WeightGradSide {
  const bf16_t* dpsi;   // [BH, N, 2d]
  const bf16_t* x;      // [BH, N, d]
  const uint32_t* signs;   // [BH, 2d/32, N]
  const bf16_t* w1;     // [H, 2d, d]
  const float* b1;      // [H, 2d]
  const bf16_t* w2t;    // [H, hidden, dp]  W2 transposed
  float* part_w2;       // [BH * n2, 2d, 2d]
  float* part_w1;       // [BH * n1, d*hidden + hidden]
  int64_t lo, hi;       // token range [lo, hi) of every (b, h)
};
struct WeightGradArgs {
  WeightGradSide side[2];   // queries, keys
  int H, BH;
  int64_t N;
  int n2, n1;               // pieces per side and (b, h) for dW2 and for dW1
  int n_items, items_per_xcd;
};

// out[h][..] = sum over b and the per_bh partials of (b, h) of an [R][C] block found at
// part_off inside each partial; transposed on the way out if `transpose`
struct ReduceArgs {
  const float* part;
  float* out;           // [H, R*C]
  int B, H, per_bh;
  int64_t part_stride, part_off;
  int R, C, transpose;
};
// up to eight such sums in one launch (one per gradient tensor)
struct ReduceJobs {
  ReduceArgs job[8];
  int n;
  int first[8];   // first block of each (set by launch_reduce)
};

hipError_t launch_prep(const PrepArgs& a, hipStream_t stream);
// with `prefix`: that pass in the same launch
hipError_t launch_suffix(const SuffixArgs& a, const PrefixArgs* prefix, hipStream_t stream);
// of one side (the other null) or of both
hipError_t launch_act_grad(const ActGradArgs* queries, const ActGradArgs* keys, int d, hipStream_t stream);
hipError_t launch_weight_grad(const WeightGradArgs& a, int d, int grid, hipStream_t stream);
// pieces of the tokens (`tiles` of 64) of each side and (b, h) in that launch: n2 for dW2, n1 for dW1
void weight_pieces(int BH, int64_t tiles, int d, int* n2, int* n1);
hipError_t launch_reduce(const ReduceJobs& jobs, hipStream_t stream);
hipError_t launch_fill_zero(float* p, int64_t n, hipStream_t stream);

hipError_t launch_state(const StateArgs& a, int d, int grid, hipStream_t stream);
// the sums behind the gradient of the chunk states (tok_scale, tok_weight set); with `keys`: those sums in the same launch
hipError_t launch_state_gradient(const StateArgs& queries, const StateArgs* keys, int d, hipStream_t stream);
hipError_t launch_prefix(const PrefixArgs& a, hipStream_t stream);
// `split`: attn_split_kernel, otherwise attn_kernel.  `absorb` (streaming step with split only):
// chunk-state pieces run by further workgroups of the launch.
hipError_t launch_attn(const AttnArgs& a, const StateArgs* absorb, int d, bool split, hipStream_t stream);
// whether attn_split_kernel is the better one for a launch of n_items 128-query workgroups whose
// softmax windows hold n_keys keys; `read_out`: some of them read a chunk state
bool attn_splits(int64_t n_items, int64_t n_keys, int d, bool read_out);
int attn_query_tile(int d);  // query tokens per workgroup of the attention kernel
const char* attn_kernel_name(int d);  // the instance launched for head width d, as profilers show it
hipError_t launch_state_out(const StateOutArgs& a, hipStream_t stream);
hipError_t launch_step_state(const StepStateArgs& a, hipStream_t stream);
hipError_t launch_bidir_state(const BidirArgs& a, hipStream_t stream);
// S [BH, dprime, d] and z [BH, dprime] <- 0
hipError_t launch_zero_state(float* S, float* z, int BH, int d, int dprime, hipStream_t stream);

}  // namespace rehyat
