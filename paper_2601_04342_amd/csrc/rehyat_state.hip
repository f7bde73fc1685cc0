// Chunk-state kernel for gfx950: for a range of key/value tokens of one
// (batch, head) computes the partial sums of the linear-attention state,
//   dS^T = V^T phi_k(K)   (d x D', fp32)      dz = sum_rows phi_k(K)   (D')
// i.e. the increments of Eq. 17-18, with the feature map phi_k (two-layer MLP,
// second half of the output squared) evaluated on the fly from K -- phi_k(K)
// never goes to HBM.
//
// One workgroup of NW waves walks its token range in tiles of 64 tokens.  Wave
// w owns hidden units and output features [32w, 32w+32): it produces that slice
// of U = relu(K W1^T + b1) for the tile, the waves exchange U through LDS, then
// each wave forms its feature slice psi = relu(U W2^T + b2), squares it if it
// lies in the upper half, and accumulates V^T phi into its d x 32 slice of the
// state, held in MFMA accumulators for the whole token range.  The wave's rows
// of W1 and W2 stay in registers as MFMA operands; what makes room for them is
// that no per-lane LDS offset is held across the tile loop (U rows are padded so
// that k-steps are immediate offsets; offsets into the permuted K and V tiles
// are one XOR away from a per-lane base and are derived per tile).
//
// K and V tiles arrive by direct global->LDS loads (chunk-swizzled rows) into two
// buffers each, picked by the parity of the tile: K and V are read exactly once,
// so every tile comes from HBM.  Step t (second half of tile t, first half of
// tile t+1) requests the K tile of t+2 and the V tile of t+1 when it begins; they
// have landed at its barrier.  The loads are inline asm (with buffers picked at run time
// the compiler must not see them, or it orders every LDS read behind all of them).
#include "rehyat_state_body.h"

namespace rehyat {

// Two waves per SIMD, also where a workgroup has four waves: with the whole register file to use the
// compiler keeps accumulators in AGPRs and copies each one out before vector work.
template <int D, int NW>
__global__ void __launch_bounds__(64 * NW, 2)
state_kernel(StateArgs a) {
  __shared__ __attribute__((aligned(1024))) char XV[StateLds<D>::XV];   // K tiles 0/1, then V tiles 0/1
  __shared__ __attribute__((aligned(1024))) char Us[StateLds<D>::US];   // U of the current and of the next tile
  __shared__ __attribute__((aligned(256))) float B1s[StateLds<D>::B1 / 4];
  state_body<D, NW>(a, blockIdx.x, XV, Us, B1s);
}

// The sums behind the gradient of the chunk states (phi_q of the queries, G), and of the keys in the same launch where
// both are wanted at once: the first k_blocks workgroups.
template <int D, int NW>
__global__ void __launch_bounds__(64 * NW, 2)
state_gradient_kernel(StateArgs queries, StateArgs keys, int k_blocks) {
  __shared__ __attribute__((aligned(1024))) char XV[StateLds<D>::XV];
  __shared__ __attribute__((aligned(1024))) char Us[StateLds<D>::US];
  __shared__ __attribute__((aligned(256))) float B1s[StateLds<D>::B1 / 4];
  __shared__ __attribute__((aligned(256))) float Tok[4 * 64];
  if ((int)blockIdx.x < k_blocks) state_body<D, NW>(keys, blockIdx.x, XV, Us, B1s);
  else state_body<D, NW, true>(queries, blockIdx.x - k_blocks, XV, Us, B1s, Tok);
}

hipError_t launch_state(const StateArgs& a, int d, int grid, hipStream_t stream) {
  if (d == 128) {
    hipLaunchKernelGGL((state_kernel<128, 8>), dim3(grid), dim3(512), 0, stream, a);
  } else {
    hipLaunchKernelGGL((state_kernel<64, 4>), dim3(grid), dim3(256), 0, stream, a);
  }
  return hipGetLastError();
}

hipError_t launch_state_gradient(const StateArgs& queries, const StateArgs* keys, int d, hipStream_t stream) {
  const int k_blocks = keys ? keys->items_per_xcd * 8 : 0, grid = k_blocks + queries.items_per_xcd * 8;
  const StateArgs& k = keys ? *keys : queries;
  if (d == 128) {
    hipLaunchKernelGGL((state_gradient_kernel<128, 8>), dim3(grid), dim3(512), 0, stream, queries, k, k_blocks);
  } else {
    hipLaunchKernelGGL((state_gradient_kernel<64, 4>), dim3(grid), dim3(256), 0, stream, queries, k, k_blocks);
  }
  return hipGetLastError();
}

}  // namespace rehyat
