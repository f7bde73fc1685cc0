// Kernels of the feature-map gradient for gfx950: dL/d(phi_q, phi_k parameters) for a given
// dL/dy_hat -- what one step of the attention distillation of section 3.4 (Eq. 19) needs,
// which trains nothing but the two feature maps of a block.
//
// With the per-row stabiliser the softmax terms of Eq. 5 do not depend on phi, so the
// chain rule runs through the linear terms only (Eq. 7, 9, 16):
//   u_i = G_i / den_i,  w_i = -(G_i . y_i) / den_i,  den_i = n^S_i + n^L_i
//   dL/dPhi_q,i = S_t u_i + w_i z_t
//   dL/dS_t = sum_i Phi_q,i u_i^T,  dL/dz_t = sum_i w_i Phi_q,i           (queries i of chunk t)
//   dL/dPhi_k,j = R_tau v_j + r_tau,  R_tau = sum_{t > tau} dL/dS_t        (keys j of segment tau)
// and then through phi = [psi_1, psi_2^2], psi = relu(W2 U + b2), U = relu(W1 x + b1).
//
// Kernels, in launch order (queries, then keys, where there are two):
//   prep_kernel        1 / den, w per token (HBM-bound)
//   state_gradient_kernel   (rehyat_state.hip) dL/dS_t, dL/dz_t partial sums
//   act_grad_kernel    recomputes U and psi, forms dPhi and dpsi per token; writes dpsi token-major, the
//                      signs of U, and the partial sums of db2; both sides in one launch where the workspace
//                      has room (rehyat_api.hip)
//   suffix_kernel      (rehyat_prefix.hip, before it) R_tau, r_tau from the partial sums
//   weight_grad_kernel of both sides: dW2 = dpsi^T U over tokens (U recomputed from x);
//                      dU = (dpsi W2) [U > 0], dW1 = dU^T x, db1 = sum dU
//   reduce_kernel      sums the per-workgroup partials over batch and pieces
// The contraction kernels follow the chunk-state kernel's scheme: wave w owns 32 hidden
// units or features, weights of its slice live in registers as MFMA B operands, tiles of 64
// tokens arrive by direct global->LDS loads, products are computed with tokens in the
// accumulator rows so that an accumulator is directly the B operand of the token
// contraction that follows, and their order is written out and fenced.
#include <type_traits>

#include "rehyat_device.h"
#include "rehyat_kernels.h"

namespace rehyat {

// ------------------------------------------------------------------------------------
// 1 / den_i, w_i = -(G_i . y_i) / den_i; u = G / den itself is not written (48.4 us at 480p with it, 34.6 without; the
// sums over it gain as well: 11 % less error of the gradients, G being exact in bf16).  Eight elements per thread, D/8
// consecutive lanes per token.  The last blocks of the launch transpose the second-layer weights of both
// maps (32 x 32 per block, through a padded LDS tile): 5 us as a launch of their own, nothing beside
// this one, which is bound by memory.
// ------------------------------------------------------------------------------------
__device__ __forceinline__ void transpose_block(const PrepArgs& a, int W, int block) {
  __shared__ bf16_t tile[32][33];
  const int nb = W / 32, m = block / (nb * nb), rc = block % (nb * nb);
  const bool second = m >= a.H;
  const int64_t off = (int64_t)(second ? m - a.H : m) * W * W;
  const bf16_t* const in = (second ? a.w2_k : a.w2_q) + off;
  bf16_t* const out = a.w2t + (second ? (int64_t)a.H * W * W : 0) + off;
  const int r0 = rc / nb * 32, c0 = rc % nb * 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;  // 32 x 8
#pragma unroll
  for (int j = 0; j < 4; ++j) tile[ty + 8 * j][tx] = in[(r0 + ty + 8 * j) * W + c0 + tx];
  __syncthreads();
#pragma unroll
  for (int j = 0; j < 4; ++j) out[(c0 + ty + 8 * j) * W + r0 + tx] = tile[tx][ty + 8 * j];
}

template <int D>
__global__ void __launch_bounds__(256)
prep_kernel(PrepArgs a, int token_blocks) {
  if ((int)blockIdx.x >= token_blocks) {
    transpose_block(a, 2 * D, blockIdx.x - token_blocks);
    return;
  }
  constexpr int LPT = D / 8;  // lanes per token
  const int64_t gid = (int64_t)blockIdx.x * 256 + threadIdx.x;
  int64_t tok = gid / LPT;
  const int part = (int)(gid % LPT);
  const bool live = tok < a.tokens;
  if (!live) tok = a.tokens - 1;  // keep the lane in the shuffles below
  const int64_t off = tok * D + 8 * part;
  const u32x4 gr = *reinterpret_cast<const u32x4*>(a.g + off);
  const u32x4 yr = *reinterpret_cast<const u32x4*>(a.y + off);
  const float inv = 1.0f / (a.nS[tok] + a.nL[tok]);
  float dot = 0.f;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float g0 = __builtin_bit_cast(float, gr[i] << 16), g1 = __builtin_bit_cast(float, gr[i] & 0xffff0000u);
    const float y0 = __builtin_bit_cast(float, yr[i] << 16), y1 = __builtin_bit_cast(float, yr[i] & 0xffff0000u);
    dot += g0 * y0 + g1 * y1;
  }
#pragma unroll
  for (int m = 1; m < LPT; m <<= 1) dot += __shfl_xor(dot, m);
  if (live && part == 0) {
    a.inv[tok] = inv;
    a.tokw[tok] = -dot * inv;
  }
}

hipError_t launch_prep(const PrepArgs& a, hipStream_t stream) {
  const int lpt = a.d / 8, nb = 2 * a.d / 32;
  const int64_t threads = a.tokens * lpt;
  const unsigned tokens = (unsigned)((threads + 255) / 256), grid = tokens + 2 * a.H * nb * nb;
  if (a.d == 128) hipLaunchKernelGGL(prep_kernel<128>, dim3(grid), dim3(256), 0, stream, a, (int)tokens);
  else hipLaunchKernelGGL(prep_kernel<64>, dim3(grid), dim3(256), 0, stream, a, (int)tokens);
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------
// Activation gradients.  Wave w owns hidden units and features [32w, 32w + 32); its rows of
// W1, W2 and of the segment's matrix M stay in registers as MFMA operands for the whole token
// range.  Per tile of 64 tokens:
//   psi slice = U W2[slice]^T + b2 and dPhi slice = Vec M[slice]^T, both with tokens in accumulator
//   rows and the wave's 32 features in lanes; dpsi = dPhi + w zv, times 2 psi in the squared half,
//   zero where psi = 0; dpsi goes through a wave-private LDS patch so that it leaves in 16-byte stores;
//   U^T slice of the next tile = relu(W1[slice] X^T + b1[slice]) -> LDS as U[token][hidden], and
//   the signs of its 32 hidden units as one word per token, which the first-layer gradient takes as gates.
// Order of products: psi and dPhi of tokens 0..31, of 32..63, then U(it+1); a half's vector work lies
// under the products that follow it, operands are read PD products ahead, one barrier per tile.
// x(it+2), vec(it+1) and the token weights of it+1 are requested as a step begins.  At its barrier
// they have landed: vector memory operations of a wave complete in the order issued, stores included,
// and the step's stores (four of dpsi, one of signs) are younger than its loads.
// ------------------------------------------------------------------------------------
// Bound by memory: 1.06 KB per token read and written, 3.4 - 3.8 TB/s at the 480p shape against 4.75 of a plain copy; the
// order of the products made no difference to that, the sign words cost 2 - 5 us and save the first-layer gradient a
// quarter of its products.  Both sides in one launch, the queries' dL/dz_t left to the chunk-state kernel and G
// scaled here instead of u read: 320x480 106 -> 101.5 us, 480p 240 -> 238.6.
// Two waves per SIMD, also where a workgroup has four waves: with the whole register file to use the
// compiler keeps accumulators in AGPRs and copies each one out before vector work.
template <int D, int NW>
struct ActGradLds {
  char XV[4 * 64 * 2 * D];               // x tiles 0/1, then vec tiles 0/1
  char Us[2 * 64 * (2 * D * 2 + 16)];    // U of the current and of the next tile
  char Stg[NW * 32 * 80];                // dpsi on its way out
  float Tok[4 * 64];                     // scale and weight of the tokens of two tiles
  float B1s[2 * D];
};
// TW: the query side, with a scale and a weight per token
template <int D, int NW, bool TW>
__device__ __forceinline__ void act_grad_body(const ActGradArgs& a, int block, ActGradLds<D, NW>& lds) {
  constexpr int HID = 2 * D, DP = 2 * D;
  constexpr int KS = D / 16;
  constexpr int KS2 = HID / 16;
  constexpr int TB = 64 * 2 * D;  // bytes of an x or vec tile
  constexpr int UROW = HID * 2;
  constexpr int SROW = 80;        // bytes per token row of the dpsi patch: 32 features + padding
  // U[token][hidden] with 16 bytes of padding per row: consecutive rows start four banks apart,
  // so fragment reads and writes are conflict-free without a chunk permutation and every
  // k-step is an immediate offset from one per-lane address
  constexpr int UPAD = UROW + 16;
  static_assert(DP / NW == 32, "each wave owns 32 features");

  static_assert(sizeof(lds.Us) == 2 * 64 * UPAD && sizeof(lds.Stg) == NW * 32 * SROW && sizeof(lds.XV) % 1024 == 0 &&
                (sizeof(lds.XV) + sizeof(lds.Us)) % 1024 == 0 && sizeof(lds.Stg) % 256 == 0, "LDS layout");
  char* const XV = lds.XV;
  char* const Us = lds.Us;
  char* const Stg = lds.Stg;
  float* const Tok = lds.Tok;
  float* const B1s = lds.B1s;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 5;
  const int r = lane & 31;

  const int item = xcd_swizzle(block, a.items_per_xcd);
  if (item >= a.n_items) return;
  const int sp = item % a.nsplit;
  const int rest = item / a.nsplit;
  const int seg = rest % a.n_seg;
  const int bh = rest / a.n_seg;
  const int h = bh % a.H;

  int64_t seg_lo, seg_hi;
  int slot;
  if (TW) {
    const ChunkRange cr = chunk_range(a.T, a.HW, a.chunk, a.overlap, seg + 1);
    seg_lo = cr.q_lo;
    seg_hi = cr.q_hi;
    slot = seg + 1;
  } else {  // keys that enter the linear set between chunk seg and chunk seg + 1 (Eq. 13)
    seg_lo = chunk_range(a.T, a.HW, a.chunk, a.overlap, seg).s_lo;
    seg_hi = chunk_range(a.T, a.HW, a.chunk, a.overlap, seg + 1).s_lo;
    slot = seg;
  }
  const int64_t N = (int64_t)a.T * a.HW;
  const int64_t len = seg_hi - seg_lo;
  const int64_t lo = seg_lo + (len * sp) / a.nsplit;
  const int64_t hi = seg_lo + (len * (sp + 1)) / a.nsplit;
  const int n_tokens = (int)(hi - lo), n_tiles = (n_tokens + 63) / 64;

  const int64_t row0 = (int64_t)bh * N + lo;  // first token of this piece, over all (b, h)
  char* Pg = reinterpret_cast<char*>(a.dpsi + row0 * DP);
  uint32_t* const Sgn = a.signs + ((int64_t)bh * NW + wave) * N + lo;   // this wave's word of a token

  // ---- resident operands ----------------------------------------------------
  // first-layer bias in LDS: accumulator register 4i+j is hidden unit 32w + 8i + 4g + j, so a
  // lane reads its four rows of block i with one 16-byte read
  const float b1v = tid < HID ? a.b1[(int64_t)h * HID + tid] : 0.f;
  const float* const b1rows = B1s + wave * 32 + 4 * g;
  const int unit = wave * 32 + r;  // this lane's hidden unit (U) and feature (psi, dPhi)
  float b2v = a.b2[(int64_t)h * DP + unit];
  float zvv = a.zv[((int64_t)bh * a.slots + slot) * DP + unit];
  bf16x8 w1f[KS];   // A operands: row = hidden unit, k = head dimension
  {
    const bf16_t* p = a.w1 + ((int64_t)h * HID + unit) * D + 8 * g;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) w1f[ks] = *reinterpret_cast<const bf16x8*>(p + 16 * ks);
  }
  bf16x8 w2f[KS2];  // B operands: column = feature, k = hidden
  bf16x8 mf[KS];    // B operands: column = feature, k = head dimension (row `unit` of M)
  // W2 and M come by way of the tile buffers: W2 through those of x, vec (half of the waves) and U, then M through
  // those of U while the first tiles arrive.  M is stored transposed ([d][dprime], the layout of the forward chunk
  // states): the wave's 32 columns, read back with transposing loads.  Read from memory as operands, M value by value,
  // the launch took 54.5 us (216 workgroups of ten tiles), now 53.1.
  static_assert(KS2 == 2 * KS && NW / 2 * 64 * 2 * D <= 4 * TB && NW / 2 * 64 * 2 * D <= 2 * 64 * UPAD, "staging");
  char* const stage = (wave < NW / 2 ? XV : Us) + (wave % (NW / 2)) * (64 * 2 * D);
  {
    const u32x4 W2r = make_rsrc_words(a.w2 + ((int64_t)h * DP + wave * 32) * HID);
    const uint32_t lds = __builtin_amdgcn_readfirstlane(lds_address(stage));
    stage_rows<2 * D>(W2r, 4 * D, 0, lds, lane);
    stage_rows<2 * D>(W2r, 4 * D, 2 * D, lds + 32 * 2 * D, lane);
  }

  const u32x4 Xr = make_rsrc_words(a.x + row0 * D), Vr = make_rsrc_words(a.vec + row0 * D);
  // scales by even waves, weights by odd ones
  const u32x4 Tr = make_rsrc_words(TW ? (const void*)((wave & 1 ? a.tokw : a.inv) + row0) : (const void*)a.x);
  const uint32_t x_lds = lds_address(XV), v_lds = x_lds + 2 * TB;
  const uint32_t tok_lds = __builtin_amdgcn_readfirstlane(lds_address(Tok) + 256 * (wave & 1));
  using R = RangeTiles<2 * D, NW>;
  const R range(n_tokens, wave, lane);
  auto load_tok = [&](int it) {   // of the tile's 64 tokens
    const int row = n_tokens < 64 ? 0 : 64 * it < n_tokens - 64 ? 64 * it : n_tokens - 64;
    int ln = lane;
    asm volatile("" : "+v"(ln));
    direct_load_4(Tr, 4 * (ln < n_tokens ? ln : n_tokens - 1), __builtin_amdgcn_readfirstlane(4 * row),
                  tok_lds + (it & 1) * 512);
  };
  const int uwbase = r * UPAD + wave * 64 + 8 * g;   // write: token r, units 32w + 8i + 4g .. +3 at + 16 i
  const int urbase = r * UPAD + 16 * g;              // read: A fragment of token r, k-step ks at + 32 ks
  char* const Sg = Stg + wave * (32 * SROW);   // this wave's patch: [32 tokens][32 features]

  auto u_start = [&]() {   // starts from the bias: no addition per element
    f32x16 u;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const f32x4 bb = *reinterpret_cast<const f32x4*>(b1rows + 8 * i);
#pragma unroll
      for (int j = 0; j < 4; ++j) u[4 * i + j] = bb[j];
    }
    return u;
  };
  // four hidden units of the lane's token: rectified into U, their signs (u > 0) into `s` from the right.
  // Rectified by the median of u, 0 and the largest number (which U rounds to inf): for a NaN the instruction
  // gives the least of the others, zero, and the gate closes.  With fmaxf, or inf as the bound, the compiler chooses
  // what becomes of a NaN, since -fno-honor-nans lets it assume that there is none; comparing the bits as integers
  // takes two instructions more per unit (480p step 1,249 -> 1,262 us).
  auto u_store = [&](const f32x16& u, int i, int it, int tb, uint32_t& s) {
    float rl[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      rl[j] = __builtin_amdgcn_fmed3f(u[4 * i + j], 0.f, 3.402823466e38f);
      s = __builtin_amdgcn_alignbit(s, __builtin_bit_cast(uint32_t, 0.f - rl[j]), 31);
    }
    pin(s);
    u32x2 pk;
    pk[0] = pack_bf16(rl[0], rl[1]);
    pk[1] = pack_bf16(rl[2], rl[3]);
    *reinterpret_cast<u32x2*>(Us + (it & 1) * (64 * UPAD) + uwbase + 16 * i + tb * (32 * UPAD)) = pk;
  };
  // one word per token: unit 8i + 4g + j of the slice is bit 16 g + 15 - (4i + j); lane half g stores
  // the tokens of half tile g
  auto sign_word = [&](const uint32_t (&s)[2]) {
    uint32_t w[2];
#pragma unroll
    for (int tb = 0; tb < 2; ++tb) {
      float lo = __builtin_bit_cast(float, s[tb]), hi = lo;
      half_swap(lo, hi);
      w[tb] = __builtin_bit_cast(uint32_t, lo) | (__builtin_bit_cast(uint32_t, hi) << 16);
    }
    return g ? w[1] : w[0];
  };
  auto tile_row = [&](int it) {   // first token of the tile's 64 rows in the piece
    return n_tokens < 64 ? 0 : 64 * it < n_tokens - 64 ? 64 * it : n_tokens - 64;
  };
  auto opaque_lane = [&]() {
    int ln = lane;
    asm volatile("" : "+v"(ln));
    return ln;
  };
  // fragment of token row r, k-step ks inside an x or vec tile: ^ 32 ks
  auto x_base = [&](int ln) { return tile_off<2 * D>(ln & 31, 8 * (ln >> 5)); };

  float db2acc = 0.f;
  constexpr int PD = 4;
  bf16x8 fr[PD];
  wave_loads_done();
  if (tid < HID) B1s[tid] = b1v;
#pragma unroll
  for (int ks = 0; ks < KS2; ++ks) w2f[ks] = staged_fragment<2 * D>(stage + ks / KS * (32 * 2 * D), lane, ks % KS);
  lds_barrier();   // W2 has been read by all waves, the bias is in LDS
  char* const stage_m = Us + wave * (D * 64);
  {
    const u32x4 Mr = make_rsrc_words(a.M + ((int64_t)bh * a.slots + slot) * D * DP + wave * 32);
    const uint32_t lds = __builtin_amdgcn_readfirstlane(lds_address(stage_m));
#pragma unroll
    for (int n = 0; n < D / 16; ++n)   // 16 rows of 64 bytes
      direct_load_16(Mr, (lane >> 2) * (2 * DP) + 16 * (lane & 3), n * 16 * (2 * DP), lds + n * 1024);
  }
  if (n_tiles > 0) {
    range.fill(Xr, 0, x_lds);
    if (TW) load_tok(0);
    range.fill(Vr, 0, v_lds);
    if (n_tiles > 1) range.fill(Xr, 64, x_lds + TB);
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * R::LPT) : "memory");   // M; two tiles at least are younger
  } else {
    wave_loads_done();
  }
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    const bf16_t* const p = reinterpret_cast<const bf16_t*>(stage_m) + (16 * ks + 8 * g + ((lane & 15) >> 2)) * 32 +
                            16 * (r >> 4) + 4 * (lane & 3);
    mf[ks] = join_tr(lds_read_tr(p), lds_read_tr(p + 4 * 32));
  }
  settle(w1f);
  settle(w2f);
  settle(mf);
  settle(b2v);
  settle(zvv);
  if (n_tiles > 0) {
    wait_loads_and_barrier<0>();   // also: all waves have read M
    const int xbase = x_base(opaque_lane());
    uint32_t s[2] = {0u, 0u};
#pragma unroll
    for (int tb = 0; tb < 2; ++tb) {
      f32x16 u = u_start();
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
        u = mfma(w1f[ks], *reinterpret_cast<const bf16x8*>(XV + (xbase ^ (32 * ks)) + tb * (32 * 2 * D)), u);
#pragma unroll
      for (int i = 0; i < 4; ++i) u_store(u, i, 0, tb, s[tb]);
    }
    const uint32_t word = sign_word(s);
    if (lane < n_tokens) Sgn[lane] = word;
    wait_loads_and_barrier<0>();   // U of tile 0 is complete
  }

  auto tile_step = [&](auto MOREC, auto SQC, int it) {
    constexpr bool MORE = decltype(MOREC)::value;      // a tile follows; this one is full
    constexpr bool squared = decltype(SQC)::value;     // Phi = psi^2, psi = relu(.) otherwise
    const char* const Vs = XV + (2 + (it & 1)) * TB;
    const char* const Xs = XV + ((it + 1) & 1) * TB;
    const char* const Uc = Us + (it & 1) * (64 * UPAD);
    const int ln = opaque_lane();
    const int xbase = x_base(ln);
    const int first = range.first(64 * it), count = range.count(64 * it), row = tile_row(it);
    const u32x4 Xd = rsrc_if(Xr, it + 2 < n_tiles);
    const int xs = range.soff(64 * (it + 2)), vs = range.soff(64 * (it + 1));
    const uint32_t xd = x_lds + (it & 1) * TB, vd = v_lds + ((it + 1) & 1) * TB;
    constexpr int LH = KS2 + KS, F0 = 2 * LH, LF = MORE ? KS : 0, NM = F0 + 2 * LF;
    static_assert(NM % PD == 0, "the fragment ring closes over a step");
    f32x16 ps[2], dphi[2], u[2];
    uint32_t sgn[2] = {0u, 0u};
    float pdb[2] = {0.f, 0.f};   // a half's own sums: short chains of additions in fp32
    f32x4 scale, weight;         // of four tokens
    auto read_tok = [&](int tb, int q) {
      const float* const p = Tok + (it & 1) * 128 + 32 * tb + 8 * q + 4 * g;
      scale = *reinterpret_cast<const f32x4*>(p);
      weight = *reinterpret_cast<const f32x4*>(p + 64);
    };
    auto fetch = [&](auto MC) {
      constexpr int m = decltype(MC)::value;
      if constexpr (m >= NM) {
      } else if constexpr (m < F0) {
        constexpr int tb = m / LH, n = m % LH;
        if constexpr (n < KS2) fr[m % PD] = *reinterpret_cast<const bf16x8*>(Uc + urbase + 32 * n + tb * (32 * UPAD));
        else fr[m % PD] = *reinterpret_cast<const bf16x8*>(Vs + (xbase ^ (32 * (n - KS2))) + tb * (32 * 2 * D));
      } else {
        constexpr int tb = (m - F0) / KS, n = (m - F0) % KS;
        if constexpr (n == 0) u[tb] = u_start();
        fr[m % PD] = *reinterpret_cast<const bf16x8*>(Xs + (xbase ^ (32 * n)) + tb * (32 * 2 * D));
      }
    };
    auto elements = [&](auto TBC, auto IC) {   // tokens 8 i + 4 g .. + 3 of the half, in two pairs
      constexpr int tb = decltype(TBC)::value, q = decltype(IC)::value, i = q / 2;
      float dp[2];
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int e = 2 * q + j;
        const bool live = MORE || (unsigned)(32 * tb + 8 * i + 4 * g + (e & 3) - first) < (unsigned)count;
        const float psi = fmaxf(ps[tb][e] + b2v, 0.f);
        const float base = TW ? dphi[tb][e] * scale[e & 3] + weight[e & 3] * zvv : dphi[tb][e] + zvv;   // dL/dPhi
        dp[j] = squared ? (psi + psi) * base : (psi > 0.f ? base : 0.f);
        pdb[tb] += live ? dp[j] : 0.f;
      }
      pin(pdb[tb]);
      const uint32_t pk = pack_bf16(dp[0], dp[1]);
      char* const w = Sg + (8 * i + 4 * g + 2 * (q & 1)) * SROW + 2 * r;
      *reinterpret_cast<bf16_t*>(w) = (bf16_t)pk;
      *reinterpret_cast<bf16_t*>(w + SROW) = (bf16_t)(pk >> 16);
    };
    // the patch leaves token-major: 4 chunks of 16 bytes per token row, two per lane
    auto leave = [&](int tb) {
#pragma unroll
      for (int n = 0; n < 2; ++n) {
        const int idx = ln + 64 * n, rw = idx >> 2, c = idx & 3;
        const u32x4 val = *reinterpret_cast<const u32x4*>(Sg + rw * SROW + 16 * c);
        if (MORE || (unsigned)(32 * tb + rw - first) < (unsigned)count)
          *reinterpret_cast<u32x4*>(Pg + ((int64_t)row + 32 * tb + rw) * (DP * 2) + wave * 64 + 16 * c) = val;
      }
    };
    constexpr int kQ = 2;   // element pairs per slot
    static_assert(!MORE || F0 + 2 + 8 / kQ < NM, "the second half leaves before the barrier");
    static_for<NM>([&](auto MC) {
      constexpr int m = decltype(MC)::value;
      if constexpr (m < F0) {
        constexpr int tb = m / LH, n = m % LH;
        if constexpr (n < KS2) ps[tb] = mfma(fr[m % PD], w2f[n], n == 0 ? f32x16{} : ps[tb]);
        else dphi[tb] = mfma(fr[m % PD], mf[n - KS2], n == KS2 ? f32x16{} : dphi[tb]);
      } else {
        constexpr int tb = (m - F0) / KS, n = (m - F0) % KS;
        u[tb] = mfma(w1f[n], fr[m % PD], u[tb]);
      }
      fetch(std::integral_constant<int, m + PD>{});
      if constexpr (MORE && m % 2 == 1 && m / 2 < 2 * R::LPT) {
        constexpr int i = m / 2;
        if constexpr (i < R::LPT) range.template load<i>(Xd, xs, xd);
        else range.template load<i - R::LPT>(Vr, vs, vd);
      }
      if constexpr (MORE && TW && m == 4 * R::LPT + 1) load_tok(it + 1);
      static_for<2>([&](auto TBC) {
        constexpr int tb = decltype(TBC)::value, p = m - (tb + 1) * LH - 2;
        if constexpr (p >= 0 && p * kQ < 8) {
          static_for<kQ>([&](auto JC) { elements(TBC, std::integral_constant<int, p * kQ + decltype(JC)::value>{}); });
        }
        if constexpr (TW && p >= -1 && (p + 1) * kQ < 8) read_tok(tb, (p + 1) * kQ / 2);   // a slot ahead
        if constexpr (p == 8 / kQ) leave(tb);
      });
      if constexpr (MORE) {
        constexpr int q = m - F0 - KS - 2;   // U of tokens 0..31 under the products of 32..63
        if constexpr (D == 128 && q >= 0 && q < 4) u_store(u[0], q, it + 1, 0, sgn[0]);
        if constexpr (D == 64 && m == NM - 1) static_for<4>([&](auto IC) { u_store(u[0], decltype(IC)::value, it + 1, 0, sgn[0]); });
      }
      __builtin_amdgcn_sched_barrier(0);
    });
    if constexpr (MORE) {
#pragma unroll
      for (int i = 0; i < 4; ++i) u_store(u[1], i, it + 1, 1, sgn[1]);
      Sgn[tile_row(it + 1) + opaque_lane()] = sign_word(sgn);
      wait_loads_and_barrier<5>();
      static_for<PD>([&](auto MC) {
        fr[decltype(MC)::value] = *reinterpret_cast<const bf16x8*>(Us + ((it + 1) & 1) * (64 * UPAD) + urbase +
                                                                  32 * decltype(MC)::value);
      });
    } else {
      static_for<8>([&](auto IC) {
        if constexpr (TW && decltype(IC)::value % 2 == 0) read_tok(1, decltype(IC)::value / 2);
        elements(std::integral_constant<int, 1>{}, IC);
      });
      leave(1);
    }
    db2acc += pdb[0];
    db2acc += pdb[1];
  };
  auto all_tiles = [&](auto SQC) {   // the waves of both instances meet at the same barriers
    // (fragments read before the branch would be kept, spilled, for the instance behind the other)
    if (n_tiles > 0) {
      static_for<PD>([&](auto MC) {
        fr[decltype(MC)::value] = *reinterpret_cast<const bf16x8*>(Us + urbase + 32 * decltype(MC)::value);
      });
    }
    for (int it = 0; it + 1 < n_tiles; ++it) tile_step(std::true_type{}, SQC, it);
    if (n_tiles > 0) tile_step(std::false_type{}, SQC, n_tiles - 1);
  };
  if (wave * 32 >= DP / 2) all_tiles(std::true_type{});
  else all_tiles(std::false_type{});

  const float db2 = half_swap_sum(db2acc);
  if (g == 0) a.db2_part[(int64_t)item * DP + unit] = db2;
}

// One side or both in one launch, the queries in the first q_blocks workgroups.
template <int D, int NW>
__global__ void __launch_bounds__(64 * NW, 2)
act_grad_kernel(ActGradArgs queries, ActGradArgs keys, int q_blocks) {
  __shared__ __attribute__((aligned(1024))) ActGradLds<D, NW> lds;
  if ((int)blockIdx.x < q_blocks) act_grad_body<D, NW, true>(queries, blockIdx.x, lds);
  else act_grad_body<D, NW, false>(keys, blockIdx.x - q_blocks, lds);
}

hipError_t launch_act_grad(const ActGradArgs* queries, const ActGradArgs* keys, int d, hipStream_t stream) {
  const int q_blocks = queries ? queries->items_per_xcd * 8 : 0, grid = q_blocks + (keys ? keys->items_per_xcd * 8 : 0);
  const ActGradArgs &q = queries ? *queries : *keys, &k = keys ? *keys : *queries;
  if (d == 128)
    hipLaunchKernelGGL((act_grad_kernel<128, 8>), dim3(grid), dim3(512), 0, stream, q, k, q_blocks);
  else
    hipLaunchKernelGGL((act_grad_kernel<64, 4>), dim3(grid), dim3(256), 0, stream, q, k, q_blocks);
  return hipGetLastError();
}

// token range of piece sp of nsplit: whole tiles of 64 from `lo`, the last one ragged
struct Piece {
  int64_t tok0;
  int tokens;
};
__device__ __forceinline__ Piece piece_of(int64_t lo, int64_t hi, int sp, int nsplit) {
  const int64_t nt = (hi - lo + 63) / 64;
  const int64_t t0 = nt * sp / nsplit, t1 = nt * (sp + 1) / nsplit;
  const int64_t end = lo + 64 * t1 < hi ? lo + 64 * t1 : hi;
  return Piece{lo + 64 * t0, (int)(end - (lo + 64 * t0))};
}

// first-layer bias of the wave's accumulator rows: register 4i+j is hidden unit
// 32 wave + 8i + 4g + j, two wave-uniform values per register picked by the lane half
struct BiasRows {
  float lo[16], hi[16];
};
__device__ __forceinline__ BiasRows load_bias_rows(const float* bp) {
  BiasRows b;
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      b.lo[4 * i + j] = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, bp[8 * i + j])));
      b.hi[4 * i + j] = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, bp[8 * i + 4 + j])));
    }
  return b;
}

// Per-lane offsets into the tiles, recomputed per tile from an opaque copy of the lane index: held
// across a loop they would push resident operands out of registers.
template <int D>
struct GradOffsets {
  int p, x, v;   // dpsi row, x row (k-step ks at ^ 32 ks), transposing reads of x (column block db at ^ 64 db)
  __device__ __forceinline__ explicit GradOffsets(int lane) {
    asm volatile("" : "+v"(lane));
    const int r = lane & 31, g = lane >> 5;
    p = tile_off<4 * D>(r, 8 * g);
    x = tile_off<2 * D>(r, 8 * g);
    v = tile_off<2 * D>(4 * g + ((lane & 15) >> 2), 16 * (r >> 4) + 4 * (lane & 3));
  }
};
// transposing read of 16 tokens x 32 columns; the second half lies eight rows further down
template <int ROWBYTES>
__device__ __forceinline__ bf16x8 tr_fragment(const char* p, int off) {
  return join_tr(lds_read_tr(reinterpret_cast<const bf16_t*>(p + off)),
                 lds_read_tr(reinterpret_cast<const bf16_t*>(p + (off ^ 32) + 8 * ROWBYTES)));
}

// ------------------------------------------------------------------------------------
// dW2 partial: part[f][hid] = sum_tok dpsi[tok][f] U[tok][hid].  The waves rebuild U = relu(W1 x + b1)
// of tile it+1 in LDS (token-major, as the chunk-state kernel does; 16 MFMAs per wave against 512
// bytes per token that U would cost through HBM) while they multiply tile `it`; both operands
// are token-major LDS tiles read with transposing loads (tokens become the contraction index).
// Each wave owns 64 rows f and half of the columns.
// Order of products: 16 tokens of dW2, U of 32 tokens, 16 tokens, U, 16, 16 -- U is rectified and stored
// under the products that follow it.  Operands are read kLook reads ahead into a ring of kRing; one
// barrier per tile, behind the last read of it.  X(it+2) and dpsi(it+1) are requested as a
// step begins and have landed at its barrier.
// ------------------------------------------------------------------------------------
template <int D, int NW>
__device__ __forceinline__ void tn_body(const WeightGradSide& a, int H, int64_t N, int bh, int sp, int nsplit, char* Ts) {
  constexpr int W = 2 * D;          // features = hidden units
  constexpr int KS = D / 16;
  constexpr int ROWB = 2 * W;       // bytes per token row of dpsi and of U
  constexpr int TBY = 64 * ROWB;    // dpsi tile
  constexpr int TB = 64 * 2 * D;    // x tile
  constexpr int HB = W / 64;        // 32-column blocks per wave (half of the columns)
  static_assert(W / 64 == NW / 2, "waves form a (W/64) x 2 grid");
  static_assert(W / NW == 32, "each wave rebuilds 32 hidden units");
  char* const Pt = Ts;              // dpsi tiles 0/1
  char* const Xt = Ts + 2 * TBY;    // x tiles 0/1
  char* const Us = Xt + 2 * TB;     // U of the current and of the next tile

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 5, r = lane & 31;
  const int wf = wave >> 1, wh = wave & 1;
  const int h = bh % H;
  const Piece pc = piece_of(a.lo, a.hi, sp, nsplit);
  const int n_tiles = (pc.tokens + 63) / 64;
  const int64_t row0 = (int64_t)bh * N + pc.tok0;
  const u32x4 Pr = make_rsrc_words(a.dpsi + row0 * W), Xr = make_rsrc_words(a.x + row0 * D);
  const uint32_t p_lds = lds_address(Pt), x_lds = lds_address(Xt);
  using RP = RangeTiles<ROWB, NW>;
  using RX = RangeTiles<2 * D, NW>;
  const RP prange(pc.tokens, wave, lane);
  const RX xrange(pc.tokens, wave, lane);

  const BiasRows b1 = load_bias_rows(a.b1 + (int64_t)h * W + wave * 32);
  bf16x8 w1f[KS];   // A operands: row = hidden unit 32 wave + r, k = head dimension; by way of the buffers of U
  char* const stage = Us + wave * (32 * 2 * D);
  stage_rows<2 * D>(make_rsrc_words(a.w1 + ((int64_t)h * W + wave * 32) * D), 2 * D, 0,
                    __builtin_amdgcn_readfirstlane(lds_address(stage)), lane);
  f32x16 acc[2][HB];
#pragma unroll
  for (int fb = 0; fb < 2; ++fb)
#pragma unroll
    for (int hb = 0; hb < HB; ++hb) acc[fb][hb] = f32x16{};

  if (n_tiles > 0) {
    xrange.fill(Xr, 0, x_lds);
    prange.fill(Pr, 0, p_lds);
    if (n_tiles > 1) xrange.fill(Xr, 64, x_lds + TB);
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(RX::LPT + RP::LPT) : "memory");   // W1; these tiles at least are younger
  } else {
    wave_loads_done();
  }
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) w1f[ks] = staged_fragment<2 * D>(stage, lane, ks);
  settle(w1f);
  auto u_start = [&]() {
    f32x16 u;
#pragma unroll
    for (int e = 0; e < 16; ++e) u[e] = g ? b1.hi[e] : b1.lo[e];
    return u;
  };
  auto u_store = [&](const f32x16& u, int i, int it, int tb) {
    int ln = lane;
    asm volatile("" : "+v"(ln));
    const int tok = ln & 31;
    u32x2 pk;
    pk[0] = pack_bf16(fmaxf(u[4 * i], 0.f), fmaxf(u[4 * i + 1], 0.f));
    pk[1] = pack_bf16(fmaxf(u[4 * i + 2], 0.f), fmaxf(u[4 * i + 3], 0.f));
    *reinterpret_cast<u32x2*>(Us + (it & 1) * TBY + tb * (32 * ROWB) + tok * ROWB + (((wave * 4 + i) ^ swz<ROWB>(tok)) << 4) +
                              8 * (ln >> 5)) = pk;
  };
  auto x_fragment = [&](int it, const GradOffsets<D>& o, int tb, int ks) {
    return *reinterpret_cast<const bf16x8*>(Xt + (it & 1) * TB + (o.x ^ (32 * ks)) + tb * (32 * 2 * D));
  };
  constexpr int kRing = 8, kLook = D == 128 ? 3 : 4;
  bf16x8 fr[kRing];
  // column of the wave's first 32 of dpsi (rows of dW2) and of U
  auto f_base = [&](int col) {
    int ln = lane;
    asm volatile("" : "+v"(ln));
    return tile_off<ROWB>(4 * (ln >> 5) + ((ln & 15) >> 2), col + 16 * ((ln & 31) >> 4) + 4 * (ln & 3));
  };
  // read q of the dW2 part of a tile: per 16 tokens two blocks of 32 rows, then HB blocks of 32 columns
  auto s_read = [&](int it, int pb, int ub, int s, int q) {
    if (q < 2) return tr_fragment<ROWB>(Pt + (it & 1) * TBY + s * 16 * ROWB, pb ^ (64 * q));
    return tr_fragment<ROWB>(Us + (it & 1) * TBY + s * 16 * ROWB, ub ^ (64 * (q - 2)));
  };
  if (n_tiles > 0) {
    wait_loads_and_barrier<0>();
    const GradOffsets<D> o(lane);
#pragma unroll
    for (int tb = 0; tb < 2; ++tb) {
      f32x16 u = u_start();
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) u = mfma(w1f[ks], x_fragment(0, o, tb, ks), u);
#pragma unroll
      for (int i = 0; i < 4; ++i) u_store(u, i, 0, tb);
    }
    lds_barrier();   // U of tile 0 is complete
    const int pb = f_base(64 * wf), ub = f_base((W / 2) * wh);
    static_for<kLook>([&](auto QC) { fr[decltype(QC)::value] = s_read(0, pb, ub, 0, decltype(QC)::value); });
  }
  auto tile_step = [&](auto MOREC, int it) {
    constexpr bool MORE = decltype(MOREC)::value;
    const GradOffsets<D> o(lane);
    const int pb = f_base(64 * wf), ub = f_base((W / 2) * wh);
    const u32x4 Xd = rsrc_if(Xr, it + 2 < n_tiles);
    const int xs = xrange.soff(64 * (it + 2)), ps = prange.soff(64 * (it + 1));
    const uint32_t xd = x_lds + (it & 1) * TB, pd = p_lds + ((it + 1) & 1) * TBY;
    // groups of products: S0 U0 S1 U1 S2 S3; a group S has LS products on RS reads, a group U KS on KS
    constexpr int LS = 2 * HB, RS = 2 + HB, LU = MORE ? KS : 0;
    constexpr int NM = 4 * LS + 2 * LU, NR = 4 * RS + 2 * LU;
    static_assert(!MORE || NR % kRing == 0, "the ring closes over a step");
    // group of product m (0..5), its first product and its first read
    auto group = [](int m) {
      return m < LS ? 0 : m < LS + LU ? 1 : m < 2 * LS + LU ? 2 : m < 2 * LS + 2 * LU ? 3 : m < 3 * LS + 2 * LU ? 4 : 5;
    };
    auto s_of = [](int gr) { return gr == 5 ? 3 : gr / 2; };
    auto is_u = [](int gr) { return gr == 1 || gr == 3; };
    f32x16 u[2];
    auto base_m = [](int gr) {   // products before group gr
      const int sg = gr == 0 ? 0 : gr == 1 ? 1 : gr == 2 ? 1 : gr == 3 ? 2 : gr == 4 ? 2 : 3;
      const int ug = gr <= 1 ? 0 : gr <= 3 ? 1 : 2;
      return sg * LS + ug * LU;
    };
    auto base_r = [](int gr) {   // reads before group gr
      const int sg = gr == 0 ? 0 : gr == 1 ? 1 : gr == 2 ? 1 : gr == 3 ? 2 : gr == 4 ? 2 : 3;
      const int ug = gr <= 1 ? 0 : gr <= 3 ? 1 : 2;
      return sg * RS + ug * LU;
    };
    auto need = [=](int m) {     // last read that product m takes
      const int gr = group(m), n = m - base_m(gr);
      return base_r(gr) + (is_u(gr) ? n : 2 + n / 2);
    };
    auto read = [&](auto QC) {
      constexpr int q = decltype(QC)::value;
      if constexpr (q >= NR) {
        if constexpr (MORE) fr[q % kRing] = s_read(it + 1, pb, ub, 0, q - NR);
      } else {
        constexpr int gr = q < base_r(1) ? 0 : q < base_r(2) ? 1 : q < base_r(3) ? 2 : q < base_r(4) ? 3 : q < base_r(5) ? 4 : 5;
        constexpr int n = q - base_r(gr);
        if constexpr (is_u(gr)) {
          fr[q % kRing] = x_fragment(it + 1, o, gr / 2, n);
        } else {
          fr[q % kRing] = s_read(it, pb, ub, s_of(gr), n);
        }
      }
    };
    // the barrier stands behind the last read of the tile and before the first of the next one
    constexpr int BAR = base_m(5) + (need(base_m(5) - 1) + 1 + kLook < NR ? 1 : 0);
    static_assert(need(BAR - 1) + 1 + kLook == NR, "all of the tile has been read at the barrier");
    static_assert(base_m(4) + 6 <= BAR + (D == 64 ? 2 : 0), "U is stored before the barrier that publishes it");
    static_for<NM>([&](auto MC) {
      constexpr int m = decltype(MC)::value, gr = group(m), n = m - base_m(gr), rb = base_r(gr);
      if constexpr (MORE && m == BAR) wait_loads_and_barrier<0>();
      if constexpr (is_u(gr) && n == 0) u[gr / 2] = u_start();
      if constexpr (is_u(gr)) u[gr / 2] = mfma(w1f[n], fr[(rb + n) % kRing], u[gr / 2]);
      else acc[n & 1][n / 2] = mfma(fr[(rb + (n & 1)) % kRing], fr[(rb + 2 + n / 2) % kRing], acc[n & 1][n / 2]);
      constexpr int from = m == 0 ? kLook : need(m - 1) + 1 + kLook, to = need(m) + 1 + kLook;
      static_for<(to > from ? to - from : 0)>([&](auto JC) { read(std::integral_constant<int, from + decltype(JC)::value>{}); });
      if constexpr (MORE && m % 2 == 1 && m / 2 < RX::LPT + RP::LPT) {
        constexpr int i = m / 2;
        if constexpr (i < RX::LPT) xrange.template load<i>(Xd, xs, xd);
        else prange.template load<i - RX::LPT>(Pr, ps, pd);
      }
      static_for<2>([&](auto TBC) {   // U goes to LDS under the group behind it
        constexpr int tb = decltype(TBC)::value, q = m - base_m(tb ? 4 : 2) - 2;
        if constexpr (MORE && D == 128 && q >= 0 && q < 4) u_store(u[tb], q, it + 1, tb);
        if constexpr (MORE && D == 64 && q >= 0 && q < 2) {
          u_store(u[tb], 2 * q, it + 1, tb);
          u_store(u[tb], 2 * q + 1, it + 1, tb);
        }
      });
      __builtin_amdgcn_sched_barrier(0);
    });
  };
  for (int it = 0; it + 1 < n_tiles; ++it) tile_step(std::true_type{}, it);
  if (n_tiles > 0) {
    const int it = n_tiles - 1, first = prange.first(64 * it), count = prange.count(64 * it);
    // Rows of dpsi and U that do not belong are cleared, both, so that an infinity in either meets no zero; the
    // fragments that were read ahead are read again.  (U masked as it is stored cost every tile of the loop four
    // instructions per store: 320x480 96 us a launch, this way 91.)
    if (count < 64) {
      clear_other_rows<ROWB, 64 * NW>(Pt + (it & 1) * TBY, first, count, tid);
      clear_other_rows<ROWB, 64 * NW>(Us + (it & 1) * TBY, first, count, tid);
      lds_barrier();
      const GradOffsets<D> o(lane);
      const int pb = f_base(64 * wf), ub = f_base((W / 2) * wh);
      static_for<kLook>([&](auto QC) { fr[decltype(QC)::value] = s_read(it, pb, ub, 0, decltype(QC)::value); });
    }
    tile_step(std::false_type{}, it);
  }

  float* P = a.part_w2 + ((int64_t)bh * nsplit + sp) * W * W;
#pragma unroll
  for (int fb = 0; fb < 2; ++fb)
#pragma unroll
    for (int hb = 0; hb < HB; ++hb)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int f = 64 * wf + 32 * fb + 8 * (e >> 2) + 4 * g + (e & 3);
        P[f * W + (W / 2) * wh + 32 * hb + r] = acc[fb][hb][e];
      }
}

// ------------------------------------------------------------------------------------
// First-layer gradients.  Wave w owns hidden units [32w, 32w + 32): its rows of W2^T stay in
// registers as B operands.  Per tile, with tokens in accumulator rows and the wave's hidden units in
// lanes: dU slice = dpsi W2[:, slice], zero where U <= 0 (the sign words of act_grad_kernel; with U formed
// again for its sign alone, 16 of 64 products per tile and 32 registers, nothing was left to read
// ahead into); then x^T dU into the wave's [d][32] slice of dW1^T, exactly as the chunk-state kernel
// accumulates V^T phi.
// Order of products: dU of tokens 0..31, of 32..63, x^T dU of both; the gates of a half lie under
// the products that follow it.
// ------------------------------------------------------------------------------------
template <int D, int NW>
__device__ __forceinline__ void hid_body(const WeightGradSide& a, int H, int64_t N, int bh, int sp, int nsplit, char* Ts,
                                         uint32_t* Sw) {
  constexpr int HID = 2 * D, DP = 2 * D;
  constexpr int KS2 = DP / 16;      // k-steps across the features
  constexpr int DB = D / 32;
  constexpr int TB = 64 * 2 * D;    // x tile
  constexpr int UROW = DP * 2;      // bytes of a dpsi row
  constexpr int TBU = 64 * UROW;
  static_assert(HID / NW == 32, "each wave owns 32 hidden units");
  char* const Pt = Ts;              // dpsi tiles 0/1
  char* const Xt = Ts + 2 * TBU;    // x tiles 0/1

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 5, r = lane & 31;
  const int h = bh % H;
  const Piece pc = piece_of(a.lo, a.hi, sp, nsplit);
  const int n_tiles = (pc.tokens + 63) / 64;
  const int64_t row0 = (int64_t)bh * N + pc.tok0;
  const u32x4 Pr = make_rsrc_words(a.dpsi + row0 * DP), Xr = make_rsrc_words(a.x + row0 * D);
  const u32x4 Sr = make_rsrc_words(a.signs + ((int64_t)bh * NW + wave) * N + pc.tok0);
  const uint32_t p_lds = lds_address(Pt), x_lds = lds_address(Xt);
  uint32_t* const sw = Sw + wave * 128;   // this wave's words of two tiles
  const uint32_t s_lds = lds_address(Sw) + wave * 512;
  using RP = RangeTiles<UROW, NW>;
  using RX = RangeTiles<2 * D, NW>;
  const RP prange(pc.tokens, wave, lane);
  const RX xrange(pc.tokens, wave, lane);
  auto load_signs = [&](int it) {
    const int row = pc.tokens < 64 ? 0 : 64 * it < pc.tokens - 64 ? 64 * it : pc.tokens - 64;
    direct_load_4(Sr, 4 * (lane < pc.tokens ? lane : pc.tokens - 1), __builtin_amdgcn_readfirstlane(4 * row),
                  s_lds + (it & 1) * 256);
  };

  const int unit = wave * 32 + r;   // this lane's hidden unit
  // where its sign stands in a word: unit 8i + 4g + j of the slice is bit 16 g + 15 - (4i + j)
  const int bit = 16 * ((r >> 2) & 1) + 15 - (4 * (r >> 3) + (r & 3));
  // B operands: column = hidden unit, k = feature; in two halves by way of the second dpsi buffer (half of the waves)
  // and of LDS that only dW2 uses otherwise
  bf16x8 w2tf[KS2];
  static_assert(KS2 == 2 * D / 16 && NW / 2 * 32 * 2 * D <= TBU, "staging");
  char* const stage = (wave < NW / 2 ? Pt + TBU : Xt + 2 * TB + 512 * NW) + (wave % (NW / 2)) * (32 * 2 * D);
  const uint32_t stage_lds = __builtin_amdgcn_readfirstlane(lds_address(stage));
  const u32x4 Wr = make_rsrc_words(a.w2t + ((int64_t)h * HID + wave * 32) * DP);
  stage_rows<2 * D>(Wr, 4 * D, 0, stage_lds, lane);
  f32x16 acc[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db) acc[db] = f32x16{};
  float dbacc = 0.f;

  if (n_tiles > 0) {
    prange.fill(Pr, 0, p_lds);
    xrange.fill(Xr, 0, x_lds);
    load_signs(0);
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(RX::LPT + RP::LPT) : "memory");   // the first half of W2^T
  } else {
    wave_loads_done();
  }
#pragma unroll
  for (int ks = 0; ks < KS2 / 2; ++ks) w2tf[ks] = staged_fragment<2 * D>(stage, lane, ks);
  wave_reads_done();
  stage_rows<2 * D>(Wr, 4 * D, 2 * D, stage_lds, lane);
  wave_loads_done();
#pragma unroll
  for (int ks = 0; ks < KS2 / 2; ++ks) w2tf[KS2 / 2 + ks] = staged_fragment<2 * D>(stage, lane, ks);
  settle(w2tf);
  constexpr int PD = 4;   // fragments read ahead of their products
  bf16x8 fr[PD];
  auto p_fragment = [&](int it, const GradOffsets<D>& o, int tb, int ks) {
    return *reinterpret_cast<const bf16x8*>(Pt + (it & 1) * TBU + (o.p ^ (32 * ks)) + tb * (32 * UROW));
  };
  if (n_tiles > 0) {
    wait_loads_and_barrier<0>();
    const GradOffsets<D> o(lane);
    static_for<PD>([&](auto MC) { fr[decltype(MC)::value] = p_fragment(0, o, 0, decltype(MC)::value); });
  }
  auto tile_step = [&](auto MOREC, int it) {
    constexpr bool MORE = decltype(MOREC)::value;
    const GradOffsets<D> o(lane);
    const int first = xrange.first(64 * it), count = xrange.count(64 * it);
    const int xs = xrange.soff(64 * (it + 1)), ps = prange.soff(64 * (it + 1));
    const uint32_t xd = x_lds + ((it + 1) & 1) * TB, pd = p_lds + ((it + 1) & 1) * TBU;
    constexpr int LH = KS2, LA = 2 * DB, A0 = 2 * LH, NM = A0 + 2 * LA;
    static_assert(NM % PD == 0, "the fragment ring closes over a step");
    f32x16 du[2];
    uint32_t fb[2][8];
    u32x4 words;
    float part[2] = {0.f, 0.f};
    auto fetch = [&](auto MC) {
      constexpr int m = decltype(MC)::value;
      if constexpr (m >= NM) {
        if constexpr (MORE) fr[m % PD] = p_fragment(it + 1, o, 0, m - NM);
      } else if constexpr (m < A0) {
        fr[m % PD] = p_fragment(it, o, m / LH, m % LH);
      } else {
        constexpr int n = m - A0;   // 16-token step n / DB, column block n % DB
        fr[m % PD] = tr_fragment<2 * D>(Xt + (it & 1) * TB + n / DB * (16 * 2 * D), o.v ^ (64 * (n % DB)));
      }
    };
    auto gate = [&](auto TBC, auto IC) {   // elements 2i, 2i+1: tokens 8 (i/2) + 4g + 2 (i%2) ..
      constexpr int tb = decltype(TBC)::value, i = decltype(IC)::value;
      if constexpr (i % 2 == 0)
        words = *reinterpret_cast<const u32x4*>(sw + (it & 1) * 64 + 32 * tb + 8 * (i / 2) + 4 * g);
      float x[2];
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int e = 2 * i + j;
        const int open = __builtin_amdgcn_sbfe((int)words[e & 3], bit, 1);   // 0 or all ones
        const float d = du[tb][e];   // by value: a bit cast of du[tb][e] itself reads element 0
        x[j] = __builtin_bit_cast(float, __builtin_bit_cast(int, d) & open);
        if (!MORE && (unsigned)(32 * tb + 8 * (e >> 2) + 4 * g + (e & 3) - first) >= (unsigned)count) x[j] = 0.f;
      }
      fb[tb][i] = pack_bf16(x[0], x[1]);
      part[tb] = sum_pair<false>(fb[tb][i], part[tb]);   // db1 sums what dW1 sums
      pin(part[tb]);
      pin(fb[tb][i]);
    };
    constexpr int kPairs = 8 / LA;   // element pairs per slot
    static_for<NM>([&](auto MC) {
      constexpr int m = decltype(MC)::value;
      if constexpr (MORE && m == NM - PD) wait_loads_and_barrier<0>();
      if constexpr (m < A0) {
        constexpr int tb = m / LH, n = m % LH;
        du[tb] = mfma(fr[m % PD], w2tf[n], n == 0 ? f32x16{} : du[tb]);
      } else {
        constexpr int tb = (m - A0) / LA, n = (m - A0) % LA, s = n / DB;
        const u32x4 w = {fb[tb][4 * s], fb[tb][4 * s + 1], fb[tb][4 * s + 2], fb[tb][4 * s + 3]};
        acc[n % DB] = mfma(fr[m % PD], __builtin_bit_cast(bf16x8, w), acc[n % DB]);
      }
      fetch(std::integral_constant<int, m + PD>{});
      if constexpr (MORE && m % 2 == 1 && m / 2 < RX::LPT + RP::LPT) {
        constexpr int i = m / 2;
        if constexpr (i < RX::LPT) xrange.template load<i>(Xr, xs, xd);
        else prange.template load<i - RX::LPT>(Pr, ps, pd);
      }
      if constexpr (MORE && m == 2 * (RX::LPT + RP::LPT) + 1) load_signs(it + 1);
      static_for<2>([&](auto TBC) {
        constexpr int tb = decltype(TBC)::value, p = m - (tb ? A0 : LH) - 2;
        if constexpr (p >= 0 && kPairs * p < 8)
          static_for<kPairs>([&](auto JC) { gate(TBC, std::integral_constant<int, kPairs * p + decltype(JC)::value>{}); });
      });
      __builtin_amdgcn_sched_barrier(0);
    });
    dbacc += part[0];
    dbacc += part[1];
  };
  for (int it = 0; it + 1 < n_tiles; ++it) tile_step(std::true_type{}, it);
  if (n_tiles > 0) tile_step(std::false_type{}, n_tiles - 1);

  float* P = a.part_w1 + ((int64_t)bh * nsplit + sp) * (D * HID + HID);
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int row = 32 * db + 8 * (e >> 2) + 4 * g + (e & 3);
      P[row * HID + unit] = acc[db][e];
    }
  const float tot = half_swap_sum(dbacc);
  if (g == 0) P[D * HID + unit] = tot;
}

// Both kinds of weight gradient of both sides in one launch: per side and (b, h), n2 pieces of
// the tokens for dW2 and n1 for dW1.  Four launches (dW2 and dW1 of the queries, then of the keys), each
// with its weights to load, its last tile to wait for and 21 partial sums per (b, h), took 436 us at
// the 480p shape and 157 at 320x480; this one 340 and 103 on that box, half as many partial sums, and the two
// kinds share what they read in the last-level cache (on another 282 and 103, and 254 and 95 since U is not masked
// in every tile).  Bound by memory and by the products about alike: 1.15 GB of operands through the caches at 480p
// and 0.29 TFLOP, 4.5 TB/s and 1.14 PFLOP/s there.
template <int D, int NW>
__global__ void __launch_bounds__(64 * NW, 2)
weight_grad_kernel(WeightGradArgs a) {
  // dW2: two dpsi, x and U tiles (all of the CU's LDS at d = 128); dW1: two dpsi and x tiles, sign words
  __shared__ __attribute__((aligned(1024))) char Ts[2 * 64 * (4 * D + 2 * D + 4 * D)];
  const int item = xcd_swizzle(blockIdx.x, a.items_per_xcd);
  if (item >= a.n_items) return;
  const int per = a.n2 + a.n1, which = item / per, j = item % per;
  const int bh = which % a.BH;
  const WeightGradSide& s = a.side[which / a.BH];
  if (j < a.n2) tn_body<D, NW>(s, a.H, a.N, bh, j, a.n2, Ts);
  else hid_body<D, NW>(s, a.H, a.N, bh, j - a.n2, a.n1, Ts, reinterpret_cast<uint32_t*>(Ts + 2 * 64 * 6 * D));
}

// The launch is cut to fill the chip once, twice or three times, whichever ends first, in even shares of both
// kinds.  A tile takes 3.0 us for dW2 with every CU busy at d = 128 and 1.6 at d = 64, for dW1 a tenth less, and a
// piece 20 and 10 us for its weights and its partial sums; in a single round what is left when some pieces have ended
// runs faster, so it counts between its longest and its mean piece.  One round alone, rounded down to whole
// pieces, leaves up to half of the chip idle behind the longest ones, or has a second round that is nearly empty.
// Saved gradients, whole calls, one round and this rule:
//   d = 128, 12,600 tokens: 33 heads 2 + 1 pieces 874 us, 4 + 3 831; 36 928 and 858; 65 1 + 1 1,976, 3 + 2 1,675; 96
//   2,523 and 2,385; 24 stay at 3 + 2 (677; 5 + 5 689).  32,760 tokens: 24 heads 3 + 2 1,615, 8 + 8 1,579
//   d = 64, 12,600 tokens: 72 heads 2 + 1 683, 4 + 3 628; 96 1 + 1 884, 4 + 4 824
// Of all cuts tried at 44 such counts of heads and tokens the rule's was nowhere slower than one round's, and the best
// or within 1 % of it but for four (1 - 6 % at 48, 72 and 130 heads of 64 and 36 of 128).
void weight_pieces(int BH, int64_t tiles, int d, int* n2, int* n1) {
  const int64_t slots = d == 128 ? 256 : 512;   // workgroups resident at once
  const double tile2 = d == 128 ? 3.0 : 1.6, tile1 = 0.9 * tile2, piece = d == 128 ? 20.0 : 10.0;
  // Few heads: pieces of two tiles where there are enough of them for the partial sums to count (one head of 128 with
  // 2,331 tokens 102 us in 37 + 37 pieces, 99 in 19 + 19; three with 900 tokens 91 in 15 + 15, 94 in 8 + 8).
  const int64_t most = tiles < 16 ? tiles : (tiles + 1) / 2;
  double best = 1e300;
  for (int rounds = 1; rounds <= 3; ++rounds) {
    int64_t p = rounds * slots / (2 * (int64_t)BH);   // both kinds together
    if (p < 2) p = 2;
    int64_t c2 = (p + 1) / 2, c1 = p / 2;
    if (c2 > most) c2 = most;
    if (c1 > most) c1 = most;
    const double t2 = piece + tile2 * (double)((tiles + c2 - 1) / c2), t1 = piece + tile1 * (double)((tiles + c1 - 1) / c1);
    const double mean = (c2 * t2 + c1 * t1) / (double)(c2 + c1), longest = t2 > t1 ? t2 : t1;
    const int64_t groups = 2 * (int64_t)BH * (c2 + c1), full = (groups + slots - 1) / slots - 1;
    const double cost = full > 0 ? (double)full * mean + longest : 0.6 * longest + 0.4 * mean;
    if (cost < 0.98 * best) {
      best = cost;
      *n2 = (int)c2;
      *n1 = (int)c1;
    }
  }
}

hipError_t launch_weight_grad(const WeightGradArgs& a, int d, int grid, hipStream_t stream) {
  if (d == 128) hipLaunchKernelGGL((weight_grad_kernel<128, 8>), dim3(grid), dim3(512), 0, stream, a);
  else hipLaunchKernelGGL((weight_grad_kernel<64, 4>), dim3(grid), dim3(256), 0, stream, a);
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------
// Sum of the per-workgroup partials over batch and pieces, in a fixed order.
// ------------------------------------------------------------------------------------
// A wave sums 256 elements, 16 bytes per lane and kReduceDepth partials in flight; a block holds four
// such waves, or, for a tensor of no more elements (the biases, with up to a few hundred partials),
// four waves of every fourth partial, combined in a fixed order.  A transposed job (dW1, whose
// partials are [d][hidden]) takes its 256 elements as 8 rows of 32, so that reads are whole 128-byte
// lines and the stores leave in runs of 32 bytes.
// Bound by launching the blocks and one round trip to the partials (26 MB at 12 heads of 128, mostly in
// the last-level cache): with a grid of 256 blocks for every tensor, most of them idle for the
// biases, and the partials of every element split over four waves, 15 us; now 11.
constexpr int kReduceDepth = 6;
__global__ void __launch_bounds__(256)
reduce_kernel(ReduceJobs jobs) {
  __shared__ __attribute__((aligned(16))) float sums[4][256];
  int j = 0;
  while (j + 1 < jobs.n && (int)blockIdx.x >= jobs.first[j + 1]) ++j;
  const ReduceArgs& a = jobs.job[j];
  const int h = blockIdx.y;
  const int q = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int n = a.R * a.C;   // a multiple of 4 (of 256 with rows of whole 32s when transposed)
  const bool tall = n <= 256;
  const int group = tall ? 0 : 4 * ((int)blockIdx.x - jobs.first[j]) + q;   // of 256 elements
  int i = 256 * group + 4 * lane, r0 = 0, c0 = 0;
  if (a.transpose) {   // 8 x 32 elements
    const int cbs = a.C / 32;
    r0 = 8 * (group / cbs);
    c0 = 32 * (group % cbs);
    i = (r0 + (lane >> 3)) * a.C + c0 + 4 * (lane & 7);
  }
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  if (256 * group + 4 * lane < n) {
    const int total = a.B * a.per_bh, step = tall ? 4 : 1;
    const float* const p0 = a.part + a.part_off + i;
    int b = 0, s = tall ? q : 0;   // partial m = b * per_bh + s
    for (int m = s; m < total; m += step * kReduceDepth) {
      f32x4 x[kReduceDepth];
#pragma unroll
      for (int u = 0; u < kReduceDepth; ++u) {
        x[u] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (m + step * u < total) {
          while (s >= a.per_bh) {
            s -= a.per_bh;
            ++b;
          }
          x[u] = *reinterpret_cast<const f32x4*>(p0 + ((int64_t)(b * a.H + h) * a.per_bh + s) * a.part_stride);
          s += step;
        }
      }
#pragma unroll
      for (int u = 0; u < kReduceDepth; ++u) acc += x[u];
    }
  }
  float* const out = a.out + (int64_t)h * n;
  if (!tall && !a.transpose) {
    if (256 * group + 4 * lane < n) *reinterpret_cast<f32x4_u*>(out + i) = acc;
    return;
  }
  *reinterpret_cast<f32x4*>(&sums[q][4 * lane]) = acc;
  __syncthreads();
  if (tall) {
    const int t = threadIdx.x;
    if (t < n) out[t] = ((sums[0][t] + sums[1][t]) + sums[2][t]) + sums[3][t];
    return;
  }
  if (256 * group >= n) return;
  const int col = lane >> 1, row = 4 * (lane & 1);
  const f32x4 y = {sums[q][row * 32 + col], sums[q][(row + 1) * 32 + col], sums[q][(row + 2) * 32 + col],
                   sums[q][(row + 3) * 32 + col]};
  *reinterpret_cast<f32x4_u*>(out + (int64_t)(c0 + col) * a.R + r0 + row) = y;
}

hipError_t launch_reduce(const ReduceJobs& given, hipStream_t stream) {
  ReduceJobs jobs = given;
  int blocks = 0;
  for (int j = 0; j < jobs.n; ++j) {
    jobs.first[j] = blocks;
    blocks += (jobs.job[j].R * jobs.job[j].C + 1023) / 1024;
  }
  hipLaunchKernelGGL(reduce_kernel, dim3(blocks, jobs.job[0].H), dim3(256), 0, stream, jobs);
  return hipGetLastError();
}

__global__ void __launch_bounds__(256)
fill_zero_kernel(float* p, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) p[i] = 0.f;
}

hipError_t launch_fill_zero(float* p, int64_t n, hipStream_t stream) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(fill_zero_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream, p, n);
  return hipGetLastError();
}

}  // namespace rehyat
