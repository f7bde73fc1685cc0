// Body of the chunk-state kernel (rehyat_state.hip), also run by workgroups of the streaming
// step's attention launch (rehyat_attn.hip).
#pragma once
#include <type_traits>

#include "rehyat_device.h"
#include "rehyat_kernels.h"

namespace rehyat {

// LDS of the body: K and V tiles (two of each), U of two tiles, the first-layer bias
template <int D>
struct StateLds {
  static constexpr int XV = 4 * 64 * 2 * D;             // bytes
  static constexpr int US = 2 * 64 * (2 * D * 2 + 16);
  static constexpr int B1 = 2 * D * 4;
};

// The work of workgroup `block`; XV, Us and B1s as in StateLds, 1024-, 1024- and 256-byte aligned.
// Waves beyond NW must not enter.  QUERIES: query segments with a scale and a weight per token (StateArgs), which
// arrive with the tiles: Tok holds 64 of both for two tiles.
template <int D, int NW, bool QUERIES = false>
__device__ __forceinline__ void state_body(const StateArgs& a, int block, char* XV, char* Us, float* B1s,
                                           float* Tok = nullptr) {
  constexpr int HID = 2 * D, DP = 2 * D;
  constexpr int KS = D / 16;      // k-steps across the head dimension
  constexpr int KS2 = HID / 16;   // k-steps across the hidden layer
  constexpr int DB = D / 32;      // 32-row blocks of the head dimension
  constexpr int TB = 64 * 2 * D;  // bytes of a K, V or W1 tile (64 rows of 2D bytes)
  constexpr int UROW = HID * 2;   // bytes of a row of U
  static_assert(DP / NW == 32, "each wave owns 32 features");
  // Dot products for z where vector work bounds a tile (d = 64; unpacked 2 - 4 % slower).  At
  // d = 128 the state kernel takes the same time either way, and the pieces in an attention launch less
  // unpacked (steps of 64 heads with 2,048 tokens absorbed: 167.6 us, 161.5 unpacked).
  constexpr bool kDotSum = D == 64;

  // U[token][hidden] with 16 bytes of padding per row: consecutive rows start four banks
  // apart, so fragment reads and writes are conflict-free without a chunk permutation
  constexpr int UPAD = UROW + 16;
  static_assert(KS2 == 2 * KS && NW * 32 * 2 * D <= StateLds<D>::XV && NW * 32 * 2 * D <= StateLds<D>::US, "staging");
  static_assert(StateLds<D>::XV == 4 * TB && StateLds<D>::US == 2 * 64 * UPAD && StateLds<D>::B1 == HID * 4, "LDS layout");

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform for the compiler too
  const int g = lane >> 5;
  const int r = lane & 31;

  const int item = xcd_swizzle(block, a.items_per_xcd);
  if (item >= a.n_items) return;
  const int sp = item % a.nsplit;
  const int rest = item / a.nsplit;
  const int seg = rest % a.n_seg;
  const int bh = rest / a.n_seg;
  const int h = bh % a.H;

  // token range of this piece
  int64_t seg_lo = 0, seg_hi = a.step_n;
  if (a.step_n <= 0) {
    const int tt = a.chunk0 + seg;
    const int nchunks = num_chunks(a.T, a.chunk);
    const ChunkRange cr = chunk_range(a.T, a.HW, a.chunk, a.overlap, tt);
    if (QUERIES) {   // the queries of chunk tt
      seg_lo = cr.q_lo;
      seg_hi = cr.q_hi;
    } else {
      seg_lo = cr.s_lo;
      seg_hi = (tt + 1 < nchunks) ? chunk_range(a.T, a.HW, a.chunk, a.overlap, tt + 1).s_lo
                                  : (int64_t)a.T * a.HW;
    }
  }
  const int64_t len = seg_hi - seg_lo;
  const int64_t lo = seg_lo + (len * sp) / a.nsplit;
  const int64_t hi = seg_lo + (len * (sp + 1)) / a.nsplit;
  const int n_tokens = (int)(hi - lo), n_tiles = (n_tokens + 63) / 64;

  const char* Kb = reinterpret_cast<const char*>(a.k + (int64_t)bh * a.kv_bh_stride + lo * D);
  const char* Vb = reinterpret_cast<const char*>(a.v + (int64_t)bh * a.kv_bh_stride + lo * D);

  // ---- resident operands ----------------------------------------------------
  // first-layer bias in LDS: accumulator register 4i+j is hidden unit 32w + 8i + 4g + j, so a
  // lane reads its four rows of block i with one 16-byte read
  const float b1v = tid < HID ? a.b1_k[(int64_t)h * HID + tid] : 0.f;
  const float* const b1rows = B1s + wave * 32 + 4 * g;
  const int unit = wave * 32 + r;  // this lane's hidden unit (first half) and feature (second half)
  float b2v = a.b2_k[(int64_t)h * DP + unit];
  bf16x8 w1f[KS];   // A operands: row = hidden unit, k = head dimension
  bf16x8 w2f[KS2];  // B operands: column = feature, k = hidden
  // They come by way of the tile buffers (K and V: W1, U: W2 in two halves of its columns), whole rows to an
  // instruction: U of the first tile begins 3.2 us after the workgroup's start (108 workgroups, 2 x 3 heads of 333-token
  // frames; 6.2 with 240), as operands read from memory 6.8 (and 9.7).
  const u32x4 W1r = make_rsrc_words(a.w1_k + ((int64_t)h * HID + wave * 32) * D);
  const u32x4 W2r = make_rsrc_words(a.w2_k + ((int64_t)h * DP + wave * 32) * HID);
  char* const stage1 = XV + wave * (32 * 2 * D);
  char* const stage2 = Us + wave * (32 * 2 * D);
  stage_rows<2 * D>(W1r, 2 * D, 0, lds_address(stage1), lane);
  stage_rows<2 * D>(W2r, 4 * D, 0, lds_address(stage2), lane);
  // tile `it` of K or V goes into the buffer of its parity
  const u32x4 Kr = make_rsrc_words(Kb), Vr = make_rsrc_words(Vb);
  const uint32_t k_lds = lds_address(XV), v_lds = k_lds + 2 * TB;
  using R = RangeTiles<2 * D, NW>;
  const R range(n_tokens, wave, lane);
  // scales by even waves, weights by odd ones
  const int64_t tok0 = QUERIES ? (int64_t)bh * a.T * a.HW + lo : 0;
  const u32x4 Tr = make_rsrc_words(QUERIES ? (const void*)((wave & 1 ? a.tok_weight : a.tok_scale) + tok0) : (const void*)Kb);
  const uint32_t tok_lds = QUERIES ? __builtin_amdgcn_readfirstlane(lds_address(Tok) + 256 * (wave & 1)) : 0u;
  auto load_tok = [&](int it) {
    const int row = n_tokens < 64 ? 0 : 64 * it < n_tokens - 64 ? 64 * it : n_tokens - 64;
    int ln = lane;
    asm volatile("" : "+v"(ln));
    direct_load_4(Tr, 4 * (ln < n_tokens ? ln : n_tokens - 1), __builtin_amdgcn_readfirstlane(4 * row),
                  tok_lds + (it & 1) * 512);
  };
  const int uwbase = r * UPAD + wave * 64 + 8 * g;   // write: token r, units 32w + 8i + 4g .. +3 at + 16 i
  const int urbase = r * UPAD + 16 * g;              // read: A fragment of token r, k-step ks at + 32 ks

  // state slice: acc[db] register 4i+j = (row d = 32db+8i+4g+j, feature 32w+r)
  f32x16 acc[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[db][e] = 0.f;
  float zacc = 0.f;

  // U^T slice of a tile = relu(W1[slice] X^T + b1[slice]) -> U[token][hidden]: accumulators that start
  // from the bias (no addition per element), rectified and stored four units at a time
  auto u_start = [&]() {
    f32x16 u;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const f32x4 bb = *reinterpret_cast<const f32x4*>(b1rows + 8 * i);
#pragma unroll
      for (int j = 0; j < 4; ++j) u[4 * i + j] = bb[j];
    }
    return u;
  };
  auto u_store = [&](const f32x16& u, int i, char* Ud, int tb) {   // register 4i+j = (hidden 32w+8i+4g+j, token 32tb+r)
    u32x2 pk;
    pk[0] = pack_bf16(fmaxf(u[4 * i], 0.f), fmaxf(u[4 * i + 1], 0.f));
    pk[1] = pack_bf16(fmaxf(u[4 * i + 2], 0.f), fmaxf(u[4 * i + 3], 0.f));
    *reinterpret_cast<u32x2*>(Ud + uwbase + 16 * i + tb * (32 * UPAD)) = pk;
  };
  auto opaque_lane = [&]() {   // offsets derived from it are recomputed per tile, not held in registers
    int ln = lane;
    asm volatile("" : "+v"(ln));
    return ln;
  };
  // fragment of token row r, k-step ks of a K tile: ^ 32 ks (the chunk bits of the permuted layout do
  // not overlap the row bits)
  auto x_base = [&](int ln) { return tile_off<2 * D>(ln & 31, 8 * (ln >> 5)); };
  // transposing reads of V: columns 32 db .. at ^ 64 db, tokens eight rows further down at ^ 32 there
  auto v_base = [&](int ln) {
    return tile_off<2 * D>(4 * (ln >> 5) + ((ln & 15) >> 2), 16 * ((ln & 31) >> 4) + 4 * (ln & 3));
  };
  auto u_fragment = [&](const char* Uc, int tb, int ks) {
    return *reinterpret_cast<const bf16x8*>(Uc + urbase + 32 * ks + tb * (32 * UPAD));
  };

  constexpr int PD = 4;   // fragments read ahead of their products
  bf16x8 fr[PD];
  wave_loads_done();
  if (tid < HID) B1s[tid] = b1v;
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    w1f[ks] = staged_fragment<2 * D>(stage1, lane, ks);
    w2f[ks] = staged_fragment<2 * D>(stage2, lane, ks);
  }
  wave_reads_done();
  stage_rows<2 * D>(W2r, 4 * D, 2 * D, lds_address(stage2), lane);
  lds_barrier();   // W1 has been read by all waves, the bias is in LDS
  if (n_tiles > 0) {
    range.fill(Kr, 0, k_lds);
    range.fill(Vr, 0, v_lds);
    if (n_tiles > 1) range.fill(Kr, 64, k_lds + TB);
    if (QUERIES) load_tok(0);
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * R::LPT) : "memory");   // W2; two tiles at least are younger
  } else {
    wave_loads_done();
  }
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) w2f[KS + ks] = staged_fragment<2 * D>(stage2, lane, ks);
  settle(w1f);
  settle(w2f);
  settle(b2v);
  if (n_tiles > 0) {
    wait_loads_and_barrier<0>();   // also: all waves have read W2
    const int ln = opaque_lane();
    const int xbase = x_base(ln);
#pragma unroll
    for (int tb = 0; tb < 2; ++tb) {
      f32x16 u = u_start();
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
        u = mfma(w1f[ks], *reinterpret_cast<const bf16x8*>(XV + (xbase ^ (32 * ks)) + tb * (32 * 2 * D)), u);
#pragma unroll
      for (int i = 0; i < 4; ++i) u_store(u, i, Us, tb);
    }
    lds_barrier();   // U of tile 0 is complete
  }

  // Step `it` runs the second half of tile `it` -- psi, phi and V^T phi -- together with the first
  // half of tile it+1 (independent instruction streams inside every wave), in this order of
  // products: psi of tokens 0..31, U(it+1) of 0..31, psi of 32..63, U(it+1) of 32..63, the state
  // products of both.  Each group's vector work lies under the products of the next group and every
  // operand is read PD products ahead; the order is fenced slot by slot, because the compiler waits
  // for each LDS read right after issuing it otherwise.
  // One barrier per tile, with PD products still to be issued: U(it+1) is complete, every wave has
  // read its last operands of tile `it`, and K(it+2) and V(it+1), requested as the step began, have landed.
  auto tile_step = [&](auto MOREC, auto SQC, int it) {
    constexpr bool MORE = decltype(MOREC)::value;        // a tile follows; this one is full
    constexpr bool squared = decltype(SQC)::value;
    const char* const Vs = XV + (2 + (it & 1)) * TB;
    const char* const Xs = XV + ((it + 1) & 1) * TB;
    const char* const Uc = Us + (it & 1) * (64 * UPAD);
    char* const Ud = Us + ((it + 1) & 1) * (64 * UPAD);
    const int ln = opaque_lane();
    const int xbase = x_base(ln), vbase = v_base(ln);
    const int first = range.first(64 * it), count = range.count(64 * it);   // tokens of the last tile
    const u32x4 Kd = rsrc_if(Kr, it + 2 < n_tiles);
    const int ks = range.soff(64 * (it + 2)), vs = range.soff(64 * (it + 1));
    const uint32_t kd = k_lds + (it & 1) * TB, vd = v_lds + ((it + 1) & 1) * TB;
    constexpr int LP = KS2, LF = MORE ? KS : 0, LS = 2 * DB;
    constexpr int F0 = LP, P1 = LP + LF, F1 = P1 + LP, S0 = F1 + LF, S1 = S0 + LS, NM = S1 + LS;
    static_assert(NM % PD == 0, "the fragment ring closes over a step");
    static_assert(S0 + 3 < NM - PD, "U is stored before the barrier that publishes it");
    f32x16 u[2], ps[2];
    uint32_t fb[2][8];   // phi as operands
    constexpr int kPairs = 8 / LS;       // element pairs per slot
    f32x2 scale[kPairs], weight[kPairs]; // of a slot's tokens, read one slot ahead
    auto read_tok = [&](int tb, int i) {
#pragma unroll
      for (int n = 0; n < kPairs; ++n) {
        const float* const p = Tok + (it & 1) * 128 + 32 * tb + 8 * ((i + n) >> 1) + 4 * g + 2 * ((i + n) & 1);
        scale[n] = *reinterpret_cast<const f32x2*>(p);
        weight[n] = *reinterpret_cast<const f32x2*>(p + 64);
      }
    };
    float part[2] = {0.f, 0.f};
    auto fetch = [&](auto MC) {   // the LDS operand of product m
      constexpr int m = decltype(MC)::value;
      if constexpr (m >= NM) {
        if constexpr (MORE) fr[m % PD] = u_fragment(Ud, 0, m - NM);   // psi of the next tile
      } else if constexpr (m < F0 || (m >= P1 && m < F1)) {
        fr[m % PD] = u_fragment(Uc, m >= P1, m - (m >= P1 ? P1 : 0));
      } else if constexpr (m < S0) {
        constexpr int tb = m >= F1, ks = m - (tb ? F1 : F0);
        if constexpr (ks == 0) u[tb] = u_start();
        fr[m % PD] = *reinterpret_cast<const bf16x8*>(Xs + (xbase ^ (32 * ks)) + tb * (32 * 2 * D));
      } else {
        constexpr int tb = m >= S1, n = m - (tb ? S1 : S0), s = n / DB, db = n % DB;
        const char* const p = Vs + (2 * tb + s) * (16 * 2 * D);
        fr[m % PD] = join_tr(lds_read_tr(reinterpret_cast<const bf16_t*>(p + (vbase ^ (64 * db)))),
                             lds_read_tr(reinterpret_cast<const bf16_t*>(p + (vbase ^ (64 * db) ^ 32) + 8 * 2 * D)));
      }
    };
    auto product = [&](auto MC) {
      constexpr int m = decltype(MC)::value;
      if constexpr (m < F0 || (m >= P1 && m < F1)) {
        constexpr int tb = m >= P1, ks = m - (tb ? P1 : 0);   // rows = tokens, columns = features
        ps[tb] = mfma(fr[m % PD], w2f[ks], ks == 0 ? f32x16{} : ps[tb]);
      } else if constexpr (m < S0) {
        constexpr int tb = m >= F1, ks = m - (tb ? F1 : F0);
        u[tb] = mfma(w1f[ks], fr[m % PD], u[tb]);
      } else {
        constexpr int tb = m >= S1, n = m - (tb ? S1 : S0), s = n / DB, db = n % DB;
        const u32x4 w = {fb[tb][4 * s], fb[tb][4 * s + 1], fb[tb][4 * s + 2], fb[tb][4 * s + 3]};
        acc[db] = mfma(fr[m % PD], __builtin_bit_cast(bf16x8, w), acc[db]);
      }
    };
    auto phi = [&](auto TBC, auto IC) {   // elements 2i, 2i+1 of psi
      constexpr int tb = decltype(TBC)::value, i = decltype(IC)::value;
      float x[2];
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int e = 2 * i + j;
        x[j] = fmaxf(ps[tb][e] + b2v, 0.f);
        if (squared) x[j] = x[j] * x[j];
        if (!MORE && (unsigned)(32 * tb + 8 * (e >> 2) + 4 * g + (e & 3) - first) >= (unsigned)count) x[j] *= kAgain;
        if (QUERIES) {
          part[tb] += weight[i % kPairs][j] * x[j];
          x[j] *= scale[i % kPairs][j];
        }
      }
      fb[tb][i] = pack_bf16(x[0], x[1]);
      // The normaliser sums the features as rounded for the product: with unrounded ones S and z
      // weigh a token differently, and for keys that resemble each other the differences add up
      // (equal keys: error of y against fp64 up to 30 % larger, of gradients 40 %).
      if (!QUERIES) part[tb] = sum_pair<kDotSum>(fb[tb][i], part[tb]);
      pin(part[tb]);
      pin(fb[tb][i]);
    };
    static_for<NM>([&](auto MC) {
      constexpr int m = decltype(MC)::value;
      if constexpr (MORE && m == NM - PD) wait_loads_and_barrier<0>();
      product(MC);
      fetch(std::integral_constant<int, m + PD>{});
      if constexpr (MORE && m % 2 == 1 && m < 4 * R::LPT) {
        constexpr int i = m / 2;
        if constexpr (i < R::LPT) range.template load<i>(Kd, ks, kd);
        else range.template load<i - R::LPT>(Vr, vs, vd);
      }
      if constexpr (QUERIES && MORE && m == 4 * R::LPT + 1) load_tok(it + 1);
      static_for<2>([&](auto TBC) {
        constexpr int tb = decltype(TBC)::value;
        constexpr int p = m - (tb ? F1 : F0) - 2;   // two products behind the group's last one
        if constexpr (p >= 0 && kPairs * p < 8)
          static_for<kPairs>([&](auto JC) { phi(TBC, std::integral_constant<int, kPairs * p + decltype(JC)::value>{}); });
        if constexpr (QUERIES && p >= -1 && kPairs * (p + 1) < 8) read_tok(tb, kPairs * (p + 1));
        constexpr int q = m - (tb ? S0 : P1) - 2;   // two quads of units per slot: done before the barrier
        if constexpr (MORE && q >= 0 && q < 2) {
          u_store(u[tb], 2 * q, Ud, tb);
          u_store(u[tb], 2 * q + 1, Ud, tb);
        }
      });
      __builtin_amdgcn_sched_barrier(0);
    });
    zacc += part[0];
    zacc += part[1];
  };

  // A loop for each half of the features: decided per element, squaring costs a select each (the
  // waves of both loops meet at the same number of barriers).
  // What bounds a tile: products at the rate that power allows with all CUs busy (26.6 ns each per SIMD; a
  // loop of nothing but the same products, vector work and LDS reads 21 - 24.5, by box, and 14.1 with 32 CUs; at
  // d = 64 33 ns against 25 and 14.2).  With the groups one after the other and each LDS read waited
  // for as it was issued: 480p and 320x480 launches of 12 heads of 128 together 68.4 us, now 66.3; 24 heads of 64
  // at 480p 70.3, now 64.5; 2 x 3 heads of 333-token frames 19.5, now 18.1.
  auto all_tiles = [&](auto SQC) {
    // (Read here and not before the branch: there they were kept, spilled, for the loop behind the other one, whose
    // every step then waited for all loads in flight at their first use.)
    if (n_tiles > 0) {
      static_for<PD>([&](auto MC) { fr[decltype(MC)::value] = u_fragment(Us, 0, decltype(MC)::value); });
    }
    for (int it = 0; it + 1 < n_tiles; ++it) tile_step(std::true_type{}, SQC, it);
    if (n_tiles > 0) tile_step(std::false_type{}, SQC, n_tiles - 1);
  };
  if (wave * 32 >= DP / 2) all_tiles(std::true_type{});
  else all_tiles(std::false_type{});

  // ---- write the partial: S^T [d][DP] fp32, then z [DP] ---------------------------
  // Through the XCD's L2 to memory at once (stores of agent scope): what a launch leaves dirty there is written back when
  // it ends, before the next one begins.  2 x 3 heads of 333-token frames 47.0 -> 45.0 us a call, 21 streaming steps at
  // 480p, whose pieces end long before their launch, 1,205 -> 1,179, one layer at 480p 498 -> 496.6.  (The outputs'
  // 8-byte pieces that way: 480p +11 %, they need the L2 to become whole lines.  States, the weight gradients' partial sums
  // and dpsi: even.)
  float* P = a.partial + ((int64_t)bh * a.partial_slots + (int64_t)seg * a.nsplit + sp) * (int64_t)(D * DP + DP);
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int row = 32 * db + 8 * (e >> 2) + 4 * g + (e & 3);
      __hip_atomic_store(P + row * DP + unit, acc[db][e], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  const float ztot = half_swap_sum(zacc);
  if (g == 0) P[D * DP + unit] = ztot;
}

}  // namespace rehyat
