// Fused hybrid-attention output kernel for gfx950.
//
// One workgroup (4 waves) owns 128 consecutive query tokens of one chunk of one (batch, head); each
// wave owns 32 of them and keeps, per query, the running softmax maximum and sum and the d-wide
// numerator in MFMA accumulators.
//
//   phase S (Eq. 6, 8): exponents K Q^T over the chunk's softmax window
//            (Eq. 12), online maximum/sum, numerator V^T P.
//   phase L (Eq. 7, 9, 16): phi_q of the wave's queries (two-layer MLP, second
//            half squared), then the read-out S_t^T phi_q and z_t . phi_q of
//            the chunk state, accumulated INTO the softmax numerator and
//            normaliser -- to the MFMA pipeline the D' state rows are just D'
//            more "keys" whose weights are the phi_q features.
//   merge  (Eq. 5): divide, round to bf16, store.
//
// Everything is computed transposed (keys / features in accumulator rows,
// queries in lanes) so that per-query statistics live in one lane and each
// product's accumulator is directly the B operand of the next product.
//
// All operands that are shared by the four waves (K and V tiles, then W1, W2
// and the chunk state) travel global -> LDS with direct loads into four LDS
// tile buffers, issued one or more steps ahead of their use (as inline asm: the
// compiler must not order LDS reads behind loads into other buffers).
#include <cstdio>
#include <type_traits>

#include "rehyat_device.h"
#include "rehyat_kernels.h"
#include "rehyat_state_body.h"

namespace rehyat {

// The exponentials of a row are taken relative to a reference that follows the row's
// running maximum lazily: it moves only when a tile's maximum exceeds it by more than
// this many powers of two, so the rescale of the running sums is rare after the first
// tile, and weights stay below 2^kLazyMax (harmless for bf16 weights and fp32 sums; the
// final division cancels the reference).  The true maximum is tracked beside it.
constexpr float kLazyMax = 8.0f;
// Where the reference starts: finite, so that a row whose first key tiles score -inf (or a group
// of waves that sees no key of a row) weighs them exp2(-inf - reference) = 0, not a NaN.
constexpr float kLowest = -3.402823466e38f;
constexpr int kAttnNW = 4;                      // waves that share the 128 queries of a workgroup
constexpr int kQueryTile = 32 * kAttnNW;

template <int D>
struct AttnShape {
  static constexpr int HID = 2 * D;
  static constexpr int DP = 2 * D;
  static constexpr int KS = D / 16;    // k-steps across the head dimension
  static constexpr int DB = D / 32;    // 32-row blocks across the head dimension
  static constexpr int TILE_BYTES = 64 * D * 2;  // one LDS tile: 64 rows of 2D bytes
};

// Fragment reads inside a K / V tile.  K rows r (+32 per key block), k-step ks: `k` ^ 32 ks.
// Transposing reads of V, tokens 4g..4g+3 of a 16-token step, features 32 db..: `v` ^ 64 db, and
// tokens 8+4g..: ^ 32 of that, eight rows further down.  (The chunk permutation of a row is an
// exclusive-or that looks at the low four bits of the row only.)
struct FragBase {
  int k, v;
};
template <int D>
__device__ __forceinline__ FragBase make_frag_base(int lane) {
  FragBase f;
  f.k = tile_off<2 * D>(lane & 31, 8 * (lane >> 5));
  f.v = tile_off<2 * D>(4 * (lane >> 5) + ((lane & 15) >> 2), 16 * ((lane & 31) >> 4) + 4 * (lane & 3));
  return f;
}
template <int D>
__device__ __forceinline__ bf16x8 k_fragment(const char* Ks, const FragBase& fo, int ks, int kb) {
  return *reinterpret_cast<const bf16x8*>(Ks + (fo.k ^ (32 * ks)) + kb * (32 * D * 2));
}
template <int D>
__device__ __forceinline__ bf16x8 v_fragment(const char* Vs, const FragBase& fo, int step, int db) {
  const char* const p = Vs + step * (16 * D * 2);
  return join_tr(lds_read_tr(reinterpret_cast<const bf16_t*>(p + (fo.v ^ (64 * db)))),
                 lds_read_tr(reinterpret_cast<const bf16_t*>(p + (fo.v ^ (64 * db) ^ 32) + 8 * 2 * D)));
}

// Fragments of A operands that a wave keeps ahead of its products.
constexpr int kAhead = 4;

// What a wave keeps of its 32 queries (one per lane, both lane halves) over the key tiles.
template <int D>
struct SoftmaxRows {
  f32x16 O[D / 32];   // numerator: O[db] register 4i+j = (row d = 32db + 8i + 4g + j, query r)
  float ref;          // reference of the exponentials (log2 units), lags the running maximum
  float max;          // running maximum of exponent * log2(e)/sqrt(d)
  float sum;          // this lane half's share of the sum
};

template <int D>
__device__ __forceinline__ void softmax_rescale(SoftmaxRows<D>& s, float tile_max) {
  s.max = fmaxf(s.max, tile_max);
  const bool grow = tile_max > s.ref + kLazyMax;
  if (__any(grow)) {
    const float ref = grow ? tile_max : s.ref;
    const float alpha = __builtin_amdgcn_exp2f(s.ref - ref);
    s.ref = ref;
    s.sum *= alpha;
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
      for (int e = 0; e < 16; ++e) s.O[db][e] *= alpha;
  }
}

// Exponents K Q^T of one 64-key tile (Eq. 6): E[kb] register 4i+j = (key 32kb + 8i + 4g + j, query r).
template <int D>
__device__ __forceinline__ void softmax_scores(const char* Ks, const FragBase& fo, const bf16x8 (&Qr)[D / 16],
                                               f32x16 (&E)[2]) {
  constexpr int NM = D / 8;
  bf16x8 fr[kAhead];
  static_for<kAhead>([&](auto MC) {
    constexpr int m = decltype(MC)::value;
    fr[m] = k_fragment<D>(Ks, fo, m / 2, m & 1);
  });
  static_for<NM>([&](auto MC) {
    constexpr int m = decltype(MC)::value;
    E[m & 1] = mfma(fr[m % kAhead], Qr[m / 2], m < 2 ? f32x16{} : E[m & 1]);
    if constexpr (m + kAhead < NM) fr[m % kAhead] = k_fragment<D>(Ks, fo, (m + kAhead) / 2, (m + kAhead) & 1);
    __builtin_amdgcn_sched_barrier(0);
  });
}

// One 64-key tile t of the softmax part (Eq. 6, 8) for the wave's 32 queries, together with the
// exponents of tile t+1: online maximum and sum of E, numerator += V^T P, and En = K(t+1) Q^T.
//
// A wave's own chain over one tile (scores, maximum, exponentials, numerator) leaves the matrix
// unit idle for more than half of its time, and a second wave on the SIMD cannot fill all of that: both
// chains have the same gaps.  Here the products of the next tile's scores run over the maximum
// and the first exponentials of this one, and the numerator's over the rest.  The order is written out
// slot by slot -- a slot is one product, one fragment read kAhead products ahead, its share of
// the vector work -- and fenced, because the compiler's own order waits for every LDS read right
// after issuing it.
// What bounds it: on a filled chip power (a loop of nothing but the same products, vector work and LDS reads,
// on random operands: 23 - 27 ns per product and SIMD with all CUs busy, by box, 14.5 with 32; here 28 - 30, 25
// without the tile loads), at d = 64 power and vector work (32 - 34 ns in such a loop, 23 with 32 CUs); with CUs to spare the
// issue of some 300 instructions per tile and wave.  Against the tile loop that ran the four phases one after
// the other: 1,488 -> 1,389 us summed over the 480p, 720p and three-frame-chunk guidance-pair launches,
// streaming step at 480p with T_o = 1 60 -> 55 us, d = 64 at 480p 441 -> 430 us.
//
// The one barrier per tile stands where the last K fragment of tile t+1 has been read and kAhead
// products are still to be issued, so that its wait and the first V fragments' latency lie under
// those; the first K fragments of tile t+2 are read under the last products of the numerator.  At the barrier
// K(t+2) and V(t) have landed, and everyone is done with K(t+1) and V(t-1): `issue(i)`, i <
// 2 LPT, requests K(t+3) and V(t+1), spread over the slots that follow (a wave that issues its
// loads in one go stalls until the address unit has taken them all).
// fr: the first kAhead K fragments of tile t+1 on entry, of tile t+2 on exit.
template <int D, int LPT, typename Issue>
__device__ __forceinline__ void softmax_trip(const char* Kn, const char* Kn2, const char* Vc, const FragBase& fo,
                                             const bf16x8 (&Qr)[D / 16], f32x16 (&E)[2], f32x16 (&En)[2],
                                             bf16x8 (&fr)[kAhead], SoftmaxRows<D>& rows, float sc, Issue issue) {
  constexpr int KS = D / 16, DB = D / 32;
  constexpr int NQ = 2 * KS, NV = 4 * DB, NM = NQ + NV;
  static_assert(NM % kAhead == 0, "the fragment ring closes over a trip");
  constexpr int BAR = NQ - kAhead;                  // slot that the barrier precedes
  constexpr int MS = D == 128 ? 4 : 2;              // slots of the maximum
  constexpr int S0 = MS + 3;                        // slot of the first exponential
  constexpr int W = NQ + 3 * DB - 1 - S0;           // .. and how many slots they spread over
  constexpr int LS = 2;                             // slots per load
  static_assert(BAR + 1 + LS * (2 * LPT - 1) < NM, "the loads fit behind the barrier");
  uint32_t pw[16];
  float sum = 0.f, mx[2], pe[8];
  auto fetch = [&](auto MC) {
    constexpr int m = decltype(MC)::value;
    if constexpr (m < NQ) fr[m % kAhead] = k_fragment<D>(Kn, fo, m / 2, m & 1);
    else if constexpr (m < NM) fr[m % kAhead] = v_fragment<D>(Vc, fo, (m - NQ) / DB, (m - NQ) % DB);
    else fr[m % kAhead] = k_fragment<D>(Kn2, fo, (m - NM) / 2, m & 1);
  };
  auto product = [&](auto MC) {
    constexpr int m = decltype(MC)::value;
    if constexpr (m < NQ) {
      En[m & 1] = mfma(fr[m % kAhead], Qr[m / 2], m < 2 ? f32x16{} : En[m & 1]);
    } else {
      constexpr int step = (m - NQ) / DB, db = (m - NQ) % DB;
      const u32x4 w = {pw[4 * step], pw[4 * step + 1], pw[4 * step + 2], pw[4 * step + 3]};
      rows.O[db] = mfma(fr[m % kAhead], __builtin_bit_cast(bf16x8, w), rows.O[db]);
    }
  };
  // element i of the tile is register i & 15 of key block i >> 4; eight of them make the operand of a
  // 16-key step.  Its exponential stands in slot_of(i), its sum and rounding one slot later.
  auto slot_of = [](int i) { return S0 + i * W / 32; };
  static_for<NM>([&](auto MC) {
    constexpr int m = decltype(MC)::value;
    if constexpr (m == BAR) wait_loads_and_barrier<0>();
    product(MC);
    fetch(std::integral_constant<int, m + kAhead>{});
    if constexpr (m > BAR && (m - BAR - 1) % LS == 0 && (m - BAR - 1) / LS < 2 * LPT)
      issue(std::integral_constant<int, (m - BAR - 1) / LS>{});
    if constexpr (m < MS) {
#pragma unroll
      for (int e = m * 16 / MS; e < (m + 1) * 16 / MS; e += 2)
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
          const float pair = fmaxf(E[kb][e], E[kb][e + 1]);
          mx[kb] = e == 0 ? pair : fmaxf(pair, mx[kb]);
        }
    }
    // exponents are kept unscaled; sc = log2(e)/sqrt(d) > 0 is folded into the exp2 argument
    if constexpr (m == MS + 1) mx[0] = half_swap_max(fmaxf(mx[0], mx[1])) * sc;
    if constexpr (m == MS + 2) softmax_rescale<D>(rows, mx[0]);
    static_for<32>([&](auto IC) {
      constexpr int i = decltype(IC)::value;
      if constexpr (slot_of(i) + 1 == m) {
        sum += pe[i & 7];
        if constexpr (i & 1) pw[i >> 1] = pack_bf16(pe[(i & 7) - 1], pe[i & 7]);
      }
    });
    static_for<32>([&](auto IC) {
      constexpr int i = decltype(IC)::value;
      if constexpr (slot_of(i) == m)
        pe[i & 7] = __builtin_amdgcn_exp2f(__builtin_fmaf(E[i >> 4][i & 15], sc, -rows.ref));
    });
    __builtin_amdgcn_sched_barrier(0);
  });
  rows.sum += sum;
}

// The last tile: keys outside [first, first + count) of it have been weighed already.
// `issue(i)`, i < NI, requests tiles of the next phase, one load behind a product.
template <int D, int NI, typename Issue>
__device__ __forceinline__ void softmax_last(const char* Vc, const FragBase& fo, f32x16 (&E)[2], SoftmaxRows<D>& rows,
                                             float sc, int first, int count, int lane, Issue issue) {
  constexpr int DB = D / 32, NM = 4 * DB;
  static_assert(NI <= NM, "a load behind each product");
  const int g = lane >> 5;
  bf16x8 fr[kAhead];
  static_for<kAhead>([&](auto MC) {
    constexpr int m = decltype(MC)::value;
    fr[m] = v_fragment<D>(Vc, fo, m / DB, m % DB);
  });
  float mx = -INFINITY;   // of all 64 keys: the others stand in the window as well
#pragma unroll
  for (int kb = 0; kb < 2; ++kb)
#pragma unroll
    for (int e = 0; e < 16; ++e) mx = fmaxf(mx, E[kb][e]);
  softmax_rescale<D>(rows, half_swap_max(mx) * sc);
  const float again = kAgainLog2 - rows.ref;
  float sum = 0.f;
  uint32_t pw[4];
  static_for<NM>([&](auto MC) {
    constexpr int m = decltype(MC)::value, step = m / DB;
    if constexpr (m % DB == 0) {
#pragma unroll
      for (int i = 0; i < 8; i += 2) {
        float p[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const int e = 8 * (step & 1) + i + j;
          const bool first_time = (unsigned)(32 * (step >> 1) + 8 * (e >> 2) + 4 * g + (e & 3) - first) < (unsigned)count;
          p[j] = __builtin_amdgcn_exp2f(__builtin_fmaf(E[step >> 1][e], sc, first_time ? -rows.ref : again));
          sum += p[j];
        }
        pw[i >> 1] = pack_bf16(p[0], p[1]);
      }
    }
    const u32x4 w = {pw[0], pw[1], pw[2], pw[3]};
    rows.O[m % DB] = mfma(fr[m % kAhead], __builtin_bit_cast(bf16x8, w), rows.O[m % DB]);
    if constexpr (m + kAhead < NM)
      fr[m % kAhead] = v_fragment<D>(Vc, fo, (m + kAhead) / DB, (m + kAhead) % DB);
    if constexpr (m < NI) issue(MC);
  });
  rows.sum += sum;
}

// The softmax part over a wave's key tiles 0 .. n-1 (tile t of it is tile first_tile + t * stride
// of the window): four waves share K in buffers 0/1 and V in 2/3 of `tiles`, picked by the parity of
// t.  Meets n + 1 barriers.  Behind the last of them the K tiles are dead: with `last` the NI loads `issue(i)` go out
// under the last tile.  EARLY: on entry K of tile 0 has landed, the rest of request() is waited for behind its scores.
// Waves that are not live move their share of the tiles and compute nothing.
template <int D>
struct SoftmaxTiles {
  using R = RangeTiles<2 * D, 4>;
  static constexpr int TB = R::TB, LPT = R::LPT;
  u32x4 K, V;
  uint32_t lds;        // address of the four buffers
  const char* tiles;
  R range;             // the window
  int first_tile, stride, n;
  int lane;

  __device__ __forceinline__ int row(int t) const { return 64 * (first_tile + t * stride); }
  __device__ __forceinline__ void request() const {   // what has to be there before run()
    if (n > 0) {
      range.fill(K, row(0), lds);
      range.fill(V, row(0), lds + 2 * TB);
    }
    if (n > 1) range.fill(K, row(1), lds + TB);
  }
  template <bool LIVE, bool EARLY, int NI, typename Issue>
  __device__ __forceinline__ void run(const bf16x8 (&Qr)[D / 16], SoftmaxRows<D>& rows, float sc, bool last,
                                      Issue issue) const {
    FragBase fo = make_frag_base<D>(lane);
    const char *const K0 = tiles, *const K1 = tiles + TB, *const V0 = tiles + 2 * TB, *const V1 = tiles + 3 * TB;
    f32x16 E0[2], E1[2];
    bf16x8 fr[kAhead];
    auto first_fragments = [&]() {
      static_for<kAhead>([&](auto MC) {
        constexpr int m = decltype(MC)::value;
        fr[m] = k_fragment<D>(K1, fo, m / 2, m & 1);
      });
    };
    if constexpr (LIVE) softmax_scores<D>(K0, fo, Qr, E0);
    if constexpr (LIVE && !EARLY) first_fragments();
    if constexpr (EARLY) wait_loads_and_barrier<0>();
    else lds_barrier();
    if constexpr (LIVE && EARLY) first_fragments();
    if (n > 2) range.fill(K, row(2), lds);
    auto trip = [&](int t, const char* Kn, const char* Kn2, const char* Vc, int kbuf, int vbuf, f32x16 (&E)[2],
                    f32x16 (&En)[2]) {
      const u32x4 Kd = rsrc_if(K, t + 3 < n);
      const int ks = range.soff(row(t + 3)), vs = range.soff(row(t + 1));
      const uint32_t kd = lds + kbuf * TB, vd = lds + vbuf * TB;
      auto issue = [&](auto IC) {
        constexpr int i = decltype(IC)::value;
        if constexpr (i < LPT) range.template load<i>(Kd, ks, kd);
        else range.template load<i - LPT>(V, vs, vd);
      };
      if constexpr (LIVE) {
        softmax_trip<D, LPT>(Kn, Kn2, Vc, fo, Qr, E, En, fr, rows, sc, issue);
      } else {
        wait_loads_and_barrier<0>();
        static_for<2 * LPT>([&](auto IC) { issue(IC); });
      }
    };
    int t = 0;
    for (; t + 2 < n; t += 2) {
      trip(t, K1, K0, V0, 1, 3, E0, E1);
      trip(t + 1, K0, K1, V1, 0, 2, E1, E0);
    }
    const char* Vl = V0;
    if (t + 1 < n) {
      trip(t, K1, K0, V0, 1, 3, E0, E1);
      if constexpr (LIVE) {
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) E0[kb] = E1[kb];
      }
      Vl = V1;
      ++t;
    }
    wait_loads_and_barrier<0>();
    const int first = range.first(row(t)), count = range.count(row(t));
    if (NI > 0 && last) {
      if constexpr (LIVE) softmax_last<D, NI>(Vl, fo, E0, rows, sc, first, count, lane, issue);
      else static_for<NI>([&](auto IC) { issue(IC); });
    } else if constexpr (LIVE) {
      softmax_last<D, 0>(Vl, fo, E0, rows, sc, first, count, lane, issue);
    }
  }
};

// ---------------------------------------------------------------------------
// Phase L operand tiles and the order in which they stream through the four
// LDS tile buffers.  Tile kinds:
//   W1 tile j : W1 rows [64j, 64j+64), rows of 2D bytes (contiguous in memory)
//   W2 tile pb: W2 rows [32pb, 32pb+32); tile rows 0..31 hold their first k-half
//               (2D bytes), tile rows 32..63 the second
//   S tile pp : S_t^T columns [64pp, 64pp+64) of all D rows, rows of 128 bytes
// A step of the hidden layer needs its W1 tile landed (at most `younger` tiles issued after it may
// still be in flight) and, after its barrier, issues at most one further tile into a buffer whose last
// readers have passed that barrier.
// ---------------------------------------------------------------------------
enum { kNone = -1, kW1 = 0, kW2 = 1, kS = 2 };
struct LinStep {
  int younger;          // tiles that may still be in flight when the step starts
  int buf_w;            // buffer read by the step
  int kind, idx, buf;   // tile issued after the step's barrier
};

// The first requests (pro) and the steps of the hidden layer, a W1 tile each; then W2 of feature block p lies in w_buf(p),
// S of pair p of blocks in s_buf(p).
template <int D>
struct LinSched;
template <>
struct LinSched<128> {
  static constexpr int NPRO = 4;
  static constexpr LinStep pro(int i) { return LinStep{0, 0, kW1, i, i}; }
  static constexpr LinStep step(int st) {
    switch (st) {
      case 0: return LinStep{3, 0, kNone, 0, 0};
      case 1: return LinStep{2, 1, kS, 0, 0};
      case 2: return LinStep{2, 2, kW2, 0, 1};
      default: return LinStep{2, 3, kW2, 1, 2};
    }
  }
  static constexpr int w_buf(int p) { return 1 + (p & 1); }
  static constexpr int s_buf(int p) { return p & 1 ? 3 : 0; }
};
template <>
struct LinSched<64> {
  static constexpr int NPRO = 4;
  static constexpr LinStep pro(int i) {
    switch (i) {
      case 0: return LinStep{0, 0, kW1, 0, 0};
      case 1: return LinStep{0, 0, kW1, 1, 1};
      case 2: return LinStep{0, 0, kS, 0, 2};
      default: return LinStep{0, 0, kW2, 0, 3};
    }
  }
  static constexpr LinStep step(int st) { return st == 0 ? LinStep{3, 0, kNone, 0, 0} : LinStep{2, 1, kW2, 1, 0}; }
  static constexpr int w_buf(int p) { return p & 1 ? 0 : 3; }
  static constexpr int s_buf(int p) { return p & 1 ? 1 : 2; }
};

// Requests of phase L tiles by NW waves (kinds as above), one per-lane offset for all blocks a wave
// moves: W1 and S rows are contiguous or evenly strided, a W2 tile is two halves of 32 rows.
template <int D, int NW>
struct LinTiles {
  static constexpr int TB = 64 * D * 2;
  static constexpr int LPT = TB / (1024 * NW);   // direct loads per wave per tile
  static constexpr int CPR = 2 * D / 16, RPB = 1024 / (2 * D);
  u32x4 W1, W2, S;
  uint32_t lds;
  int wave, lane;

  __device__ __forceinline__ void issue(int kind, int idx, int buf) const {
#pragma unroll
    for (int n = 0; n < LPT; ++n) load(kind, idx, buf, n);
  }
  __device__ __forceinline__ void load(int kind, int idx, int buf, int n) const {
    const int jr = lane / CPR, cw = ((lane % CPR) ^ swz<2 * D>(wave * RPB + jr)) << 4;
    const int js = lane >> 3, cs = ((lane & 7) ^ swz<128>(wave * 8 + js)) << 4;
    const int blk = wave + NW * n, R = blk * RPB;
    const uint32_t dst = __builtin_amdgcn_readfirstlane(lds + buf * TB + blk * 1024);
    // (scalar also where the compiler has lost sight of that, in a branch for instance)
    auto uniform = [](int x) { return __builtin_amdgcn_readfirstlane(x); };
    if (kind == kW1)
      direct_load_16(W1, jr * (2 * D) + cw, uniform(idx * TB + blk * 1024), dst);
    else if (kind == kW2)
      direct_load_16(W2, jr * (4 * D) + cw, uniform(idx * 32 * (4 * D) + (R & 31) * (4 * D) + (R >> 5) * (2 * D)), dst);
    else
      direct_load_16(S, js * (4 * D) + cs, uniform(idx * 128 + blk * 8 * (4 * D)), dst);
  }
};

// The 32 rows of a W1 / W2 block are read in "quad-swapped" order (lane r takes block row sigma(r),
// sigma exchanging bits 2 and 3 of r), so that the accumulator of one product is, register for
// register, the B operand of the next one in natural k order and no operand needs a permuted copy
// in memory.  Accumulator register 4i+j of lane half g is block row 8i+4g+j, which after the row
// permutation is unit 16(i>>1) + 8g + 4(i&1) + j of the block.
template <int D>
__device__ __forceinline__ int lin_row_base(int lane) {   // k-step ks of the lane's row at ^ 32 ks
  const int r = lane & 31;
  return tile_off<2 * D>((r & 0x13) | ((r & 4) << 1) | ((r & 8) >> 1), 8 * (lane >> 5));
}
__device__ __forceinline__ void lin_vector(const float* v, int g, f32x16& x) {   // 32 units in accumulator order
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const f32x4 q = *reinterpret_cast<const f32x4*>(v + 16 * (i >> 1) + 8 * g + 4 * (i & 1));
#pragma unroll
    for (int j = 0; j < 4; ++j) x[4 * i + j] = q[j];
  }
}

// U^T = relu(W1 Q^T + b1) of NB blocks of 32 hidden units: Ub[2 nb], Ub[2 nb + 1] as B operands.  Fragments
// are read kAhead products ahead, a block is rectified under the products of the next one.  The second half of
// the blocks lies GAP bytes further on.  `issue(i)`, i < NI, requests tiles, one load behind every other product.
template <int D, int NB, int GAP, int NI, typename Issue>
__device__ __forceinline__ void lin_hidden(const char* Ws, int wbase, const float* bias, int g,
                                           const bf16x8 (&Qr)[D / 16], bf16x8* Ub, Issue issue) {
  constexpr int KS = D / 16, NM = NB * KS;
  static_assert(2 * NI <= NM, "the loads fit");
  f32x16 acc[2];
  bf16x8 fr[kAhead];
  auto fetch = [&](auto MC) {
    constexpr int m = decltype(MC)::value;
    if constexpr (m < NM) {
      if constexpr (m % KS == 0) lin_vector(bias + 32 * (m / KS), g, acc[(m / KS) & 1]);
      fr[m % kAhead] = *reinterpret_cast<const bf16x8*>(Ws + (wbase ^ (32 * (m % KS))) + (m / KS) * (32 * 2 * D) +
                                                        (m / KS >= NB / 2 ? GAP : 0));
    }
  };
  auto finish = [&](int nb, int half) {   // one of the two operands of block nb
    f32x16& x = acc[nb & 1];
#pragma unroll
    for (int e = 8 * half; e < 8 * half + 8; ++e) x[e] = fmaxf(x[e], 0.f);
    Ub[2 * nb + half] = acc_to_operand(x, half);
  };
  asm volatile("" : "+v"(wbase));
  static_for<kAhead>([&](auto MC) { fetch(MC); });
  static_for<NM>([&](auto MC) {
    constexpr int m = decltype(MC)::value, nb = m / KS;
    acc[nb & 1] = mfma(fr[m % kAhead], Qr[m % KS], acc[nb & 1]);
    // before the fetch that refills the other accumulator (bias of the next block)
    if constexpr (nb > 0 && m % KS == (KS > kAhead ? 1 : 0)) finish(nb - 1, 0);
    if constexpr (nb > 0 && m % KS == (KS > kAhead ? 2 : 0)) finish(nb - 1, 1);
    fetch(std::integral_constant<int, m + kAhead>{});
    if constexpr (m % 2 == 1 && m / 2 < NI) issue(std::integral_constant<int, m / 2>{});
    __builtin_amdgcn_sched_barrier(0);
  });
  finish(NB - 1, 0);
  finish(NB - 1, 1);
}

// NB feature blocks of a wave as one stream of products: psi of block 0, then psi of p + 1 and O += S^T phi of p in turn.
// phi of a block lies under the psi of the next one (of the last: under the read-out of the one before it), and operands
// are read kAhead products ahead, across the blocks.
template <int D, int NB>
struct LinStream {
  static constexpr int KS = D / 16, DB = D / 32, NW = 2 * KS, NS = 2 * DB, BL = NW + NS, NM = NB * BL;
  bool psi;
  int p, n;   // product n of block p
  static constexpr LinStream at(int m) {
    if (m < NW) return LinStream{true, 0, m};
    const int q = (m - NW) / BL, n = (m - NW) % BL;
    return q == NB - 1 ? LinStream{false, q, n} : n < NW ? LinStream{true, q + 1, n} : LinStream{false, q, n - NW};
  }
  static constexpr int psi_at(int p) { return p == 0 ? 0 : NW + (p - 1) * BL; }
  static constexpr int s_at(int p) { return NW + p * BL + (p == NB - 1 ? 0 : NW); }
  static constexpr int phi_at(int p, int i) {   // the slot of pair i of phi of block p
    return p < NB - 1 ? psi_at(p + 1) + 2 + i * (NW - 4) / 8 : s_at(NB - 2) + 1 + i * (NS - 1) / 8;
  }
  // The other way round, what stands in slot m.  As functions: with an `if constexpr` per slot, block and pair this file took
  // 131 s to compile, now 34, to the same instructions.
  struct Part {
    int p, first, n;   // elements first .. first + n - 1 of block p
  };
  static constexpr Part phi_in(int m) {   // pairs of phi
    Part x{0, 0, 0};
    for (int p = 0; p < NB; ++p)
      for (int i = 7; i >= 0; --i)
        if (phi_at(p, i) == m) x = Part{p, i, x.n + 1};
    return x;
  }
  static constexpr Part quads_in(int m) {   // the four features that pairs 2q and 2q + 1 need, a slot ahead of them
    Part x{0, 0, 0};
    for (int p = 0; p < NB; ++p)
      for (int q = 3; q >= 0; --q)
        if (phi_at(p, 2 * q) == m + 1) x = Part{p, q, x.n + 1};
    return x;
  }
  static constexpr int bias_in(int m) {   // the block whose bias is read, 0: none
    int x = 0;
    for (int p = 1; p < NB; ++p)
      if (psi_at(p) == m + 2) x = p;
    return x;
  }
  // kAhead products before the psi of block p: slot m lies n slots behind that of the last such p (p = 0: of none)
  static constexpr Part since_psi(int m) {
    Part x{0, 0, 0};
    for (int p = 1; p < NB; ++p)
      if (m + kAhead >= psi_at(p)) x = Part{p, 0, m + kAhead - psi_at(p)};
    return x;
  }
};
// Block p: W2 tile at tiles + w_off(p), S tile at s_off(p) (its upper 32 features if s_half(p)), bias and z at
// + VSTRIDE p.  `before(m)` stands in front of product m (barriers), `behind(m)` behind it (requests); with LIVE false they
// are all that is left.  Returns the wave's share of n^L, added to nL block by block.
template <int D, int NB, int VSTRIDE, bool LIVE, typename WOff, typename SOff, typename SHalf, typename Before, typename Behind>
__device__ __forceinline__ float lin_stream(const char* tiles, int wk, int sk, const float* bias, const float* z, int g,
                                            float lin_scale, const bf16x8 (&Ub)[D / 8], f32x16 (&O)[D / 32], float nL,
                                            WOff w_off, SOff s_off, SHalf s_half, Before before, Behind behind) {
  using L = LinStream<D, NB>;
  constexpr int KS = L::KS, DB = L::DB;
  f32x16 ps[2];
  // z of four features and of the next four; at d = 64 pairs of three quads stand in one slot
  constexpr int ZR = D == 128 ? 2 : 4;
  f32x4 zq[ZR];
  uint32_t fb[2][8];
  float part[2];
  bf16x8 fr[kAhead];
  auto fetch = [&](auto MC) {
    constexpr int m = decltype(MC)::value;
    if constexpr (m < L::NM) {
      constexpr L t = L::at(m);
      if constexpr (t.psi)
        fr[m % kAhead] = *reinterpret_cast<const bf16x8*>(tiles + w_off(t.p) + (wk ^ (32 * (t.n % KS))) + t.n / KS * (32 * 2 * D));
      else
        fr[m % kAhead] = *reinterpret_cast<const bf16x8*>(tiles + s_off(t.p) + (sk ^ (64 * s_half(t.p)) ^ (32 * (t.n / DB))) +
                                                          t.n % DB * (32 * 128));
    }
  };
  auto phi = [&](auto PC, auto IC) {   // elements 2i, 2i+1
    constexpr int p = decltype(PC)::value, i = decltype(IC)::value;
    if constexpr (i == 0) part[p & 1] = 0.f;
    float x[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      // the read-out rounds phi to bf16 (MFMA operand); the normaliser takes it unrounded: the
      // 256 rounding errors of a row have random signs and relative size 2^-9, far below the
      // bar on n^L, and the rounding costs two instructions per feature
      x[j] = fmaxf(ps[p & 1][2 * i + j], 0.f);
      if (p >= NB / 2) x[j] = x[j] * x[j];
      x[j] = x[j] * lin_scale;
      part[p & 1] += x[j] * zq[(i >> 1) % ZR][2 * (i & 1) + j];
    }
    fb[p & 1][i] = pack_bf16(x[0], x[1]);
    if constexpr (i == 7) nL += part[p & 1];
  };
  if constexpr (LIVE) {
    lin_vector(bias, g, ps[0]);
    static_for<kAhead>([&](auto MC) { fetch(MC); });
  }
  static_for<L::NM>([&](auto MC) {
    constexpr int m = decltype(MC)::value;
    constexpr L t = L::at(m);
    if constexpr (t.n == 0) asm volatile("" : "+v"(wk), "+v"(sk));   // offsets of a block are not kept for the next
    before(MC);
    if constexpr (LIVE) {
      if constexpr (t.psi) {
        ps[t.p & 1] = mfma(fr[m % kAhead], Ub[t.n], ps[t.p & 1]);
      } else {
        constexpr int ks = t.n / DB, db = t.n % DB, b = t.p & 1;
        const u32x4 w = {fb[b][4 * ks], fb[b][4 * ks + 1], fb[b][4 * ks + 2], fb[b][4 * ks + 3]};
        O[db] = mfma(fr[m % kAhead], __builtin_bit_cast(bf16x8, w), O[db]);
      }
      fetch(std::integral_constant<int, m + kAhead>{});
    }
    behind(MC);
    if constexpr (LIVE) {
      constexpr int bias_p = L::bias_in(m);
      if constexpr (bias_p > 0) lin_vector(bias + VSTRIDE * bias_p, g, ps[bias_p & 1]);
      constexpr typename L::Part quads = L::quads_in(m), pairs = L::phi_in(m);
      static_for<quads.n>([&](auto QC) {   // features of accumulator registers 4q .. 4q + 3
        constexpr int q = quads.first + decltype(QC)::value;
        zq[q % ZR] = *reinterpret_cast<const f32x4*>(z + VSTRIDE * quads.p + 16 * (q >> 1) + 8 * g + 4 * (q & 1));
      });
      static_for<pairs.n>([&](auto IC) {
        phi(std::integral_constant<int, pairs.p>{}, std::integral_constant<int, pairs.first + decltype(IC)::value>{});
      });
    }
    __builtin_amdgcn_sched_barrier(0);
  });
  return nL;
}

template <int D, int ST>
struct LinStepC { static constexpr LinStep value = LinSched<D>::step(ST); };
template <int D, int I>
struct LinProC { static constexpr LinStep value = LinSched<D>::pro(I); };

// Which (batch*head, chunk of the window, query tile) this workgroup computes; false: none.
__device__ __forceinline__ bool attn_item(const AttnArgs& a, int& bh, int& tc, int& qt) {
  if (a.n_short == 0) {
    const int item = xcd_swizzle(blockIdx.x, a.items_per_xcd);
    if (item >= a.n_items) return false;
    // item = bh * bh_items + tc * qtiles + qt, qt fastest
    bh = item / a.bh_items;
    const int rest = item % a.bh_items;
    tc = rest / a.qtiles;
    qt = rest % a.qtiles;
  } else {
    // The window starts at chunk 0, whose items have no read-out phase and are the shortest:
    // every XCD runs its share of them last, so that the launch does not end on long items.
    const int xcd = blockIdx.x & 7, i = blockIdx.x >> 3;
    const int n_long = a.n_items - a.n_short;
    const int per_long = (n_long + 7) / 8, per_short = (a.n_short + 7) / 8;
    if (i < per_long) {
      const int li = xcd * per_long + i;
      if (li >= n_long) return false;
      const int per_bh = a.bh_items - a.qtiles;
      bh = li / per_bh;
      const int rest = li % per_bh;
      tc = 1 + rest / a.qtiles;
      qt = rest % a.qtiles;
    } else {
      const int si = xcd * per_short + (i - per_long);
      if (si >= a.n_short) return false;
      bh = si / a.qtiles;
      tc = 0;
      qt = si % a.qtiles;
    }
  }
  return true;
}

// Token ranges of chunk t.
__device__ __forceinline__ ChunkRange attn_range(const AttnArgs& a, int t) {
  ChunkRange cr;
  if (a.step_nq > 0) {  // streaming step: explicit ranges, state always read
    cr.q_lo = 0;
    cr.q_hi = a.step_nq;
    cr.s_lo = 0;
    cr.s_hi = a.step_nwin;
    cr.l_hi = 1;
  } else {
    cr = chunk_range(a.T, a.HW, a.chunk, a.overlap, t);
    if (a.all_linear) cr.l_hi = 1;
  }
  return cr;
}

// second bound: waves per SIMD that the register budget is sized for
template <int D>
__global__ void __launch_bounds__(64 * kAttnNW, D == 64 ? 3 : 2)
attn_kernel(AttnArgs a) {
  using C = AttnShape<D>;
  constexpr int HID = C::HID, DP = C::DP, KS = C::KS, DB = C::DB;
  constexpr int TB = C::TILE_BYTES;
  // four tile buffers; phase S: K tiles in 0/1, V tiles in 2/3
  __shared__ __attribute__((aligned(1024))) char tiles[4 * TB];
  // the queries on their way into registers (d = 128: half of them, the others in the V buffer of tile 1, so that two
  // workgroups have 80 KB each); then the per-head vectors of phase L
  constexpr int QB = 32 * 2 * D;   // a wave's queries
  __shared__ __attribute__((aligned(1024))) char spare[kAttnNW * QB - (D == 128 ? TB : 0)];
  static_assert(sizeof(spare) >= (HID + 2 * DP) * sizeof(float), "the vectors fit");
  float* const sb1 = reinterpret_cast<float*>(spare);
  float* const sb2 = sb1 + HID;
  float* const sz = sb2 + DP;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform for the compiler too
  const int g = lane >> 5;
  const int r = lane & 31;

  // ---- which work item -------------------------------------------------
  if (!((a.xcd_mask >> (blockIdx.x & 7)) & 1u)) return;   // measurement hook; all bits set normally
  int qt, tc, bh;
  if (!attn_item(a, bh, tc, qt)) return;
  const int t = a.chunk0 + tc;
  const int h = bh % a.H;
  const ChunkRange cr = attn_range(a, t);
  const int64_t q0 = cr.q_lo + (int64_t)qt * kQueryTile;
  if (q0 >= cr.q_hi) return;   // never with the item counts of the host layer; without it the code before
                               // the first loads is ordered worse (24 heads x 11 chunks of 63 tokens
                               // 47.0 us a call, 45.1 with it)
  const int64_t N = (int64_t)a.T * a.HW;  // rows per (b, h) of the debug outputs
  const bf16_t* Qg = a.q + (int64_t)bh * a.q_bh_stride;
  const bf16_t* Kg = a.k + (int64_t)bh * a.kv_bh_stride;
  const bf16_t* Vg = a.v + (int64_t)bh * a.kv_bh_stride;
  bf16_t* Og = a.out + (int64_t)bh * a.q_bh_stride;
  const bool has_linear = cr.l_hi > 0;

  // ---- queries of this wave, held as B operands ---------------------------
  const int64_t qw0 = q0 + wave * 32;
  const int64_t row = qw0 + r;   // this lane's query
  // a wave whose 32 queries all lie beyond the chunk (last query tile) still moves its
  // share of every tile and meets every barrier, but computes nothing
  const bool wave_live = qw0 < cr.q_hi;
  // They come by way of a block of LDS of the wave's own, whole rows to an instruction.  As operands, 32 bytes of each of 32
  // rows to one, one layer at 480p took 505.8 us, now 503.7; 720p 1,949 and 1,939.5, 24 heads of 64 at 480p 476.7 and 474.2.
  bf16x8 Qr[KS];
  char* const q_block = D == 64 ? spare + wave * QB : wave < 2 ? tiles + 3 * TB + wave * QB : spare + (wave - 2) * QB;
  if (wave_live)
    tile_load_asm<2 * D, QB, 1>(make_rsrc_words(Qg + qw0 * D), 0, __builtin_amdgcn_readfirstlane(lds_address(q_block)), 0, lane,
                                (int)(cr.q_hi - qw0 < 32 ? cr.q_hi - qw0 : 32));
  SoftmaxRows<D> rows;
#pragma unroll
  for (int db = 0; db < DB; ++db) rows.O[db] = f32x16{};
  rows.ref = kLowest;
  rows.max = -INFINITY;
  rows.sum = 0.f;

  // =========================== phase S =====================================
  {
    const int n_keys = (int)(cr.s_hi - cr.s_lo);
    const SoftmaxTiles<D> st{make_rsrc_words(Kg + cr.s_lo * D), make_rsrc_words(Vg + cr.s_lo * D), lds_address(tiles),
                             tiles, RangeTiles<2 * D, 4>(n_keys, wave, lane), 0, 1, (n_keys + 63) / 64, lane};
    st.request();
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * SoftmaxTiles<D>::LPT) : "memory");   // the queries; K and V are younger
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) Qr[ks] = staged_fragment<2 * D>(q_block, lane, ks);
    wait_loads_and_barrier<0>();
    // per-head vectors of phase L, 64 values to an instruction (the tile loop waits for them, long before phase L, whose
    // counted waits must see tile loads only)
    if (has_linear) {
      const float* const zt = a.state_z + ((int64_t)bh * a.state_slots + tc) * DP;
      for (int i = wave; i < 3 * (DP / 64); i += kAttnNW) {
        const int which = i / (DP / 64), part = i % (DP / 64);
        const float* const src = which == 0 ? a.b1_q + (int64_t)h * HID : which == 1 ? a.b2_q + (int64_t)h * DP : zt;
        direct_load_4(make_rsrc_words(src), 4 * lane, 256 * part,
                      __builtin_amdgcn_readfirstlane(lds_address(spare) + 256 * i));
      }
    }
    auto none = [](auto) {};
    if (wave_live) st.template run<true, false, 0>(Qr, rows, a.scale_log2e, false, none);
    else st.template run<false, false, 0>(Qr, rows, a.scale_log2e, false, none);
    lds_barrier();   // all K/V tiles are dead
  }

  // =========================== phase L: first tiles =========================
  using SCH = LinSched<D>;
  const LinTiles<D, kAttnNW> lt{make_rsrc_words(a.w1_q + (int64_t)h * HID * D), make_rsrc_words(a.w2_q + (int64_t)h * DP * HID),
                                make_rsrc_words(a.state_s + ((int64_t)bh * a.state_slots + tc) * (int64_t)D * DP),
                                lds_address(tiles), wave, lane};
  auto issue = [&](auto SD) {   // the tile that a step (or the prologue) issues
    constexpr LinStep sd = decltype(SD)::value;
    if constexpr (sd.kind != kNone) lt.issue(sd.kind, sd.idx, sd.buf);
  };
  // complete the softmax normaliser across the two lane halves
  // All sums are relative to 2^-ref; the components are reported relative to the
  // true maximum: dscale = 2^(ref - max) <= 1.
  const float nS = half_swap_sum(rows.sum);
  const float dscale = __builtin_amdgcn_exp2f(rows.ref - rows.max);

  // debug: softmax components
  if (a.dbg_m || a.dbg_nS || a.dbg_aS) {
    if (row < cr.q_hi) {
      const int64_t o = (int64_t)bh * N + row;
      if (g == 0) {
        if (a.dbg_m) a.dbg_m[o] = rows.max * 0.6931471805599453f;  // back from base 2
        if (a.dbg_nS) a.dbg_nS[o] = nS * dscale;
      }
      if (a.dbg_aS) {
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            f32x4 x = {rows.O[db][4 * i], rows.O[db][4 * i + 1], rows.O[db][4 * i + 2], rows.O[db][4 * i + 3]};
            *reinterpret_cast<f32x4*>(a.dbg_aS + o * D + 32 * db + 8 * i + 4 * g) = x * dscale;
          }
      }
    }
    // the counted waits of phase L must see tile loads only
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  }

  // =========================== phase L =====================================
  float nL = 0.f;
  if (has_linear) {
    static_for<SCH::NPRO>([&](auto I) { issue(LinProC<D, decltype(I)::value>{}); });
    constexpr int NW1 = HID / 64, NPB = DP / 32;
    // The softmax sums are relative to 2^-ref: with c_i = row maximum (Eq. 6, 8) the
    // linear terms weigh 2^(max - ref) beside them, with c = 0 they weigh 2^-ref.
    const float lin_scale = __builtin_amdgcn_exp2f((a.stab_mode == 1 ? 0.f : rows.max) - rows.ref);
    const int wbase = lin_row_base<D>(lane), sbase = tile_off<128>(r, 8 * g);
    bf16x8 Ub[HID / 16];  // U^T = relu(W1 Q^T + b1) as B operands, natural k order
    static_for<NW1>([&](auto ST) {
      constexpr int st = decltype(ST)::value;
      constexpr LinStep sd = LinStepC<D, st>::value;
      wait_loads_and_barrier<sd.younger * LinTiles<D, kAttnNW>::LPT>();
      issue(LinStepC<D, st>{});
      if (!wave_live) return;  // this step of this wave only (the lambda is one step)
      lin_hidden<D, 2, 0, 0>(tiles + sd.buf_w * TB, wbase, sb1 + 64 * st, g, Qr, Ub + 4 * st, [](auto) {});
    });
    // The feature blocks, W2 of even and odd blocks and S of even and odd pairs of blocks in two buffers each.  A barrier stands
    // kAhead products before the end of psi 0 and of the read-outs: W2 of the block after the next has landed there, its
    // predecessor's buffer is free for W2 of the one behind that, and after an odd block that of its S.
    // As one stream because phi and the first fragments of a block stood between its products and the next block's: block by
    // block one layer at 480p took 498.1 us, now 489.8; 720p 1,857 and 1,838, 101 frames of 600 tokens 1,193 and 1,179, two
    // 480p layers with three-frame chunks 1,968 and 1,955, 24 heads of 64 at 480p 472.7 and 471.1; the same results bit for bit.
    using L = LinStream<D, NPB>;
    using T = LinTiles<D, kAttnNW>;
    auto stream = [&](auto LIVEC) {
      auto before = [&](auto MC) {
        constexpr typename L::Part at = L::since_psi(decltype(MC)::value);
        if constexpr (at.p > 0 && at.n == 0) wait_loads_and_barrier<0>();
      };
      auto behind = [&](auto MC) {
        constexpr int m = decltype(MC)::value;
        if constexpr (m % 2 == 1 && m / 2 < T::LPT) lt.load(kS, 1, SCH::s_buf(1), m / 2);
        // behind the barrier before psi p: W2 of block p + 1, and with an odd p S of its pair
        constexpr typename L::Part at = L::since_psi(m);
        constexpr int p = at.p, i = at.n - 1;
        if constexpr (p > 0 && p + 1 < NPB && i >= 0 && i / 2 < T::LPT) {
          if constexpr (i % 2 == 0) lt.load(kW2, p + 1, SCH::w_buf(p + 1), i / 2);
          else if constexpr (p > 2 && p % 2 == 1) lt.load(kS, (p + 1) / 2, SCH::s_buf((p + 1) / 2), i / 2);
        }
      };
      nL = lin_stream<D, NPB, 32, decltype(LIVEC)::value>(
          tiles, wbase, sbase, sb2, sz, g, lin_scale, Ub, rows.O, nL, [](int p) { return SCH::w_buf(p) * TB; },
          [](int p) { return SCH::s_buf(p / 2) * TB; }, [](int p) { return p & 1; }, before, behind);
    };
    wait_loads_and_barrier<0>();   // W2 of blocks 0 and 1 and the first S; W1 is dead
    if (wave_live) stream(std::true_type{});
    else stream(std::false_type{});
    nL = half_swap_sum(nL);
  }

  // =========================== merge (Eq. 5) ================================
  // The rows leave by way of LDS, whole lines to an instruction: two buffers that the last step does not read hold a
  // block for each wave.  In the accumulator's pieces (8 bytes a lane, 16 of each of 32 rows per instruction) one layer
  // at 480p took 531.1 us, now 521.6; 720p 1,981 and 1,965, 24 heads of 64 at 480p 497.5 and 491.6; with the split
  // kernel 2 x 3 heads of 333-token frames 42.5 and 41.5, 21 streaming steps at 480p 1,197 and 1,176.
  if (!wave_live) return;
  const bool valid = row < cr.q_hi;
  const int64_t o = (int64_t)bh * N + row;
  if (valid && g == 0 && a.dbg_nL) a.dbg_nL[o] = nL * dscale;
  const float inv = 1.0f / (nS + nL);
  char* const rows_out = tiles + (D == 128 ? 0 : 2) * TB + wave * (32 * 2 * D);
#pragma unroll
  for (int db = 0; db < DB; ++db) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int col = 32 * db + 8 * i + 4 * g;
      if (valid && a.dbg_aL) {
        f32x4 as = {0.f, 0.f, 0.f, 0.f};
        if (a.dbg_aS) as = *reinterpret_cast<const f32x4*>(a.dbg_aS + o * D + col);
        f32x4 x;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          // the product is rounded as it was when a^S was stored (no fused multiply-subtract),
          // so an empty linear set reports exactly zero
          float t = rows.O[db][4 * i + j] * dscale;
          asm volatile("" : "+v"(t));
          x[j] = t - as[j];
        }
        *reinterpret_cast<f32x4*>(a.dbg_aL + o * D + col) = x;
      }
      u32x2 pk;
      pk[0] = pack_bf16(rows.O[db][4 * i] * inv, rows.O[db][4 * i + 1] * inv);
      pk[1] = pack_bf16(rows.O[db][4 * i + 2] * inv, rows.O[db][4 * i + 3] * inv);
      *reinterpret_cast<u32x2*>(rows_out + tile_off<2 * D>(r, col)) = pk;
    }
  }
#pragma unroll
  for (int n = 0; n < D / 16; ++n) {
    constexpr int CPR = D / 8;   // chunks of 16 bytes per row
    const int rw = n * (64 / CPR) + lane / CPR, c = lane % CPR;
    const u32x4 x = *reinterpret_cast<const u32x4*>(rows_out + tile_off<2 * D>(rw, 8 * c));
    if (qw0 + rw < cr.q_hi) store_through(Og + q0 * D, (32 * wave + rw) * (2 * D) + 16 * c, x);
  }
}

// ---------------------------------------------------------------------------
// The same result for launches too small to fill the chip: a workgroup of eight waves owns 128
// queries, and two groups of four waves share the work of each query block.  Group kg takes the
// key tiles with index = kg mod 2 in phase S and the feature blocks with index = kg mod 2 in
// phase L; the two numerators and normalisers are brought to one reference after phase S and
// added through LDS at the end.
//
// What bounds it: the same loop as attn_kernel, but a launch of at most 256 attn_kernel workgroups
// leaves one wave on a SIMD, whose instruction stream alone does not fill it.  Here every SIMD that
// has work has two waves, each with half of the tiles, at the price of the meeting and of a lower
// clock.  Streaming step at the 480p shape with T_o = 1, 156 items: 47 us from the first workgroup's start, 34 of them
// for the tiles, 2.9 before the first and 9 after the last, 2.4 - 2.7 of those for each of the hidden layer (128 products
// on a SIMD) and the merge's two round trips, 4.2 for the features; with phase L's first tiles requested
// behind the last key tile and its blocks one after the other 50.1, 10.9 behind the tiles.
// 144 KB of tile buffers (K and V of two tiles per group): one workgroup per CU, which is why
// attn_kernel stays the better one as soon as its own launch fills the chip (attn_splits).
// ---------------------------------------------------------------------------
// STEP (streaming step): explicit ranges; S and z are the caller's, in its layout and precision, so that no
// launch has to prepare them (a kernel that wrote S as the bf16 operand that phase L reads stood
// before this one: 4 of 64 us per step at the 480p shape); further workgroups absorb rows.  A
// thread carries a block of 4 features x 4 columns of S through registers, rounded as that kernel did.
template <int D, bool STEP>
__global__ void __launch_bounds__(512, 2)
attn_split_kernel(AttnArgs a, StateArgs sa, int attn_blocks) {
  using C = AttnShape<D>;
  constexpr int HID = C::HID, DP = C::DP, KS = C::KS, DB = C::DB;
  constexpr int TB = C::TILE_BYTES;
  constexpr int GB = 4 * TB;   // tile buffers of one group: K 0/1, V 2/3; of group 1: K 4/5, V 6/7
  constexpr int NBUF = D == 128 ? 9 : 8;   // one more for the first S tile where W1 takes all K buffers
  using SL = StateLds<D>;
  __shared__ __attribute__((aligned(1024))) char tiles[!STEP || NBUF * TB > SL::XV + SL::US ? NBUF * TB : SL::XV + SL::US];
  __shared__ __attribute__((aligned(256))) float sb1[HID];
  __shared__ __attribute__((aligned(16))) float sb2[DP];
  __shared__ __attribute__((aligned(16))) float sz[DP];
  __shared__ float xref[2][kQueryTile], xmax[2][kQueryTile], xsum[2][kQueryTile], xlin[2][kQueryTile];

  // streaming step: the workgroups beyond the attention items absorb the tokens that leave the
  // window (pieces of the chunk-state increment) on CUs that the attention items leave free
  if constexpr (STEP) {
    if ((int)blockIdx.x >= attn_blocks) {
      constexpr int NW = D / 16;   // waves of the chunk-state body; the others are done
      if (__builtin_amdgcn_readfirstlane(threadIdx.x >> 6) < NW)
        state_body<D, NW>(sa, blockIdx.x - attn_blocks, tiles, tiles + SL::XV, sb1);
      return;
    }
  }

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kg = wave >> 2, qg = wave & 3;   // key group, query block
  const int g = lane >> 5;
  const int r = lane & 31;

  if (!((a.xcd_mask >> (blockIdx.x & 7)) & 1u)) return;   // measurement hook; all bits set normally
  int qt, tc, bh;
  if (!attn_item(a, bh, tc, qt)) return;
  const int h = bh % a.H;
  const ChunkRange cr = attn_range(a, a.chunk0 + tc);
  const int64_t q0 = cr.q_lo + (int64_t)qt * kQueryTile;
  if (q0 >= cr.q_hi) return;   // as in attn_kernel
  const int64_t N = (int64_t)a.T * a.HW;
  const bf16_t* Qg = a.q + (int64_t)bh * a.q_bh_stride;
  const bf16_t* Kg = a.k + (int64_t)bh * a.kv_bh_stride;
  const bf16_t* Vg = a.v + (int64_t)bh * a.kv_bh_stride;
  bf16_t* Og = a.out + (int64_t)bh * a.q_bh_stride;
  const bool has_linear = cr.l_hi > 0;

  const int64_t row = q0 + 32 * qg + r;            // this lane's query
  const bool wave_live = q0 + 32 * qg < cr.q_hi;   // else: moves tiles and meets barriers only
  SoftmaxRows<D> rows;
#pragma unroll
  for (int db = 0; db < DB; ++db) rows.O[db] = f32x16{};
  rows.ref = kLowest;
  rows.max = -INFINITY;
  rows.sum = 0.f;

  const bool dbg_soft = a.dbg_m || a.dbg_nS || a.dbg_aS;
  constexpr int NW1 = HID / 64, NP = DP / 64;
  const LinTiles<D, 8> lt{make_rsrc_words(a.w1_q + (int64_t)h * HID * D), make_rsrc_words(a.w2_q + (int64_t)h * DP * HID),
                          make_rsrc_words(STEP ? a.w1_q : a.state_s + ((int64_t)bh * a.state_slots + tc) * (int64_t)D * DP),
                          lds_address(tiles), wave, lane};
  constexpr int L8 = LinTiles<D, 8>::LPT;
  // Where the tiles of phase L lie.  W1 in the K buffers; set p is the W2 tiles of feature blocks 2p and 2p + 1 (one
  // per group) and the S tile of their 64 features.
  static_assert(NW1 <= 4 && NP <= 4, "schedule of the buffers");
  constexpr int W1GAP = NW1 > 2 ? 2 * TB : 0;
  auto w1_buf = [](int i) { return i < 2 ? i : i + 2; };
  auto w2_buf = [](int p) { return p == 0 || p == 3 ? 2 : p == 1 ? 6 : 4; };
  auto s_buf = [](int p) { return D == 64 ? 4 + p : p == 0 ? 8 : p == 3 ? 6 : p - 1; };
  // load i of W1, and of the tiles of phase L behind it: W2 of sets 0 and 1 and S of what has a free buffer
  // (under the hidden layer), W2 of 2 and S of 1 and 2 (under the first block), W2 of 3 and S of 3 (under the second)
  constexpr int N1 = NW1 * L8;
  auto load_w1 = [&](auto IC) {
    constexpr int i = decltype(IC)::value;
    lt.load(kW1, i / L8, w1_buf(i / L8), i % L8);
  };
  auto load_w2 = [&](int first, int i) {
    const int tile = first + i / L8;
    lt.load(kW2, tile, w2_buf(tile / 2) + tile % 2, i % L8);
  };
  auto load_s = [&](int first, int i) { lt.load(kS, first + i / L8, s_buf(first + i / L8), i % L8); };
  constexpr int NS0 = STEP ? 0 : D == 64 ? 2 : 1;   // S tiles under the hidden layer
  constexpr int N2 = (4 + NS0) * L8;
  auto load_first = [&](auto IC) {
    constexpr int i = decltype(IC)::value;
    if constexpr (i < 4 * L8) load_w2(0, i);
    else load_s(0, i - 4 * L8);
  };
  constexpr int N3 = NP > 2 ? (STEP ? 2 : 4) * L8 : 0;
  auto load_second = [&](auto IC) {
    constexpr int i = decltype(IC)::value;
    if constexpr (i < 2 * L8) load_w2(4, i);
    else load_s(1, i - 2 * L8);
  };
  constexpr int N4 = NP > 2 ? (STEP ? 2 : 3) * L8 : 0;
  auto load_third = [&](auto IC) {
    constexpr int i = decltype(IC)::value;
    if constexpr (i < 2 * L8) load_w2(6, i);
    else load_s(3, i - 2 * L8);
  };
  // STEP: features 64p + 4 s_f .. of columns 4 s_d .. of S are requested into registers ahead of the S tile
  // (64 features, i.e. 128 bytes, per column) that they go to, rounded as the copy of the state was
  const int s_f = tid / (D / 4), s_d = tid % (D / 4);
  const bool s_mover = 4 * D == 512 || tid < 4 * D;   // whole waves
  f32x4 sreg[4];
  auto request_s = [&](int p) {
    if (STEP && s_mover) {
      const float* const src = a.step_S + ((int64_t)bh * DP + 64 * p) * D;
      const uint32_t off = 4 * s_f * D + 4 * s_d;
#pragma unroll
      for (int i = 0; i < 4; ++i) sreg[i] = *reinterpret_cast<const f32x4_u*>(src + i * D + off);
    }
  };
  auto place_s = [&](int p) {
    if (STEP && s_mover) {
      char* const Ss = tiles + s_buf(p) * TB;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        u32x2 pk;
        pk[0] = pack_bf16(sreg[0][j], sreg[1][j]);
        pk[1] = pack_bf16(sreg[2][j], sreg[3][j]);
        *reinterpret_cast<u32x2*>(Ss + tile_off<128>(4 * s_d + j, 4 * s_f)) = pk;
      }
    }
  };

  // =========================== phase S =====================================
  bf16x8 Qr[KS];
  {
    const int n_keys = (int)(cr.s_hi - cr.s_lo), n_tiles = (n_keys + 63) / 64;
    const uint32_t lds = lds_address(tiles);
    const SoftmaxTiles<D> st{make_rsrc_words(Kg + cr.s_lo * D), make_rsrc_words(Vg + cr.s_lo * D),
                                (uint32_t)__builtin_amdgcn_readfirstlane(lds + kg * GB), tiles + kg * GB,
                                RangeTiles<2 * D, 4>(n_keys, qg, lane), kg, 2, (n_tiles + 1 - kg) / 2, lane};
    // The queries come through the V buffers of tile 1, whole rows to an instruction, once for both groups: read
    // from memory as operands (32 rows of 32 bytes an instruction, by both groups) they held up the tiles behind
    // them (K of tile 0 there 3.8 us after the workgroup's start, now 2.9).
    const u32x4 Qd = make_rsrc_words(Qg + q0 * D);
    const int q_rows = cr.q_hi - q0 < kQueryTile ? (int)(cr.q_hi - q0) : kQueryTile;
    tile_load_asm<2 * D, TB, 8>(Qd, 0, lds + 3 * TB, wave, lane, q_rows < 64 ? q_rows : 64);
    if (q_rows > 64) tile_load_asm<2 * D, TB, 8>(Qd, 64 * 2 * D, lds + 7 * TB, wave, lane, q_rows - 64);
    st.request();
    if (has_linear) {   // per-head vectors of phase L, 64 values to an instruction
      const float* const zt = STEP ? a.step_z + (int64_t)bh * DP : a.state_z + ((int64_t)bh * a.state_slots + tc) * DP;
      static_assert(HID == DP, "three vectors of one length");
      for (int i = wave; i < 3 * (DP / 64); i += 8) {
        const int which = i / (DP / 64), part = i % (DP / 64);
        const float* const src = which == 0 ? a.b1_q + (int64_t)h * HID : which == 1 ? a.b2_q + (int64_t)h * DP : zt;
        const uint32_t dst = lds_address(which == 0 ? sb1 : which == 1 ? sb2 : sz);
        direct_load_4(make_rsrc_words(src), 4 * lane, 256 * part, __builtin_amdgcn_readfirstlane(dst + 256 * part));
      }
    }
    // the queries and K of tile 0; with a second tile V and K of it are younger, and may be in flight
    if (st.n > 1) wait_loads_and_barrier<2 * SoftmaxTiles<D>::LPT>();
    else wait_loads_and_barrier<0>();
    if (wave_live) {
      const char* const Qs = tiles + (3 + 4 * (qg >> 1)) * TB + (qg & 1) * (32 * 2 * D);
      const FragBase fo = make_frag_base<D>(lane);
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) Qr[ks] = k_fragment<D>(Qs, fo, ks, 0);
    }
    // Group 1 may have a tile less than group 0, or none, and then meets its last barriers here.  Behind the last
    // one that group 0's tiles need all K buffers are free, and W1 goes there under the last tile.
    const int barriers = (n_tiles + 1) / 2 + 1;
    const bool ahead = has_linear && !dbg_soft;
    int met = 0;
    if (st.n > 0) {
      met = st.n + 1;
      const bool last = ahead && met == barriers;
      if (wave_live) st.template run<true, true, N1>(Qr, rows, a.scale_log2e, last, load_w1);
      else st.template run<false, true, N1>(Qr, rows, a.scale_log2e, last, load_w1);
    }
    if (met < barriers) {
      for (; met < barriers; ++met) wait_loads_and_barrier<0>();
      if (ahead) static_for<N1>(load_w1);
    }
    if (ahead) request_s(0);
    lds_barrier();   // the V buffers are free as well
  }

  // ---- one reference for both groups -------------------------------------------------
  {
    const float part = half_swap_sum(rows.sum);
    if (g == 0) {
      xref[kg][32 * qg + r] = rows.ref;
      xmax[kg][32 * qg + r] = rows.max;
      xsum[kg][32 * qg + r] = part;
    }
  }
  lds_barrier();
  float nS, dscale;
  {
    const float r0 = xref[0][32 * qg + r], r1 = xref[1][32 * qg + r];
    const float mref = fmaxf(r0, r1);
    rows.max = fmaxf(xmax[0][32 * qg + r], xmax[1][32 * qg + r]);
    nS = xsum[0][32 * qg + r] * __builtin_amdgcn_exp2f(r0 - mref) +
         xsum[1][32 * qg + r] * __builtin_amdgcn_exp2f(r1 - mref);
    const float f = __builtin_amdgcn_exp2f(rows.ref - mref);
    rows.ref = mref;
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int e = 0; e < 16; ++e) rows.O[db][e] *= f;
    dscale = __builtin_amdgcn_exp2f(rows.ref - rows.max);
  }
  // numerator registers 4i .. 4i+3 of feature block db, exchanged at 16 bytes per lane
  auto slot = [&](int q, int n) { return reinterpret_cast<f32x4*>(tiles + (q * (4 * DB) + n) * 1024 + lane * 16); };
  auto quad = [&](int db, int i) {
    f32x4 x = {rows.O[db][4 * i], rows.O[db][4 * i + 1], rows.O[db][4 * i + 2], rows.O[db][4 * i + 3]};
    return x;
  };
  if (dbg_soft) {   // component outputs: the two softmax parts are added for them alone
    if (kg == 1) {
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int i = 0; i < 4; ++i) *slot(qg, 4 * db + i) = quad(db, i);
    }
    lds_barrier();
    if (kg == 0 && row < cr.q_hi) {
      const int64_t o = (int64_t)bh * N + row;
      if (g == 0) {
        if (a.dbg_m) a.dbg_m[o] = rows.max * 0.6931471805599453f;   // back from base 2
        if (a.dbg_nS) a.dbg_nS[o] = nS * dscale;
      }
      if (a.dbg_aS) {
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
          for (int i = 0; i < 4; ++i)
            *reinterpret_cast<f32x4*>(a.dbg_aS + o * D + 32 * db + 8 * i + 4 * g) =
                (quad(db, i) + *slot(qg, 4 * db + i)) * dscale;
      }
    }
    // the parts have been read, a^S is in memory, and the counted waits of phase L see tile
    // loads only
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    if (has_linear) {
      static_for<N1>(load_w1);
      request_s(0);
    }
  }

  // =========================== phase L =====================================
  float nL = 0.f;
  if (has_linear) {
    const float lin_scale = __builtin_amdgcn_exp2f((a.stab_mode == 1 ? 0.f : rows.max) - rows.ref);
    const int wbase = lin_row_base<D>(lane), sbase = tile_off<128>(r, 8 * g);
    bf16x8 Ub[HID / 16];
    wait_loads_and_barrier<0>();   // W1 has landed
    if (wave_live) lin_hidden<D, HID / 32, W1GAP, N2>(tiles, wbase, sb1, g, Qr, Ub, load_first);
    else static_for<N2>(load_first);
    place_s(0);
    wait_loads_and_barrier<0>();   // sets 0 and 1; W1 is dead
    request_s(1);
    // The wave's feature blocks are 2p + kg, p = 0 .. NP-1.  Both waves of a SIMD are in the same phase here, so that
    // neither fills the other's gaps: block by block, each fragment read and each phi in the way of the products, it took
    // 5.0 us (streaming step 5.7), as one stream 3.3 (4.2).
    // Barriers stand where tiles have to have landed, kAhead products before their own.
    auto stream = [&](auto LIVEC) {
      using L = LinStream<D, NP>;
      auto before = [&](auto MC) {
        constexpr int m = decltype(MC)::value;
        constexpr typename L::Part at = L::since_psi(m);
        // before the psi of blocks 2 and 3, and before the last read-out, where everything but its S is dead
        constexpr int p = m + kAhead == L::s_at(NP - 1) ? NP - 1 : at.n == 0 ? at.p - 1 : 0;
        if constexpr (p >= 1) {
          place_s(p);
          wait_loads_and_barrier<0>();
          if constexpr (p + 1 < NP) request_s(p + 1);
        }
      };
      auto behind = [&](auto MC) {
        constexpr int m = decltype(MC)::value;
        if constexpr (m % 2 == 1 && m / 2 < N3) load_second(std::integral_constant<int, m / 2>{});
        constexpr int b1 = NP > 2 ? L::psi_at(2) - kAhead : 0, i4 = (m - b1 - 1) / 2;
        if constexpr (NP > 2 && m > b1 && (m - b1) % 2 == 1 && i4 < N4) load_third(std::integral_constant<int, i4>{});
      };
      nL = lin_stream<D, NP, 64, decltype(LIVEC)::value>(
          tiles, wbase + kg * TB, sbase ^ (kg * 64), sb2 + 32 * kg, sz + 32 * kg, g, lin_scale, Ub, rows.O, nL,
          [=](int p) { return w2_buf(p) * TB; }, [=](int p) { return s_buf(p) * TB; }, [](int) { return 0; }, before, behind);
    };
    if (wave_live) stream(std::true_type{});
    else stream(std::false_type{});
    nL = half_swap_sum(nL);
  }

  // =========================== merge (Eq. 5) ================================
  // each group hands the other half of its numerator over and finishes DB / 2 feature blocks (through buffers
  // 0 .. 3, dead since the barrier before the last read-out)
  if (g == 0) xlin[kg][32 * qg + r] = nL;
  auto finish = [&](auto GC) {
    constexpr int own = decltype(GC)::value, other = 1 - own;
#pragma unroll
    for (int n = 0; n < 2 * DB; ++n)
      *slot(qg, (2 * DB) * other + n) = quad((DB / 2) * other + (n >> 2), n & 3);
    lds_barrier();
    if (!wave_live) return;
    const bool valid = row < cr.q_hi;
    const float nLt = xlin[0][32 * qg + r] + xlin[1][32 * qg + r];
    const int64_t o = (int64_t)bh * N + row;
    if (valid && own == 0 && g == 0 && a.dbg_nL) a.dbg_nL[o] = nLt * dscale;
    const float inv = 1.0f / (nS + nLt);
    // the rows leave by way of the slots that this wave has read, as in attn_kernel
    f32x4 y[2 * DB];
#pragma unroll
    for (int n = 0; n < 2 * DB; ++n) y[n] = quad((DB / 2) * own + (n >> 2), n & 3) + *slot(qg, (2 * DB) * own + n);
    char* const rows_out = tiles + (qg * (4 * DB) + (2 * DB) * own) * 1024;
    constexpr int CPR = D / 16;                               // chunks of 16 bytes per half row
    auto place = [](int rw, int c) { return rw * D + ((c ^ ((D == 128 ? rw : rw >> 1) % CPR)) << 4); };
#pragma unroll
    for (int n = 0; n < 2 * DB; ++n) {
      const int db = (DB / 2) * own + (n >> 2), i = n & 3;
      const int col = 32 * db + 8 * i + 4 * g;
      if (valid && a.dbg_aL) {
        f32x4 as = {0.f, 0.f, 0.f, 0.f};
        if (a.dbg_aS) as = *reinterpret_cast<const f32x4*>(a.dbg_aS + o * D + col);
        f32x4 x;
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) {
          // rounded as when a^S was stored, so that an empty linear set reports exactly zero
          float t = y[n][jj] * dscale;
          asm volatile("" : "+v"(t));
          x[jj] = t - as[jj];
        }
        *reinterpret_cast<f32x4*>(a.dbg_aL + o * D + col) = x;
      }
      u32x2 pk;
      pk[0] = pack_bf16(y[n][0] * inv, y[n][1] * inv);
      pk[1] = pack_bf16(y[n][2] * inv, y[n][3] * inv);
      *reinterpret_cast<u32x2*>(rows_out + place(r, n) + 8 * g) = pk;   // chunk n of the half row
    }
    const int64_t q_w = q0 + 32 * qg;
#pragma unroll
    for (int n = 0; n < CPR / 2; ++n) {
      const int rw = n * (64 / CPR) + lane / CPR, c = lane % CPR;
      const u32x4 x = *reinterpret_cast<const u32x4*>(rows_out + place(rw, c));
      const int off = (32 * qg + rw) * (2 * D) + D * own + 16 * c;
      if (q_w + rw >= cr.q_hi) continue;
      // half a row is a whole line at d = 128 only.  Stored through at d = 64, 21 steps of 12 heads at 480p took 765 us instead
      // of 756, of 16 heads of 1,000-token frames 409.5 instead of 403; calls over a whole sequence even
      if constexpr (D == 128) store_through(Og + q0 * D, off, x);
      else *reinterpret_cast<u32x4*>(reinterpret_cast<char*>(Og + q0 * D) + off) = x;
    }
  };
  if (kg == 0) finish(std::integral_constant<int, 0>{});
  else finish(std::integral_constant<int, 1>{});
}

// The split kernel holds one workgroup per CU (144 KB of tile buffers), so it wins while its launch is a single
// round: at 256 items and fewer (not split against split, whole calls: d = 128 300 items of 540 keys 49.7 and 55.0 us,
// 405 of 1,100 72.4 and 70.0, 576 of 1,500 108.7 and 109.5; d = 64 260 of 1,600 29.2 and 34.2, 378 of 2,600 62.0 and
// 66.4, 720 of 1,500 60.5 and 67.6).  Below that the two groups' meeting has to be paid by the keys: d = 128 with a
// read-out 120 items of 192 keys 39.1 and 39.1 us, 24 of 256 34.1 and 32.8, 160 of 512 47.8 and 46.3, 225 of 600 48.1
// and 47.0, 192 of 1,000 52.2 and 50.3, 144 of 2,000 63.2 and 59.0; d = 64 160 of 448 25.7 and 25.9, 200 of 640 27.1
// and 26.5, 192 of 1,000 29.2 and 28.1.  Without a read-out at d = 128 48 of 512 14.6 and 14.5, 60 of 768 16.0 and
// 15.2, 80 of 1,024 19.1 and 17.7; at d = 64 70 of 896 14.3 and 14.5, 110 of 1,400 18.0 and 16.2.
// The lines lie where the two broke even before the split kernel's phase L was one stream (d = 128 with a read-out:
// where its smaller error began to cost little, 2.266e-3 instead of 2.297e-3 relative to fp64 at 4 heads of 333-token
// frames, T_o = 1: each group rounds its weights relative to a maximum of its own, whose weight of 1 is exact).  Time
// alone would put them at about 200, 600, 560 and 1,000 keys now, for 2 - 4 % of the calls between (at d = 64 without
// a read-out 10 %).  What the present ones keep: a row of fewer keys has the same bits in a launch of any number of items.
// From a line on its last bits depend on whether the launch has more than 256.
bool attn_splits(int64_t n_items, int64_t n_keys, int d, bool read_out) {
  return n_items <= 256 && n_keys >= (d == 128 ? (read_out ? 448 : 960) : read_out ? 960 : 1664);
}

int attn_query_tile(int) { return kQueryTile; }

const char* attn_kernel_name(int d) {
  static char name[2][48];
  char* n = name[d == 128 ? 0 : 1];
  snprintf(n, sizeof(name[0]), "attn_kernel<%d>", d == 128 ? 128 : 64);
  return n;
}

hipError_t launch_attn(const AttnArgs& a, const StateArgs* absorb, int d, bool split, hipStream_t stream) {
  const int grid = a.items_per_xcd * 8;
  if (split) {
    StateArgs s{};
    if (absorb) s = *absorb;
    const int blocks = grid + (absorb ? s.items_per_xcd * 8 : 0);
    const bool step = a.step_S != nullptr;
    auto kernel = d == 128 ? (step ? attn_split_kernel<128, true> : attn_split_kernel<128, false>)
                           : (step ? attn_split_kernel<64, true> : attn_split_kernel<64, false>);
    hipLaunchKernelGGL(kernel, dim3(blocks), dim3(512), 0, stream, a, s, grid);
  } else if (d == 128) {
    hipLaunchKernelGGL(attn_kernel<128>, dim3(grid), dim3(64 * kAttnNW), 0, stream, a);
  } else {
    hipLaunchKernelGGL(attn_kernel<64>, dim3(grid), dim3(64 * kAttnNW), 0, stream, a);
  }
  return hipGetLastError();
}

}  // namespace rehyat
