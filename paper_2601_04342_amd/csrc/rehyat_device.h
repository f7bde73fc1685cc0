// Device-side building blocks shared by the gfx950 kernels of the hybrid
// attention library: vector types, the bf16 MFMA wrapper with its operand
// layout, LDS tile staging and the chunk bookkeeping formulas.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>
#include <utility>

namespace rehyat {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4;
typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
typedef __attribute__((__vector_size__(2 * sizeof(float)))) float f32x2;
typedef f32x4 f32x4_u __attribute__((aligned(4)));   // in a caller's buffer aligned to single floats
typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4;
typedef __attribute__((__vector_size__(2 * sizeof(uint32_t)))) uint32_t u32x2;
typedef __attribute__((__vector_size__(4 * sizeof(short)))) short i16x4;

typedef uint16_t bf16_t;  // storage type of a bf16 value

constexpr int kWave = 64;

// compile-time loop: f(integral_constant<int, 0>) ... f(integral_constant<int, N-1>)
template <typename F, int... I>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for_impl(f, std::make_integer_sequence<int, N>{});
}

// ---------------------------------------------------------------------------
// Chunk bookkeeping (section 3.2 token layout; Eq. 12; Eq. 13).  The host
// entry point rehyat_chunk_plan and every kernel use this one function.
// ---------------------------------------------------------------------------
struct ChunkRange {
  int64_t q_lo, q_hi;  // query tokens of the chunk
  int64_t s_lo, s_hi;  // softmax window
  int64_t l_hi;        // causal linear set is [0, l_hi)
};

__host__ __device__ inline int num_chunks(int T, int chunk) {
  // 64-bit: chunk may be as large as INT_MAX ("one chunk covers everything")
  return (int)(((int64_t)T + chunk - 1) / chunk);
}

__host__ __device__ inline ChunkRange chunk_range(int T, int HW, int chunk, int overlap, int t) {
  ChunkRange r;
  int64_t f0 = (int64_t)t * chunk;
  int64_t f1 = f0 + chunk;
  if (f1 > T) f1 = T;
  r.q_lo = f0 * HW;
  r.q_hi = f1 * HW;
  int64_t s = r.q_lo - (int64_t)overlap * HW;
  r.s_lo = s < 0 ? 0 : s;
  r.s_hi = r.q_hi;
  r.l_hi = r.s_lo;
  return r;
}

// ---------------------------------------------------------------------------
// v_mfma_f32_32x32x16_bf16: D[32x32] += A[32x16] * B[16x32].
// Lane l = 32*g + r holds A[r][8g .. 8g+7] and B[8g .. 8g+7][r]; accumulator
// register 4*i + j of lane l holds D[8i + 4g + j][r].
// Because the contraction index may be permuted freely as long as A and B
// agree, an accumulator (rows 8i+4g+j in registers) converts in place into
// the B operand of a following product: registers 8s .. 8s+7 become the eight
// k-values of k-step s, which are rows 16s + {4g..4g+3, 8+4g..8+4g+3}.  The
// matching A operand is read from a tile whose 16-element groups are stored
// with their two middle quads swapped ("quad-swapped" layout, see
// stage_tile<true>), or through transposing LDS reads for row-major data.
// ---------------------------------------------------------------------------
__device__ __forceinline__ f32x16 mfma(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
  f32x2 v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

// Registers 8s .. 8s+7 of an accumulator -> one bf16 B operand.
__device__ __forceinline__ bf16x8 acc_to_operand(const f32x16& c, int s) {
  u32x4 p;
  p[0] = pack_bf16(c[8 * s + 0], c[8 * s + 1]);
  p[1] = pack_bf16(c[8 * s + 2], c[8 * s + 3]);
  p[2] = pack_bf16(c[8 * s + 4], c[8 * s + 5]);
  p[3] = pack_bf16(c[8 * s + 6], c[8 * s + 7]);
  return __builtin_bit_cast(bf16x8, p);
}

// c + the two bf16 elements of a word, in fp32.  DOT: as products with 1, one instruction; it rounds
// the pair once (2^20 draws: at most 9.9e-8 of the sum off, two fp32 additions 1.2e-7) and keeps
// denormals.  Otherwise each element is unpacked and added.
template <bool DOT>
__device__ __forceinline__ float sum_pair(uint32_t pair, float c) {
  if (DOT) {
    const bf16x2 one = __builtin_bit_cast(bf16x2, 0x3f803f80u);
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, pair), one, c, false);
  }
  c += __builtin_bit_cast(float, pair << 16);
  c += __builtin_bit_cast(float, pair & 0xffff0000u);
  return c;
}

// Transposing LDS read (ds_read_b64_tr_b16).  Within each group of 16 lanes,
// lane i passes the address of 4 consecutive bf16 of row (i / 4) at column
// group (i % 4) of a 4 x 16 block and receives column i of that block, rows
// 0..3.
__device__ __forceinline__ i16x4 lds_read_tr(const bf16_t* p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16(
      (__attribute__((address_space(3))) i16x4*)(p));
}

// ---------------------------------------------------------------------------
// LDS tiles are [rows][ROWBYTES] with unpadded rows, filled by direct
// global->LDS loads (each wave instruction moves 1 KB to consecutive LDS
// bytes, so rows cannot be padded).  Bank conflicts are avoided by permuting
// the 16-byte chunks of a row: chunk c of row `row` is stored at chunk position
// c ^ swz(row).  swz is a bijection of the rows that a 32x32x16 A-fragment read
// touches together (16 consecutive rows, same chunk) onto chunk positions, and
// it also separates the 4 consecutive rows that one transposing read touches.
// ---------------------------------------------------------------------------
template <int ROWBYTES>
__device__ __forceinline__ int swz(int row) {
  // 256- and 512-byte rows: 16 consecutive rows land on 16 distinct chunk positions (the
  // permutation touches the low four bits of the chunk index only)
  if (ROWBYTES == 256 || ROWBYTES == 512) return ((row & 3) << 2) | ((row >> 2) & 3);
  return (((row >> 1) & 1) << 2) | ((row >> 2) & 3);                  // 128-byte rows, 8 chunks
}

// byte offset of element (row, col) inside a tile whose rows hold ROWBYTES/2 bf16
template <int ROWBYTES>
__device__ __forceinline__ int tile_off(int row, int col) {
  return row * ROWBYTES + ((((col >> 3) ^ swz<ROWBYTES>(row)) << 4) | ((col & 7) << 1));
}

// Direct loads of a tile: wave w of NW moves the 1 KB blocks w, w+NW, ...; lane i of a block fills LDS
// chunk slot i, so it fetches the global chunk that the swizzle assigns to that slot.  They go through
// raw buffer descriptors, whose range check covers only the per-lane offset (never the scalar
// offset): descriptors are left open ended and callers keep every access inside their tensors
// themselves.
//
// The loads are inline asm, for kernels that rotate tile buffers at run
// time.  The compiler orders every LDS read after any direct load it can see that might
// write the same object, by waiting for ALL outstanding loads -- right for one buffer,
// but with buffers picked by a run-time index it cannot tell the tile being read from the
// tile being prefetched, and the wait would undo the prefetch.  Loads issued here are
// invisible to that analysis; callers order them against the reads themselves with
// wait_loads_and_barrier.  `rsrc` is the descriptor as four scalar words, `soff` a
// wave-uniform byte offset, `lds_addr` the wave-uniform LDS byte address of the 1 KB block
// (lane i writes bytes [16 i, 16 i + 16) of it).
__device__ __forceinline__ u32x4 make_rsrc_words(const void* base) {
  const uint64_t b = (uint64_t)base;
  u32x4 w;
  w[0] = __builtin_amdgcn_readfirstlane((uint32_t)b);
  w[1] = __builtin_amdgcn_readfirstlane((uint32_t)(b >> 32) & 0xffffu);
  w[2] = 0x7fffffffu;   // open ended
  w[3] = 0x00020000u;
  return w;
}
__device__ __forceinline__ void direct_load_16(u32x4 rsrc, int voff, int soff, uint32_t lds_addr) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
               ::"s"(lds_addr), "v"(voff), "s"(rsrc), "s"(soff)
               : "memory");
}
// The same OFF bytes further on both sides, for the blocks of a tile: two scalar additions, of which
// the second stands between the write of m0 and its use.
template <int OFF>
__device__ __forceinline__ void direct_load_16_at(u32x4 rsrc, int voff, int soff, uint32_t lds_addr) {
  int tmp;
  asm volatile("s_add_i32 m0, %1, %5\n\ts_add_i32 %0, %4, %5\n\tbuffer_load_dwordx4 %2, %3, %0 offen lds"
               : "=&s"(tmp)
               : "s"(lds_addr), "v"(voff), "s"(rsrc), "s"(soff), "n"(OFF)
               : "memory", "scc");
}
// Four bytes per lane: lane i writes bytes [4 i, 4 i + 4) of the 256-byte block at lds_addr.
__device__ __forceinline__ void direct_load_4(u32x4 rsrc, int voff, int soff, uint32_t lds_addr) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dword %1, %2, %3 offen lds"
               ::"s"(lds_addr), "v"(voff), "s"(rsrc), "s"(soff)
               : "memory");
}
__device__ __forceinline__ uint32_t lds_address(const void* p) {
  return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) char*)p;
}

// One tile through direct_load_16.  Rows at or beyond `valid` re-read the last valid row
// (finite values; callers mask what they compute from them).  Wave w of NW moves the 1 KB
// blocks w, w+NW, ...; `soff` is the tile's byte offset from the descriptor's base.
template <int ROWBYTES, int TILE_BYTES, int NW>
__device__ __forceinline__ void tile_load_asm(u32x4 rsrc, int soff, uint32_t lds_tile, int wave, int lane,
                                              int valid) {
  constexpr int CPR = ROWBYTES / 16;     // chunks per row
  constexpr int RPB = 1024 / ROWBYTES;   // rows per 1 KB block
  constexpr int NBLK = TILE_BYTES / 1024;
  static_assert(NBLK % NW == 0, "blocks of a tile are dealt evenly to the waves");
#pragma unroll
  for (int n = 0; n < NBLK / NW; ++n) {
    const int blk = wave + NW * n;
    int R = blk * RPB + lane / CPR;
    const int c = (lane % CPR) ^ swz<ROWBYTES>(R);
    if (R >= valid) R = valid - 1;
    direct_load_16(rsrc, R * ROWBYTES + c * 16, soff, lds_tile + blk * 1024);
  }
}

// The per-lane offset of a wave's first block of a full tile, which serves all of its blocks: block
// b of a wave differs from its first block by whole multiples of 16 rows, which the chunk permutation
// does not see, so the block part goes into the scalar offset.
template <int ROWBYTES, int NW>
__device__ __forceinline__ int tile_voff_full(int wave, int lane) {
  constexpr int CPR = ROWBYTES / 16;
  constexpr int RPB = 1024 / ROWBYTES;
  static_assert((NW * RPB) % 16 == 0, "blocks of a wave are whole multiples of 16 rows apart");
  const int j = lane / CPR;
  return j * ROWBYTES + (((lane % CPR) ^ swz<ROWBYTES>(wave * RPB + j)) << 4);
}
// The tiles of 64 rows of ROWBYTES of a token range, moved by NW waves through direct_load_16_at, one
// instruction at a time so that a kernel can spread them over its products.  A ragged last tile
// holds the last 64 rows of the range (`first()` of them belong to the tile before it), so that every
// load of a loop is the same; only a range of fewer than 64 rows re-reads its last row, and is moved
// by fill() alone.
template <int ROWBYTES, int NW>
struct RangeTiles {
  static constexpr int TB = 64 * ROWBYTES;
  static constexpr int LPT = TB / (1024 * NW);   // loads per wave and tile
  int rows, wave, lane, voff;

  __device__ __forceinline__ RangeTiles(int rows, int wave, int lane)
      : rows(rows), wave(wave), lane(lane), voff(tile_voff_full<ROWBYTES, NW>(wave, lane) + wave * 1024) {}
  // byte offset of the tile that starts at row `row`
  __device__ __forceinline__ int soff(int row) const {
    return __builtin_amdgcn_readfirstlane((row < rows - 64 ? row : rows - 64) * ROWBYTES);
  }
  // load I of the tile at `so` into the LDS tile at `lds`
  template <int I>
  __device__ __forceinline__ void load(u32x4 rsrc, int so, uint32_t lds) const {
    direct_load_16_at<1024 * NW * I>(rsrc, voff, so, lds + wave * 1024);
  }
  __device__ __forceinline__ void fill(u32x4 rsrc, int row, uint32_t lds) const {
    if (rows < 64) {
      tile_load_asm<ROWBYTES, TB, NW>(rsrc, 0, lds, wave, lane, rows);
      return;
    }
    const int so = soff(row);
    static_for<LPT>([&](auto IC) { load<decltype(IC)::value>(rsrc, so, lds); });
  }
  // Rows [first, first + count) of the tile that starts at `row` belong to it; the others are rows of the range that
  // have been taken already (or, of a range of fewer than 64, its last row).
  __device__ __forceinline__ int first(int row) const { return rows >= 64 && row > rows - 64 ? row + 64 - rows : 0; }
  __device__ __forceinline__ int count(int row) const { return row > rows - 64 ? rows - row : 64; }
};
// What such a row weighs when it is met again.  Not zero, which would make NaN of an infinity that the sums hold
// already; 2^-40 of its own contribution is 2^-16 of what fp32 rounds off beside that.
constexpr float kAgainLog2 = -40.f, kAgain = 0x1p-40f;
// The descriptor, or one that fetches nothing: a branch around loads that are spread over products
// would let the compiler move vector work out of its place.
__device__ __forceinline__ u32x4 rsrc_if(u32x4 rsrc, bool on) {
  rsrc[2] = on ? rsrc[2] : 0u;
  return rsrc;
}

// Resident operands by way of LDS.  A wave whose operand rows are 32 rows of memory (weights of its units) would read
// 32 bytes of each row per instruction, and the address unit takes such an instruction in some 43 cycles: 24 of them in
// each of eight waves hold a workgroup up for 3.5 - 5 us.  Whole rows through direct loads take 16 cycles per KB.
// stage_rows moves 32 rows of ROWBYTES bytes, `stride` apart in memory, into a block of LDS that only this wave uses
// (wait for its loads, no barrier), and staged_fragment reads k-step ks of the lane's row there.
template <int ROWBYTES>
__device__ __forceinline__ void stage_rows(u32x4 rsrc, int stride, int soff, uint32_t lds, int lane) {
  constexpr int CPR = ROWBYTES / 16, RPB = 1024 / ROWBYTES;
#pragma unroll
  for (int n = 0; n < 32 / RPB; ++n) {
    const int j = lane / CPR;
    direct_load_16(rsrc, j * stride + (((lane % CPR) ^ swz<ROWBYTES>(n * RPB + j)) << 4), soff + n * RPB * stride,
                   lds + n * 1024);
  }
}
template <int ROWBYTES>
__device__ __forceinline__ bf16x8 staged_fragment(const char* block, int lane, int ks) {
  return *reinterpret_cast<const bf16x8*>(block + (tile_off<ROWBYTES>(lane & 31, 8 * (lane >> 5)) ^ (32 * ks)));
}
// This wave's loads, and reads of LDS, are done.
__device__ __forceinline__ void wave_loads_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
__device__ __forceinline__ void wave_reads_done() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// Makes the compiler wait here for the loads that filled these operands.  Without it the wait
// goes to their first use inside the tile loop and stays there for every tile, as a count of
// outstanding loads in which the direct loads issued as inline asm are not known: it then
// waits for the tiles just requested and undoes their prefetch.
template <int N>
__device__ __forceinline__ void settle(bf16x8 (&x)[N]) {
#pragma unroll
  for (int i = 0; i < N; ++i) asm volatile("" : "+v"(x[i]));
}
__device__ __forceinline__ void settle(float& x) { asm volatile("" : "+v"(x)); }

// Keeps the value's computation where it stands between fenced products.  A running sum that is read
// only at the end of a tile is otherwise computed there, and its sixteen terms stay in registers.
template <typename T>
__device__ __forceinline__ void pin(T& x) {
  asm volatile("" : "+v"(x));
}

// Clears the rows of a 64-row tile in LDS that do not belong to it, by NT threads; a barrier has to follow.
// (For operands that meet zeros in those rows: an infinity there would make the product NaN.)
template <int ROWBYTES, int NT>
__device__ __forceinline__ void clear_other_rows(char* tile, int first, int count, int tid) {
#pragma unroll
  for (int o = tid * 16; o < 64 * ROWBYTES; o += NT * 16)
    if ((unsigned)(o / ROWBYTES - first) >= (unsigned)count) *reinterpret_cast<u32x4*>(tile + o) = u32x4{0u, 0u, 0u, 0u};
}

// Wait until at most N of this wave's direct loads are outstanding (and all of
// its LDS accesses are done), then workgroup barrier.  Written as one asm block:
// the compiler's own barrier would wait for every outstanding direct load and
// so serialise the prefetch with the computation.
template <int N>
__device__ __forceinline__ void wait_loads_and_barrier() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}
// Wait for this wave's LDS accesses only, then workgroup barrier (outstanding global
// stores and loads stay in flight).
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}
__device__ __forceinline__ bf16x8 join_tr(i16x4 lo, i16x4 hi) {
  typedef __attribute__((__vector_size__(8 * sizeof(short)))) short i16x8;
  i16x8 v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
  return __builtin_bit_cast(bf16x8, v);
}

// Combine a per-lane value across the two 32-lane halves of the wave with
// v_permlane32_swap: it exchanges the high half of its first register with the
// low half of its second, so starting from two copies of x one register ends
// up holding the low half's values in all lanes and the other the high half's.
// Written as inline asm with both registers read-write (the compiler builtin
// loses track of the second result when both inputs are copies of one value);
// the leading s_nop covers the VALU-write -> permlane-read hazard.
__device__ __forceinline__ void half_swap(float& a, float& b) {
  asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %1" : "+v"(a), "+v"(b));
}
__device__ __forceinline__ float half_swap_max(float x) {
  float a = x, b = x;
  half_swap(a, b);
  return fmaxf(a, b);
}
__device__ __forceinline__ float half_swap_sum(float x) {
  float a = x, b = x;
  half_swap(a, b);
  return a + b;
}

// 16 bytes a lane at base + off through the XCD's L2 to memory at once (agent scope), for whole lines that a launch writes
// last: what it leaves dirty there is written back when it ends, before the next one begins (21 streaming steps at 480p
// 1,170 -> 1,165 us, one layer 509.9 -> 509.1).  Half lines need the L2 to become whole ones.  `base` is wave-uniform, `off` below 2 GiB.
__device__ __forceinline__ void store_through(void* base, int off, u32x4 x) {
  constexpr int kAgent = 16;   // sc1
  __builtin_amdgcn_raw_buffer_store_b128(x, __builtin_amdgcn_make_buffer_rsrc(base, 0, 0x7fffffff, 0x00020000), off, 0, kAgent);
}

// Workgroup index -> logical work item so that consecutive logical items run
// on the same XCD: hardware deals workgroups round-robin over the 8 XCDs, each
// with its own L2, and items that share K/V or weights are consecutive.
__device__ __forceinline__ int xcd_swizzle(int wg, int per_xcd) {
  return (wg & 7) * per_xcd + (wg >> 3);
}

}  // namespace rehyat
