// Prefix pass over chunk states for gfx950 (Eq. 14-18): turns the per-segment
// partial sums written by the state kernel into the state S_t, z_t seen by each
// chunk of the window, s_0 = z_0 = 0, s_{t+1} = s_t + (tokens that entered the
// linear set between chunk t and chunk t+1).  Purely HBM-bound: each thread
// owns four consecutive state elements and walks the window's chunks in order
// (fixed summation order, so results are bit-reproducible).  S_t is written in
// bf16, transposed ([d][D']), ready to be an MFMA operand of the read-out; z_t
// stays fp32.  The running total is left in `carry` for the next window.
#include "rehyat_device.h"
#include "rehyat_kernels.h"

namespace rehyat {

// Pieces a thread loads before it sums them (in rehyat_kernels.h: also the suffix pass).  One
// piece at a time, each load behind the store of the state before it, the 20 segments of the 480p shape
// took 12.0 us at 47 MB, with eight loads ahead it takes 10.3 (suffix pass 18.1 and 12.5).
__device__ __forceinline__ void prefix_body(const PrefixArgs& a) {
  const int bh = blockIdx.y;
  const int idx = (blockIdx.x * 256 + threadIdx.x) * 4;
  if (idx >= a.elems) return;
  const float* part = a.partial + (int64_t)bh * a.partial_slots * a.elems + idx;
  float* carry = a.carry + (int64_t)bh * a.elems + idx;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  if (!a.first_window) acc = *reinterpret_cast<const f32x4*>(carry);
  const bool is_s = idx < a.s_elems;
  auto store = [&](int c) {   // the state of chunk c
    if (is_s) {
      u32x2 pk;
      pk[0] = pack_bf16(acc[0], acc[1]);
      pk[1] = pack_bf16(acc[2], acc[3]);
      *reinterpret_cast<u32x2*>(a.state_s + ((int64_t)bh * a.state_slots + c) * a.s_elems + idx) = pk;
    } else {
      *reinterpret_cast<f32x4*>(a.state_z + ((int64_t)bh * a.state_slots + c) * (a.elems - a.s_elems) +
                                (idx - a.s_elems)) = acc;
    }
  };
  if (a.n_chunks > 0) store(0);
  const int total = a.n_seg * a.nsplit;   // pieces, in the order they are summed
  int c = 0, sp = 0;
  for (int m = 0; m < total; m += kScanDepth) {
    f32x4 x[kScanDepth];
#pragma unroll
    for (int u = 0; u < kScanDepth; ++u)
      if (m + u < total) x[u] = *reinterpret_cast<const f32x4*>(part + (int64_t)(m + u) * a.elems);
#pragma unroll
    for (int u = 0; u < kScanDepth; ++u) {
      if (m + u < total) {
        acc += x[u];
        if (++sp == a.nsplit) {
          sp = 0;
          if (++c < a.n_chunks) store(c);
        }
      }
    }
  }
  *reinterpret_cast<f32x4*>(carry) = acc;
}

// ------------------------------------------------------------------------------------
// R_tau = sum over segments s >= tau of the chunk-state gradient partials (segment s holds
// dL/dS of chunk s+1, so this is the sum over chunks t > tau), r_tau likewise.  Each thread
// owns four consecutive elements and walks the segments from the last to the first (fixed
// order: bit-reproducible).
// ------------------------------------------------------------------------------------
__device__ __forceinline__ void suffix_body(const SuffixArgs& a) {
  const int bh = blockIdx.y;
  const int idx = (blockIdx.x * 256 + threadIdx.x) * 4;
  if (idx >= a.elems) return;
  const bool is_s = idx < a.s_elems;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  // pieces of segment c, then its sum goes out; kScanDepth pieces are loaded ahead of their sums
  const int ns = a.nsplit;
  const float* const base = a.part + (int64_t)bh * a.part_slots * a.elems + idx;
  int lc = a.n_seg - 1, lsp = 0;   // next piece to load
  int c = a.n_seg - 1, sp = 0;     // next piece to add
  while (c >= 0) {
    f32x4 x[kScanDepth];
#pragma unroll
    for (int u = 0; u < kScanDepth; ++u) {
      if (lc >= 0) {
        x[u] = *reinterpret_cast<const f32x4*>(base + ((int64_t)lc * ns + lsp) * a.elems);
        if (++lsp == ns) {
          lsp = 0;
          --lc;
        }
      }
    }
#pragma unroll
    for (int u = 0; u < kScanDepth; ++u) {
      if (c < 0) break;
      acc += x[u];
      if (++sp < ns) continue;
      if (is_s) {
        u32x2 pk;
        pk[0] = pack_bf16(acc[0], acc[1]);
        pk[1] = pack_bf16(acc[2], acc[3]);
        *reinterpret_cast<u32x2*>(a.Rt + ((int64_t)bh * a.slots + c) * a.s_elems + idx) = pk;
      } else {
        *reinterpret_cast<f32x4*>(a.r + ((int64_t)bh * a.slots + c) * a.dp + idx - a.s_elems) = acc;
      }
      sp = 0;
      --c;
    }
  }
}

__global__ void __launch_bounds__(256) prefix_kernel(PrefixArgs a) { prefix_body(a); }
// The suffix pass, and with a second layer of blocks a prefix pass.  (Layers, not rows behind the rows of the first: a
// grid holds 65,535 rows, and a call may have as many (batch, head)s.)
__global__ void __launch_bounds__(256) suffix_kernel(SuffixArgs a, PrefixArgs prefix) {
  if (blockIdx.z == 0) suffix_body(a);
  else prefix_body(prefix);
}

// Walks `total` pieces in order: add(load(0)), add(load(1)), ...  kScanDepth loads are in flight all the time; load(m) is
// called with rising m, and beyond the last piece again with total - 1.  Every load is unconditional: behind a branch the
// compiler does not know how many are in flight and waits for all of them (or for each one).
template <typename Load, typename Add>
__device__ __forceinline__ void scan_pieces(int total, Load load, Add add) {
  if (total <= 0) return;
  f32x4 x[kScanDepth], y[kScanDepth];
  auto fill = [&](f32x4 (&r)[kScanDepth], int m) {
#pragma unroll
    for (int u = 0; u < kScanDepth; ++u) r[u] = load(m + u < total ? m + u : total - 1);
  };
  fill(x, 0);
  int m = 0;
  for (; m + 2 * kScanDepth <= total; m += kScanDepth) {
#pragma unroll
    for (int u = 0; u < kScanDepth; ++u) {
      add(x[u]);
      x[u] = load(m + kScanDepth + u);
    }
  }
  if (m + kScanDepth < total) fill(y, m + kScanDepth);
#pragma unroll
  for (int u = 0; u < kScanDepth; ++u)
    if (m + u < total) add(x[u]);
#pragma unroll
  for (int u = 0; u < kScanDepth; ++u)
    if (m + kScanDepth + u < total) add(y[u]);
}

// state(c) = total - (frames of the softmax window of chunk c).  Bound by the round trips to the partial sums, which a
// second reading finds in the caches: as two launches, with the windows' loads one after the other, 20.5 us at the 480p
// shape, now 15.0.
__global__ void __launch_bounds__(256)
bidir_state_kernel(BidirArgs a) {
  const int bh = blockIdx.y;
  const int idx = (blockIdx.x * 256 + threadIdx.x) * 4;
  if (idx >= a.elems) return;
  const float* part = a.partial + (int64_t)bh * a.partial_slots * a.elems + idx;
  float* const keep = a.total + (int64_t)bh * a.elems + idx;
  const bool is_s = (int)blockIdx.x * 1024 < a.s_elems;   // the S part is a whole number of blocks
  auto store = [&](int c, f32x4 x) {
    if (is_s) {
      u32x2 pk;
      pk[0] = pack_bf16(x[0], x[1]);
      pk[1] = pack_bf16(x[2], x[3]);
      *reinterpret_cast<u32x2*>(a.state_s + ((int64_t)bh * a.state_slots + c) * a.s_elems + idx) = pk;
    } else {
      *reinterpret_cast<f32x4*>(a.state_z + ((int64_t)bh * a.state_slots + c) * (a.elems - a.s_elems) + (idx - a.s_elems)) = x;
    }
  };
  auto piece = [&](int m) { return *reinterpret_cast<const f32x4*>(part + (int64_t)m * a.elems); };
  f32x4 total = {0.f, 0.f, 0.f, 0.f};
  if (a.sum_total) {
    scan_pieces(a.T * a.nsplit, piece, [&](f32x4 x) { total += x; });
    *reinterpret_cast<f32x4*>(keep) = total;
  } else {
    total = *reinterpret_cast<const f32x4*>(keep);
  }
  auto lo = [&](int c) {   // first piece of chunk c's window (Eq. 12), and the one behind its last
    const int f = (a.chunk0 + c) * a.chunk - a.overlap;
    return ((f < 0 ? 0 : f) - a.frame0) * a.nsplit;
  };
  auto hi = [&](int c) {
    const int f = (a.chunk0 + c + 1) * a.chunk;
    return ((f > a.T ? a.T : f) - a.frame0) * a.nsplit;
  };
  int n = 0;
  for (int c = 0; c < a.n_chunks; ++c) n += hi(c) - lo(c);
  int lc = 0, lm = lo(0) - 1, next = 0;   // the piece to load, number `next` of the n
  int c = 0, left = hi(0) - lo(0);        // the chunk to finish, pieces of it to come
  f32x4 w = {0.f, 0.f, 0.f, 0.f};
  scan_pieces(n,
              [&](int m) {
                const int adv = m == next;   // (in arithmetic: no branch between loads)
                next += adv;
                lm += adv;
                const int cross = lm == hi(lc);
                lc += cross;
                lm += cross * (lo(lc) - lm);
                return piece(lm);
              },
              [&](f32x4 x) {
                w += x;
                if (--left == 0) {
                  store(c, total - w);
                  w = f32x4{0.f, 0.f, 0.f, 0.f};
                  ++c;
                  left = hi(c) - lo(c);
                }
              });
}

__global__ void __launch_bounds__(256)
state_out_kernel(StateOutArgs a) {
  const int bh = blockIdx.y;
  const int i = blockIdx.x * 256 + threadIdx.x;  // index into S_out [dprime][d]
  const int n = a.d * a.dprime;
  const float* c = a.carry + (int64_t)bh * (n + a.dprime);
  if (i < n) {
    const int e = i / a.d, col = i % a.d;
    a.S_out[(int64_t)bh * n + i] = c[col * a.dprime + e];
  }
  if (i < a.dprime) a.z_out[(int64_t)bh * a.dprime + i] = c[n + i];
}

// One tile of 64 features x 16 head-dimension columns of S per block, transposed through LDS
// both ways: the pieces -- the bulk of the bytes -- and the state slot are moved in 16-byte
// accesses along the workspace's [d][dprime] rows, the caller's [dprime][d] rows in 64-byte runs.
// Bound by its launch and one round trip to memory: the first pieces of S and of z are requested with the
// state.  With those of S behind the transpose and those of z one after the other at the end 5.6 us (12 heads of 128, 8
// pieces), now 4.9.
__global__ void __launch_bounds__(256)
step_state_kernel(StepStateArgs a) {
  __shared__ float tile[64][17];
  const int bh = blockIdx.z;
  const int f0 = blockIdx.x * 64, e0 = blockIdx.y * 16;
  const int tid = threadIdx.x;
  const int n = a.d * a.dprime, elems = n + a.dprime;
  float* S = a.S + (int64_t)bh * n;
  const float* part = a.partial + (int64_t)bh * a.partial_slots * elems;
  const int f4 = tid & 15, el = tid >> 4;   // features 4 f4 .. 4 f4 + 3 of row e0 + el of S^T
  const int64_t o = (int64_t)(e0 + el) * a.dprime + f0 + 4 * f4;
  const int zf = f0 + (tid & 63);           // z of this block's 64 features, by the first wave of the first row of blocks
  f32x4 x[kScanDepth];
  float zx[kScanDepth], zv = 0.f;
  auto piece = [&](int u) { return part + (int64_t)(u < a.nsplit ? u : a.nsplit - 1) * elems; };
  if (blockIdx.y == 0) {
    zv = a.z[(int64_t)bh * a.dprime + zf];
    if (a.nsplit > 0) {
#pragma unroll
      for (int u = 0; u < kScanDepth; ++u) zx[u] = piece(u)[n + zf];
    }
  }
  if (a.nsplit > 0) {
#pragma unroll
    for (int u = 0; u < kScanDepth; ++u) x[u] = *reinterpret_cast<const f32x4*>(piece(u) + o);
  }
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    const int idx = tid + 256 * m, row = idx >> 4, col = idx & 15;
    tile[row][col] = S[(int64_t)(f0 + row) * a.d + e0 + col];
  }
  __syncthreads();
  bf16_t* slot = a.state_s + (int64_t)bh * a.state_slots * n;
  {
    f32x4 v = {tile[4 * f4][el], tile[4 * f4 + 1][el], tile[4 * f4 + 2][el], tile[4 * f4 + 3][el]};
    if (a.write_slot) {
      u32x2 pk;
      pk[0] = pack_bf16(v[0], v[1]);
      pk[1] = pack_bf16(v[2], v[3]);
      *reinterpret_cast<u32x2*>(slot + o) = pk;
    }
#pragma unroll
    for (int u = 0; u < kScanDepth; ++u)
      if (u < a.nsplit) v += x[u];
#pragma unroll 8
    for (int sp = kScanDepth; sp < a.nsplit; ++sp) v += *reinterpret_cast<const f32x4*>(part + (int64_t)sp * elems + o);
#pragma unroll
    for (int i = 0; i < 4; ++i) tile[4 * f4 + i][el] = v[i];
  }
  __syncthreads();
  if (a.nsplit > 0) {   // nothing added: the caller's state stays as it is
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      const int idx = tid + 256 * m, row = idx >> 4, col = idx & 15;
      S[(int64_t)(f0 + row) * a.d + e0 + col] = tile[row][col];
    }
  }
  if (blockIdx.y == 0 && tid < 64) {
    if (a.write_slot) a.state_z[(int64_t)bh * a.state_slots * a.dprime + zf] = zv;
#pragma unroll
    for (int u = 0; u < kScanDepth; ++u)
      if (u < a.nsplit) zv += zx[u];
    for (int sp = kScanDepth; sp < a.nsplit; ++sp) zv += part[(int64_t)sp * elems + n + zf];
    if (a.nsplit > 0) a.z[(int64_t)bh * a.dprime + zf] = zv;
  }
}

// s_0 = 0, z_0 = 0 (Eq. 14-15) in the layout of the public state hook
__global__ void __launch_bounds__(256)
zero_state_kernel(float* S, float* z, int64_t n_s, int64_t n_z) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n_s) S[i] = 0.f;
  if (i < n_z) z[i] = 0.f;
}

hipError_t launch_zero_state(float* S, float* z, int BH, int d, int dprime, hipStream_t stream) {
  const int64_t n_s = (int64_t)BH * d * dprime, n_z = (int64_t)BH * dprime;
  hipLaunchKernelGGL(zero_state_kernel, dim3((unsigned)((n_s + 255) / 256)), dim3(256), 0, stream, S, z,
                     n_s, n_z);
  return hipGetLastError();
}

hipError_t launch_prefix(const PrefixArgs& a, hipStream_t stream) {
  dim3 grid((a.elems / 4 + 255) / 256, a.BH);
  hipLaunchKernelGGL(prefix_kernel, grid, dim3(256), 0, stream, a);
  return hipGetLastError();
}

hipError_t launch_suffix(const SuffixArgs& a, const PrefixArgs* prefix, hipStream_t stream) {
  PrefixArgs p{};
  if (prefix) p = *prefix;
  dim3 grid((a.elems / 4 + 255) / 256, a.BH, prefix ? 2 : 1);
  hipLaunchKernelGGL(suffix_kernel, grid, dim3(256), 0, stream, a, p);
  return hipGetLastError();
}

hipError_t launch_state_out(const StateOutArgs& a, hipStream_t stream) {
  dim3 grid((a.d * a.dprime + 255) / 256, a.BH);
  hipLaunchKernelGGL(state_out_kernel, grid, dim3(256), 0, stream, a);
  return hipGetLastError();
}

hipError_t launch_bidir_state(const BidirArgs& a, hipStream_t stream) {
  dim3 grid((a.elems / 4 + 255) / 256, a.BH);
  hipLaunchKernelGGL(bidir_state_kernel, grid, dim3(256), 0, stream, a);
  return hipGetLastError();
}

hipError_t launch_step_state(const StepStateArgs& a, hipStream_t stream) {
  dim3 grid(a.dprime / 64, a.d / 16, a.BH);
  hipLaunchKernelGGL(step_state_kernel, grid, dim3(256), 0, stream, a);
  return hipGetLastError();
}

}  // namespace rehyat
