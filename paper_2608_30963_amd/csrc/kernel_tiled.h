// kernel_tiled.h -- general translation kernel, fp32 arithmetic (any even
// head_dim, any layer mixing, identity or CSR alignment).  Serves fp32 plans
// and shapes the bf16 matrix-core kernel does not tile.
//
// Every product and sum is fp32 (v_mfma_f32_32x32x2_f32, exact fp32 multiply-
// add), for bf16 storage too, whose values are widened exactly.
//
// One workgroup owns (target layer l, K|V, context b, kGRows target rows, up
// to four pair blocks of outputs).  SHARE: the rows of all contexts are tiled
// as one list, so that contexts of a few rows share a tile instead of padding
// one each.  A pair block is 32 consecutive entries of
// the flattened (target head, i < Dt/2) list: the outputs i and their RoPE
// partners i + Dt/2, which the two accumulators of a wave hold in the same
// lane, so the target rotation needs no exchange.  The contraction runs over
// chunks of 64 source RoPE pairs (128 slots: first members in slots 0..63,
// second members in 64..127) of the flattened (mixed layer, head, i < Ds/2)
// list, zero-padded to whole chunks:
//   1. the workgroup gathers a chunk of its rows -- a wave takes whole rows, a
//      lane one pair, so loads are coalesced at any head_dim and alignment --
//      undoes the source RoPE, pools in fp32 and writes fp32 rows to LDS (two
//      buffers; the next chunk's first entries are loaded before the current
//      chunk's products and finished after them);
//   2. each wave contracts the chunk with its pair block.  With fewer than
//      four pair blocks in the workgroup the waves split the chunk's slots
//      instead and their sums are added through LDS at the end, in wave order;
//   3. bias, target RoPE on K, store (a half-wave stores 32 consecutive
//      elements of a row).
//
// Bound by the fp32 matrix rate (64 cycles per 4096-flop instruction).  A
// 32-row tile is the smallest a 32x32 instruction fills; it keeps the grid
// fine (four workgroups fit a CU, and hide each other's gathers) and costs
// only 16 bytes of weights per clock and CU from the L2.  Weights are packed
// at plan time so that a wave's fragment of 8 slots is one contiguous load.
// Measured, against a kernel of scalar dot products over weights read with a
// stride of din (in brackets): 28 layers of [512 -> 256] at 1024 tokens fp32
// 0.166 ms, 91 TFLOP/s of the 154 a large fp32 product reaches [5.8 ms]; 24
// layers of [640 -> 320] at head_dim 80, 1024 tokens bf16 0.27 ms [4.6 ms];
// 4 layers of [128 -> 128] at 256 tokens fp32 10.7 us a call [34.7 us].  64
// contexts of one token (SHARE, in brackets a tile each): 28 layers of [512 ->
// 256] fp32 29 us [269 us], 24 of [640 -> 320] bf16 36 us [443 us].
#pragma once

#include "common.h"

namespace kvx {

constexpr int kGRows = 32;             // target rows per workgroup
constexpr int kGSlots = 128;           // contraction slots per chunk (64 pairs)
constexpr int kGLD = kGSlots + 4;      // LDS row stride (floats): rows 4 banks apart
constexpr int kGQ = kGSlots / 8;       // 8-slot groups per chunk

template <typename T>
struct TiledArgs {
  const T* src[2];          // source K, V
  Strides ss;
  T* tgt[2];                // target K, V
  Strides ts;
  const T* w[2];            // packed [Lt][npb][nch * kGQ][2][64 lanes][4] (pack_tiled);
                            // row kernel: [Lt][dout][din], nn.Linear order
  const float* bias[2];     // [Lt][dout] (zeros when the translator has none)
  const int32_t* layer_map; // [Lt][mix]
  int32_t mix, hs, ds, ht, dt, din, dout;
  const double* fs;         // [ds/2] source theta_i / 2pi (zeros: RoPE off)
  const double* ft;         // [dt/2] target
  const int32_t* row_ptr;   // CSR alignment (unused when identity != 0)
  const int32_t* col_idx;
  const float* weight;
  int32_t identity;
  int32_t row_tiles;        // tiles of kGRows rows, all contexts
  int32_t npb, nch;         // pair blocks of the output, chunks of the contraction
  int32_t group;            // pair blocks per workgroup: 4 (with a remainder of 2, 1) or 1
  Paging pg;                // optional paged target layout
  BatchArgs ba;             // SHARE: tile_start holds the contexts' first rows in the list
};

// Context and position of row `row` of the list of all contexts' rows
// (position -1 past its end).
__device__ __forceinline__ int2 list_row(const BatchArgs& ba, int row) {
  int2 r = make_int2(0, row);
  for (int b = 1; b < ba.n; ++b)
    if (ba.tile_start[b] <= row) r = make_int2(b, row - ba.tile_start[b]);
  return row < ba.tile_start[ba.n] ? r : make_int2(0, -1);
}

// Workgroups along the output: whole groups of four pair blocks, then the
// remainder as 2 and 1, so that every wave of every workgroup has work.
__host__ __device__ constexpr int tiled_ntiles(int npb, int group) {
  return group == 1 ? npb : npb / 4 + (npb % 4 == 3 ? 2 : npb % 4 != 0);
}

__device__ __forceinline__ f32x4 load_w4(const float* p) { return *reinterpret_cast<const f32x4*>(p); }
__device__ __forceinline__ f32x4 load_w4(const bf16_t* p) {
  const uint2 r = *reinterpret_cast<const uint2*>(p);
  return f32x4{__uint_as_float(r.x << 16), __uint_as_float(r.x & 0xffff0000u),
               __uint_as_float(r.y << 16), __uint_as_float(r.y & 0xffff0000u)};
}

template <typename T, bool SHARE>
__global__ void __launch_bounds__(256, 4) tiled_kernel(TiledArgs<T> a) {
  __shared__ __attribute__((aligned(16))) float z[2][kGRows * kGLD];
  __shared__ int2 rowi[SHARE ? kGRows : 1];  // the rows' contexts and positions
  // each XCD takes a contiguous range of workgroups, row tiles fastest, so
  // the workgroups that share a layer's weights share an L2
  const int64_t total = static_cast<int64_t>(gridDim.x) * gridDim.y;
  const int64_t lin = static_cast<int64_t>(blockIdx.y) * gridDim.x + blockIdx.x;
  const int64_t xq = total / 8, xr = total % 8, xcd = lin % 8;
  const int64_t id = xcd * xq + (xcd < xr ? xcd : xr) + lin / 8;
  const int rt = static_cast<int>(id % a.row_tiles);
  const int64_t rest = id / a.row_tiles;
  const int n_tiles = tiled_ntiles(a.npb, a.group);
  const int nt = static_cast<int>(rest % n_tiles);
  const int lk = static_cast<int>(rest / n_tiles);
  const int l = lk >> 1, kv = lk & 1;
  int pb0 = nt, nb = 1;  // first pair block, pair blocks of this workgroup
  if (a.group == 4) {
    const int full = a.npb / 4;
    pb0 = nt <= full ? 4 * nt : 4 * full + 2;
    nb = nt < full ? 4 : (nt == full && a.npb % 4 >= 2 ? 2 : 1);
  }
  const int b = SHARE ? 0 : find_context(a.ba, rt);
  const int t0 = SHARE ? 0 : (rt - a.ba.tile_start[b]) * kGRows;
  const int tt = SHARE ? 0 : a.ba.t_tgt[b];
  if constexpr (SHARE) {
    if (threadIdx.x < kGRows) rowi[threadIdx.x] = list_row(a.ba, rt * kGRows + threadIdx.x);
    __syncthreads();
  }
  // context and position of row r of the tile, and whether there is such a row
  auto row_at = [&](int r) __attribute__((always_inline)) -> int2 {
    if constexpr (SHARE) return rowi[r];
    return make_int2(b, t0 + r);
  };
  auto is_row = [&](int t) __attribute__((always_inline)) { return SHARE ? t >= 0 : t < tt; };
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int hd = a.ds / 2;
  const int npairs = a.din / 2;
  const T* src = a.src[kv] + b * a.ss.b;

  // this wave's rows of the tile: w + 4 i
  constexpr int kR = kGRows / 4;
  int e0[kR], e1[kR], k0[kR];
  int ctx[SHARE ? kR : 1];
  float w0[kR];
#pragma unroll
  for (int i = 0; i < kR; ++i) {
    const int2 ri = row_at(w + 4 * i);
    const int t = SHARE ? __builtin_amdgcn_readfirstlane(ri.y) : ri.y;
    const int c = SHARE ? __builtin_amdgcn_readfirstlane(ri.x) : b;
    if constexpr (SHARE) ctx[i] = c;
    e0[i] = 0;
    e1[i] = is_row(t) ? 1 : 0;
    k0[i] = t;
    w0[i] = 1.f;
    if (!a.identity && is_row(t)) {
      e0[i] = a.row_ptr[a.ba.row_base[c] + t];
      e1[i] = a.row_ptr[a.ba.row_base[c] + t + 1];
      if (e1[i] > e0[i]) {
        k0[i] = a.col_idx[e0[i]];
        w0[i] = a.weight[e0[i]];
      }
    }
  }

  // source element offset of token k of row i's context
  auto token = [&](int i, int k) __attribute__((always_inline)) -> int64_t {
    if constexpr (SHARE) return ctx[i] * a.ss.b + k * a.ss.t;
    return k * a.ss.t;
  };

  // the lane's pair of a chunk: its first member at token 0 (SHARE: of context
  // 0; nullptr past the last pair) and its frequency.  First entries are loaded unconditionally (a
  // load inside a branch makes the compiler drain every load in flight at the
  // merge): lanes and rows without one read the frequency table, whose 8 Ds/2
  // bytes hold both members, and are cleared.
  const T* xp = nullptr;
  double f = 0.0;
  T x0[kR], x1[kR];
  auto load_first = [&](int c) __attribute__((always_inline)) {
    const int pair = 64 * c + lane;
    const bool ok = pair < npairs;
    const int hp = ok ? pair / hd : 0, i = ok ? pair - hp * hd : 0;
    const int j = hp / a.hs, h = hp - j * a.hs;
    xp = ok ? src + a.layer_map[l * a.mix + j] * a.ss.l + h * a.ss.h + i : nullptr;
    f = kv == 0 ? a.fs[i] : 0.0;
#pragma unroll
    for (int r = 0; r < kR; ++r) {
      const T* p = ok && e1[r] > e0[r] ? xp + token(r, k0[r]) : reinterpret_cast<const T*>(a.fs);
      x0[r] = p[0];
      x1[r] = p[hd];
    }
  };
  auto finish = [&](float* buf) __attribute__((always_inline)) {
#pragma unroll
    for (int r = 0; r < kR; ++r) {
      const bool any = xp && e1[r] > e0[r];
      float y0 = any ? load_f32(&x0[r]) : 0.f, y1 = any ? load_f32(&x1[r]) : 0.f;
      if (kv == 0) {  // undo the source rotation at source position k
        float cs, sn;
        rope_cs(f, k0[r], cs, sn);
        const float v0 = y0 * cs + y1 * sn, v1 = y1 * cs - y0 * sn;
        y0 = v0;
        y1 = v1;
      }
      float z0 = w0[r] * y0, z1 = w0[r] * y1;
      if (xp)
        for (int e = e0[r] + 1; e < e1[r]; ++e) {
          const int k = a.col_idx[e];
          const float we = a.weight[e];
          const T* p = xp + token(r, k);
          y0 = load_f32(p);
          y1 = load_f32(p + hd);
          if (kv == 0) {
            float cs, sn;
            rope_cs(f, k, cs, sn);
            const float v0 = y0 * cs + y1 * sn, v1 = y1 * cs - y0 * sn;
            y0 = v0;
            y1 = v1;
          }
          z0 += we * y0;
          z1 += we * y1;
        }
      buf[(w + 4 * r) * kGLD + lane] = z0;
      buf[(w + 4 * r) * kGLD + 64 + lane] = z1;
    }
  };

  // wave -> (pair block, share of each chunk's slots)
  const int pb = pb0 + w % nb, part = w / nb, parts = 4 / nb;
  const int q0 = part * kGQ / parts, q1 = (part + 1) * kGQ / parts;
  const int64_t qn = static_cast<int64_t>(a.nch) * kGQ;
  const T* wp = a.w[kv] + ((static_cast<int64_t>(l) * a.npb + pb) * qn) * 512 + lane * 4;
  f32x16 acc0 = {}, acc1 = {};
  // fragments of four 8-slot groups, each reloaded with the group four further
  // on as soon as its products have issued (the scheduling barriers keep the
  // compiler from moving the loads next to their use)
  f32x4 wa[4], wb[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    wa[u] = load_w4(wp + static_cast<int64_t>(q0 + u) * 512);
    wb[u] = load_w4(wp + static_cast<int64_t>(q0 + u) * 512 + 256);
  }
  load_first(0);
  finish(z[0]);
  __syncthreads();
  for (int c = 0; c < a.nch; ++c) {
    const bool more = c + 1 < a.nch;
    if (more) load_first(c + 1);
    // lane l holds row l % 32, slots 8 q + 4 (l / 32) + e of step (q, e)
    const float* zr = z[c & 1] + (lane % 32) * kGLD + 4 * (lane / 32);
    for (int q = q0; q < q1; q += 4) {  // shares are multiples of 4 groups
      // the wave's next four groups (after the last, the same again)
      const int64_t qnext = q + 4 < q1 ? static_cast<int64_t>(c) * kGQ + q + 4
                                       : static_cast<int64_t>(more ? c + 1 : c) * kGQ + q0;
      const T* p = wp + qnext * 512;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const f32x4 zv = *reinterpret_cast<const f32x4*>(zr + 8 * (q + u));
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          acc0 = __builtin_amdgcn_mfma_f32_32x32x2f32(zv[e], wa[u][e], acc0, 0, 0, 0);
          acc1 = __builtin_amdgcn_mfma_f32_32x32x2f32(zv[e], wb[u][e], acc1, 0, 0, 0);
        }
        wa[u] = load_w4(p + u * 512);
        wb[u] = load_w4(p + u * 512 + 256);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    if (more) finish(z[(c + 1) & 1]);
    __syncthreads();
  }

  // sums of the waves that share a pair block, in wave order
  if (parts > 1) {
    float* red = z[0];  // [wave - nb][32 registers][64 lanes], 24 KiB at most
    if (part > 0) {
      float* q = red + (w - nb) * 2048 + lane;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        q[v * 64] = acc0[v];
        q[(16 + v) * 64] = acc1[v];
      }
    }
    __syncthreads();
    if (part > 0) return;
    for (int s = 1; s < parts; ++s) {
      const float* q = red + (w + s * nb - nb) * 2048 + lane;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        acc0[v] += q[v * 64];
        acc1[v] += q[(16 + v) * 64];
      }
    }
  }

  // bias, target rotation, store: lane holds pair 32 pb + lane % 32 of rows
  // 8 (v / 4) + 4 (lane / 32) + v % 4
  const int ht2 = a.dt / 2;
  const int p = 32 * pb + lane % 32;
  if (p >= a.dout / 2) return;
  const int h = p / ht2, i = p - h * ht2;
  const int o0 = h * a.dt + i, o1 = o0 + ht2;
  const float* bl = a.bias[kv] + static_cast<int64_t>(l) * a.dout;
  const float b0 = bl[o0], b1 = bl[o1];
  const double ft = kv == 0 ? a.ft[i] : 0.0;
  T* dst = a.tgt[kv] + l * a.ts.l + h * a.ts.h + i;
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const int2 ri = row_at(8 * (v / 4) + 4 * (lane / 32) + v % 4);
    const int t = ri.y;
    if (!is_row(t)) continue;
    float u0 = acc0[v] + b0, u1 = acc1[v] + b1;
    if (kv == 0) {
      float cs, sn;
      rope_cs(ft, t, cs, sn);
      const float y0 = u0 * cs - u1 * sn, y1 = u1 * cs + u0 * sn;
      u0 = y0;
      u1 = y1;
    }
    const int32_t blk = a.pg.table ? a.pg.table[ri.x * a.pg.max_blocks + t / a.pg.block_size] : 0;
    T* q = dst + target_row(a.pg, a.ts, ri.x, t, blk);
    q[0] = store_cvt<T>(u0);
    q[ht2] = store_cvt<T>(u1);
  }
}

}  // namespace kvx
