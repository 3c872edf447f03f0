// kernel_small.h -- bf16 translation of small calls on the matrix cores.
//
// The persistent kernel (kernel_mfma.h) gives a workgroup tiles of 128 rows
// and hides the latency of a chunk behind the contraction of the one before.
// A call of a few row tiles leaves most compute units without a tile, and the
// others wait for every chunk's source rows and weights in turn.  Here a
// workgroup owns 32 target rows x 256 outputs of one (layer, K|V), reads its
// whole contraction (up to kSChunks chunks; longer ones in such segments) at
// once, with the weights of the first kSRing k-steps in flight beside it, and
// meets at one barrier before the products.  Bound by the latency of three
// dependent loads (alignment, source rows, later weights) and the launch.
//
// Operands, chunks, pair blocks and packed weights are those of the
// persistent kernel, so are the pooling, the angles, the split and the order of
// the sums: a row's bits do not depend on the size of the call it came in.  The
// product is taken as U = Z W^T, so a lane holds one output feature pair of 16
// tokens.
// Measured per call, the persistent kernel's time in brackets: 28 layers
// [512 -> 256], 16 tokens 10.8 us [21.9], 128 tokens 13.3 us [22.2]; 28 layers
// [3072 -> 512], spans of 1-2, 128 tokens 64 us [121]; with the caches flushed
// before each call 26 us [35], 25 us [32] and 111 us [144].
#pragma once

#include "kernel_mfma.h"

namespace kvx {

constexpr int kSRows = 32;  // target rows per workgroup: one matrix instruction's
constexpr int kSRing = 8;   // k-steps of weights in flight per wave (16: no faster, spills)

// The output's rotation, with the roundings of the persistent kernel's epilogue.

// Rotation of a pair by the angle of cos c, sin s.
__device__ __forceinline__ void rope(float x0, float x1, float c, float s, float& y0, float& y1) {
#pragma clang fp contract(off)
  y0 = __builtin_fmaf(x0, c, -(x1 * s));
  y1 = __builtin_fmaf(x0, s, x1 * c);
}
// cos c, sin s of an angle advanced by that of cos cd, sin sd.
__device__ __forceinline__ void advance_cs(float cd, float sd, float& c, float& s) {
#pragma clang fp contract(off)
  const float c2 = __builtin_fmaf(c, cd, -(s * sd));
  s = __builtin_fmaf(s, cd, c * sd);
  c = c2;
}

template <bool IDENT, int PREC>
__global__ void __launch_bounds__(256, 2) small_kernel(FusedArgs a) {
  // chunks per segment (the span path holds second entries and their angles
  // too); 66 KB of LDS at most, two workgroups a compute unit
  constexpr int kSChunks = IDENT ? 4 : 2;
  constexpr int kSLD = kSChunks * 128 + 8;  // LDS row stride (bf16): rows 4 banks apart
  __shared__ __attribute__((aligned(16))) bf16_t z[2][kSRows * kSLD];
  __shared__ double fsl[kMaxHalfDim];
  // each XCD takes a contiguous range of workgroups, row tiles fastest, so
  // the workgroups that share a weight slice share an L2
  const int id = xcd_remap(blockIdx.x, gridDim.x);
  const int rt = id % a.row_tiles;
  int rest = id / a.row_tiles;
  const int nt = rest % a.n_tiles;
  rest /= a.n_tiles;
  const int kv = rest & 1, l = rest >> 1;
  const bool is_k = kv == 0;
  const int b = find_context(a.ba, rt);
  const int t0 = (rt - a.ba.tile_start[b]) * kSRows;
  const int tt = a.ba.t_tgt[b];
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int half = a.ds / 2, nch = a.din / 128, ksall = a.din / 16;

  // This thread's row and 8-pair group of each chunk.  Loads are
  // unconditional: a row past the context's end, and an absent entry, read
  // the zero area.
  const int r = tid / 8, g = tid % 8;
  const double myf = tid < half ? a.fs[tid] : 0.0;
  int e0 = 0, n = t0 + r < tt ? 1 : 0, k0 = t0 + r, k1 = 0;
  float w0 = 1.f, w1 = 0.f;
  if constexpr (!IDENT) {
    const int tc = a.ba.row_base[b] + (n ? t0 + r : tt - 1);
    e0 = a.row_ptr[tc];
    n = n ? a.row_ptr[tc + 1] - e0 : 0;
    const int32_t* zi = reinterpret_cast<const int32_t*>(a.zsink);
    const float* zf = reinterpret_cast<const float*>(a.zsink);
    k0 = *(n > 0 ? a.col_idx + e0 : zi);
    w0 = *(n > 0 ? a.weight + e0 : zf);
    k1 = *(n > 1 ? a.col_idx + e0 + 1 : zi);
    w1 = *(n > 1 ? a.weight + e0 + 1 : zf);
  }
  auto group_at = [&](int c, int& i0) KVX_INLINE -> const bf16_t* {
    const int pair = 64 * c + 8 * g;
    const int hp = pair / half;
    i0 = pair - hp * half;
    const int j = hp / a.hs;
    return a.src[kv] + a.layer_map[l * a.mix + j] * a.ss.l + b * a.ss.b +
           (hp - j * a.hs) * a.ss.h + i0;
  };
  uint4 x[kSChunks][2], y[IDENT ? 1 : kSChunks][2];
  // first and second entries of the segment's chunks (chunks past the
  // contraction read the zero area)
  auto issue = [&](int c0) KVX_INLINE {
    const bf16_t* gp[kSChunks];
#pragma unroll
    for (int c = 0; c < kSChunks; ++c) {
      int i0;
      gp[c] = group_at(c0 + c < nch ? c0 + c : 0, i0);
    }
#pragma unroll
    for (int c = 0; c < kSChunks; ++c) {
      const bf16_t* p = n > 0 && c0 + c < nch ? gp[c] + k0 * a.ss.t : a.zsink;
      x[c][0] = *reinterpret_cast<const uint4*>(p);
      x[c][1] = *reinterpret_cast<const uint4*>(p + half);
      if constexpr (!IDENT) {
        const bf16_t* q = n > 1 && c0 + c < nch ? gp[c] + k1 * a.ss.t : a.zsink;
        y[c][0] = *reinterpret_cast<const uint4*>(q);
        y[c][1] = *reinterpret_cast<const uint4*>(q + half);
      }
    }
  };
  issue(0);

  // this wave's pair block: outputs c .. c + 31 of a target head and their
  // RoPE partners; a block past dout runs block 0's and stores nothing
  const int npb = a.dout / 64, per_head = a.dt / 64;
  const bool on = 4 * nt + w < npb;
  const int pb = on ? 4 * nt + w : 0;
  const int hp = pb / per_head, fo = 32 * (pb - hp * per_head);
  const bf16x8* wp = (PREC == kF16 ? a.wh[kv] : a.wp[kv]) +
                     (static_cast<int64_t>(l) * (a.dout / 32) + (hp * a.dt + fo) / 32) * ksall * 64 +
                     lane;
  const int64_t w1off = static_cast<int64_t>(per_head) * ksall * 64;
  bf16x8 wf[kSRing][2];
  // reload ring slot i with k-step ks (past the contraction: the last one again)
  auto load_w = [&](int i, int ks) KVX_INLINE {
    const int k = ks < ksall ? ks : ksall - 1;
    wf[i][0] = wp[k * 64];
    wf[i][1] = wp[w1off + k * 64];
  };
#pragma unroll
  for (int i = 0; i < kSRing; ++i) load_w(i, i);
  const int fi = fo + lane % 32;  // output pair within the head
  const float* bl = a.bias[kv] + static_cast<int64_t>(l) * a.dout + hp * a.dt + fi;
  const float b0 = bl[0], b1 = bl[a.dt / 2];
  const double ft = a.ft[fi];
  if (tid < kMaxHalfDim) fsl[tid] = myf;
  lds_barrier();

  float ca[8], sa[8], cb[IDENT ? 1 : 8], sb[IDENT ? 1 : 8];
  auto transform = [&](int c, int C) KVX_INLINE {
    bf16_t* hi = z[0] + r * kSLD + c * 128 + 8 * g;
    bf16_t* lo = z[1] + r * kSLD + c * 128 + 8 * g;
    if (IDENT && !is_k && PREC != kF16) {
      *reinterpret_cast<uint4*>(hi) = x[c][0];
      *reinterpret_cast<uint4*>(hi + 64) = x[c][1];
      return;
    }
    int i0;
    const bf16_t* gp = group_at(C, i0);
    float x0[8], x1[8], z0[8], z1[8];
    unpack8(x[c][0], x0);
    unpack8(x[c][1], x1);
    // the frequencies of a thread's group repeat every chunk at Ds = 128
    if (is_k && (C == 0 || half != 64)) {
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        rope_cs(fsl[i0 + i], k0, ca[i], sa[i]);
        if constexpr (!IDENT) rope_cs(fsl[i0 + i], n > 1 ? k1 - k0 : 0, cb[i], sb[i]);
      }
    }
    // the persistent kernel's resident order, where it would take the call, adds
    // a K row's later entries in the first one's frame, the others to the
    // rotated sum
    const bool frame = !IDENT && a.interleave == 2;
    if constexpr (!IDENT) {
      // the first two entries, K in the first one's frame
      float v0[8], v1[8];
      unpack8(y[c][0], v0);
      unpack8(y[c][1], v1);
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        if (is_k) unrope(v0[i], v1[i], cb[i], sb[i], v0[i], v1[i]);
        z0[i] = pool2(w0, x0[i], w1, v0[i]);
        z1[i] = pool2(w0, x1[i], w1, v1[i]);
      }
    } else {
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        z0[i] = x0[i];
        z1[i] = x1[i];
      }
    }
    auto rotate = [&]() KVX_INLINE {
#pragma unroll
      for (int i = 0; i < 8; ++i) unrope(z0[i], z1[i], ca[i], sa[i], z0[i], z1[i]);
    };
    if (is_k && !frame) rotate();
    if constexpr (!IDENT) {
      for (int e = e0 + 2; e < e0 + n; ++e) {
        const int k = a.col_idx[e];
        const float we = a.weight[e];
        const bf16_t* p = gp + k * a.ss.t;
        const uint4 q0 = *reinterpret_cast<const uint4*>(p);
        const uint4 q1 = *reinterpret_cast<const uint4*>(p + half);
        float v0[8], v1[8], cs[8], sn[8];
        if (is_k) {  // while the entry's rows arrive
#pragma unroll
          for (int i = 0; i < 8; ++i) rope_cs(fsl[i0 + i], frame ? k - k0 : k, cs[i], sn[i]);
        }
        unpack8(q0, v0);
        unpack8(q1, v1);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          if (is_k) unrope(v0[i], v1[i], cs[i], sn[i], v0[i], v1[i]);
          z0[i] = __builtin_fmaf(we, v0[i], z0[i]);
          z1[i] = __builtin_fmaf(we, v1[i], z1[i]);
        }
      }
    }
    if (is_k && frame) rotate();
    if (PREC == kF16) {
      *reinterpret_cast<uint4*>(hi) = pack8_f16(z0);
      *reinterpret_cast<uint4*>(hi + 64) = pack8_f16(z1);
      return;
    }
    const uint4 h0 = pack8(z0), h1 = pack8(z1);
    *reinterpret_cast<uint4*>(hi) = h0;
    *reinterpret_cast<uint4*>(hi + 64) = h1;
    if (PREC == kBF16X2) {
      residual8(z0, h0, x0);
      residual8(z1, h1, x1);
      *reinterpret_cast<uint4*>(lo) = pack8(x0);
      *reinterpret_cast<uint4*>(lo + 64) = pack8(x1);
    }
  };

  f32x16 acc0 = {}, acc1 = {};
  const bool split = PREC == kBF16X2 && (!IDENT || is_k);
  // Split k-steps of a chunk, all without a table.  The table's bytes are read
  // as whole words (it ends on a multiple of 256 bytes), by scalar loads: a
  // vector load of each byte waits for the weights in flight (28 layers [512 ->
  // 256], 288 tokens 22.4 us so, 18.5 us; [3072 -> 512], 96 tokens 98.9, 56.3).
  const uint32_t* stab = reinterpret_cast<const uint32_t*>(split ? a.split_mask : nullptr);
  const int s0 = (l * 2 + kv) * nch;
  auto split_steps = [&](int C) KVX_INLINE -> uint32_t {
    const int o = s0 + (C < nch ? C : 0);
    return !split ? 0u : stab ? stab[o / 4] >> (8 * (o % 4)) : 0xffu;
  };
  for (int c0 = 0; c0 < nch; c0 += kSChunks) {
    uint32_t ksplit[kSChunks];
#pragma unroll
    for (int c = 0; c < kSChunks; ++c) ksplit[c] = split_steps(c0 + c);
#pragma unroll
    for (int c = 0; c < kSChunks; ++c)
      if (c0 + c < nch) transform(c, c0 + c);
    const bool more = c0 + kSChunks < nch;
    if (more) issue(c0 + kSChunks);
    lds_barrier();
#pragma unroll
    for (int c = 0; c < kSChunks; ++c) {
#pragma unroll
      for (int i = 0; i < kSRing; ++i) {
        if (c0 + c < nch) {
          const bf16_t* zr = z[0] + (lane % 32) * kSLD + c * 128 + i * 16 + 8 * (lane / 32);
          auto mm = [&](const bf16_t* p) KVX_INLINE {
            const bf16x8 v = *reinterpret_cast<const bf16x8*>(p);
            if constexpr (PREC == kF16) {
              const f16x8 h = __builtin_bit_cast(f16x8, v);
              acc0 = __builtin_amdgcn_mfma_f32_32x32x16_f16(
                  h, __builtin_bit_cast(f16x8, wf[i][0]), acc0, 0, 0, 0);
              acc1 = __builtin_amdgcn_mfma_f32_32x32x16_f16(
                  h, __builtin_bit_cast(f16x8, wf[i][1]), acc1, 0, 0, 0);
            } else {
              acc0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v, wf[i][0], acc0, 0, 0, 0);
              acc1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v, wf[i][1], acc1, 0, 0, 0);
            }
          };
          mm(zr);
          if ((ksplit[c] >> i) & 1) mm(zr + kSRows * kSLD);
        }
        load_w(i, (c0 + c) * 8 + i + kSRing);
      }
    }
    if (more) lds_barrier();
  }

  // bias, target rotation, bf16; a half-wave stores 32 features of a row.  The
  // angle is the persistent kernel's: formed for the first 32 rows of its
  // 128-row tile and advanced by the rotation by 32 positions.
  if (!on) return;
  float c32 = 1.f, s32 = 0.f;
  if (is_k) rope_cs(ft, 32, c32, s32);
  const int ahead = t0 % kMT;  // rows from that tile's first to this one's
  bf16_t* dst = a.tgt[kv] + l * a.ts.l + hp * a.ts.h + fi;
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const int t = t0 + 8 * (v / 4) + 4 * (lane / 32) + v % 4;
    if (t >= tt) continue;
    float u0 = acc0[v] + b0, u1 = acc1[v] + b1;
    if (is_k) {
      float cs, sn;
      rope_cs(ft, t - ahead, cs, sn);
      for (int m = 0; m < ahead; m += kSRows) advance_cs(c32, s32, cs, sn);
      rope(u0, u1, cs, sn, u0, u1);
    }
    const int32_t blk = a.pg.table ? a.pg.table[b * a.pg.max_blocks + t / a.pg.block_size] : 0;
    bf16_t* q = dst + target_row(a.pg, a.ts, b, t, blk);
    q[0] = __builtin_bit_cast(bf16_t, static_cast<__bf16>(u0));
    q[a.dt / 2] = __builtin_bit_cast(bf16_t, static_cast<__bf16>(u1));
  }
}

}  // namespace kvx
