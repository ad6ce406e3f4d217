// Gate and up projections of a batch (3..16 rows, bf16 weights, any width) on
// the matrix cores (narrow blocks of many neurons: mlp_gateup_narrow.hip).
//
//   v_bj = SiLU(x_b . W_gate[:, j]);  (b, j) active when |v_bj| >= t
//   h_bj = v_bj * (x_b . W_up[:, j])  for active (b, j), else 0
// W_up rows are read for the union of the rows' active neurons only (Eq. 1,
// 2 and 5 with one mask per row).
//
// Measured (this kernel, us): 4096 x 11008 dense at 16 rows 32.4 (5.6 TB/s; the
// kernel that kept x in registers, one sixteenth of the columns per wave, 43),
// k = 0.7 at 8 / 16 rows 33 / 35 (40 / 44); 5120 x 13824 at 16 rows 53 (63);
// 8192 x 28672 dense at 8 rows 144 (6.5 TB/s; the fused kernel in two passes
// 2 x 283); 2856 x 7001 at 11 rows 22 (2 x 40).
//
// What bounds it: reading the weights (2 or 3 products per weight and row
// group are far below the matrix rate), as long as enough bytes are in
// flight and x, which every block needs whole, does not cost as much as the
// weights.  So:
//  - A wave goes through its columns on the outside and through the block's
//    neuron tiles on the inside, so that x is read once per pass over the
//    neurons, whatever the width.  x comes as fp32 (whole lines) and is split
//    into bf16 planes by the wave that multiplies it, in the time it waits
//    for weights (two planes: 16 of x's 24 bits; three: all of them): planes
//    made beforehand cost a launch, 3 to 4 us, and no fewer bytes.  Up to 8
//    rows two planes lie side by side in the 16 columns of one operand.
//  - The four waves split the columns, 64 at a time.  A wave's pipeline is its
//    own, without barriers: whole 128-byte lines of its rows go from memory
//    straight to its part of the LDS (no registers), BUFS steps ahead, 64 to
//    128 KB per compute unit in flight.  Piece c of row r lies at slot
//    c ^ (r mod 8), so the operand reads are free of bank conflicts.  Blocks
//    start at different columns (8192 x 28672 dense: 171 us when all start
//    alike, 162 rotated: rows a power of two apart share channels).
//  - A block owns the fused kernel's neuron range: gate tiles first, then
//    the block's active neurons, listed in order, as up tiles; DENSE takes a
//    neuron's gate and up tile in the same step (x is then read once).
#include "stream.hpp"
#include "internal.hpp"

namespace cats {

typedef __bf16 gu_bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 gu_bf16x2 __attribute__((ext_vector_type(2)));

constexpr int kGuCols = 64;  // columns of a step (one 128-byte line per weight row)
static_assert(kFusedMaxNeurons <= 4 * kWaveSize, "one thread per neuron in the compaction");

// Two values as bf16, nearest, the first in the low half.
__device__ __forceinline__ uint32_t pack_nearest(float a, float b) {
  const gu_bf16x2 v = {(__bf16)a, (__bf16)b};
  return __builtin_bit_cast(uint32_t, v);
}
// The upper halves of two fp32 values, the first in the low half.
__device__ __forceinline__ uint32_t pack_cut(float a, float b) {
  return __builtin_amdgcn_perm(__float_as_uint(b), __float_as_uint(a), 0x07060302u);
}
__device__ __forceinline__ float cut(float f) { return __uint_as_float(__float_as_uint(f) & 0xffff0000u); }

// Geometry for T tiles a step, x as NS planes, up to XR rows.
template <int T, int NS, int XR>
struct GuGeom {
  // Waves of a block: two per SIMD where the LDS holds enough steps for that
  // (a wave with one or two tiles spends its steps on splitting x, one after
  // the other: 3584 x 5000 at 8 rows 26.2 us with four waves, 18.5 with eight).
  static constexpr int W = T <= 2 ? 8 : 4;
  static constexpr int THREADS = W * kWaveSize;
  // plane p of row b is column (p XR + b) % 16 of operand (p XR + b) / 16
  static constexpr int F = (NS * XR + 15) / 16;
  static constexpr int COLS = 16 / XR;                      // planes side by side in an operand
  static constexpr int XI = XR / 4;                         // x loads of a step (4 rows of 256 bytes each)
  static constexpr int WB = T * 2048 + XI * 1024;           // LDS bytes of a wave and step
  static constexpr int SB = W * WB;
  static constexpr int OPS = 2 * T + XI;
  static constexpr int BUFS = 144 * 1024 / SB;              // steps in LDS at once
  // neurons of a block: up to three tiles a step one round, four tiles two at
  // most (gateup_tiles)
  static constexpr int VROWS = T < 4 ? 16 * T : (T == 4 ? 128 : kFusedMaxNeurons);
  static_assert(BUFS >= 2 && BUFS <= 4 && (BUFS - 1) * OPS < 64, "two to four steps, and vmcnt is six bits");
};

// STREAM: the weights are read with the non-temporal policy.
template <int T, int NS, int XR, bool DENSE, bool STREAM>
__global__ __launch_bounds__((GuGeom<T, NS, XR>::THREADS)) void k_mlp_gateup(GateUpArgs a) {
  typedef GuGeom<T, NS, XR> G;
  constexpr int W = G::W;
  constexpr int BUFS = G::BUFS, F = G::F, SB = G::SB;
  constexpr int NT = DENSE ? T / 2 : T;  // neuron tiles of a round
  static_assert(!DENSE || T % 2 == 0, "a dense step holds gate and up tiles");
  __shared__ float l_ss[W][16], l_scale[16];
  // one array per step in flight, so that the compiler sees which loads a
  // read depends on
  __shared__ __attribute__((aligned(1024))) uint8_t s0[SB], s1[SB];
  __shared__ __attribute__((aligned(1024))) uint8_t s2[BUFS > 2 ? SB : 16], s3[BUFS > 3 ? SB : 16];
  __shared__ float l_v[DENSE ? 1 : G::VROWS][XR];
  __shared__ uint32_t l_mask[DENSE ? 1 : G::VROWS];
  __shared__ int l_act[DENSE ? 1 : G::VROWS];  // the block's active neurons, ascending
  __shared__ int w_cnt[W];

  const int tid = threadIdx.x, lane = tid & (kWaveSize - 1);
  const int w = __builtin_amdgcn_readfirstlane(tid / kWaveSize);
  const int B = a.B, d = a.d, m = a.m;
  const int blk = blockIdx.x, grid = gridDim.x;
  const int n0 = (int)(((int64_t)blk * m) / grid);
  const int nb = (int)(((int64_t)(blk + 1) * m) / grid) - n0;
  const uint32_t row_bytes = (uint32_t)d * 2u;
  const uint32_t mat_bytes = (uint32_t)((uint64_t)m * row_bytes);
  const __amdgpu_buffer_rsrc_t rg = make_rsrc(a.wg, mat_bytes);
  const __amdgpu_buffer_rsrc_t ru = make_rsrc(a.wu, mat_bytes);
  const __amdgpu_buffer_rsrc_t rx = make_rsrc(a.x, (uint32_t)(B * d * sizeof(float)));
  // this wave's 64-column steps, and where in them it starts
  const int chunks = (d + kGuCols - 1) / kGuCols;
  const int c0 = (chunks * w) / W, c1 = (chunks * (w + 1)) / W;
  const int rot = c1 > c0 ? ((blk >> 3) * 5) % (c1 - c0) : 0;

  // loader: instruction (tile, half) takes 8 rows of 128 bytes, lane l the
  // piece (l % 8) ^ (l / 8) of row l / 8
  const int lr = lane >> 3;
  const int lcol = ((lane & 7) ^ lr) * 8;
  // operands: lane = row r16 (A) or column (B), k = 8 kb .. + 7 of 32
  const int r16 = lane & 15, kb = lane >> 4;
  const int rd0 = w * G::WB + r16 * 128 + ((kb ^ (r16 & 7)) * 16);
  const int rd1 = w * G::WB + r16 * 128 + (((4 + kb) ^ (r16 & 7)) * 16);
  // x: lane l of load i takes 16 bytes of row 4 i + l / 16, piece (l % 16) ^
  // (row % 8) of the row's 256; column r16 of an operand reads row r16 % XR
  uint32_t xoff[G::XI];
  int xcol[G::XI];
#pragma unroll
  for (int i = 0; i < G::XI; ++i) {
    const int r = 4 * i + (lane >> 4);
    xcol[i] = ((lane & 15) ^ (r & 7)) * 4;
    xoff[i] = r < B ? (uint32_t)(r * d + xcol[i]) * 4u : kOOB;
  }
  const int xb = r16 % XR;  // row of this lane's column; pm: its plane among those side by side
  const uint32_t pm[2] = {r16 / XR == 0 ? ~0u : 0u, r16 / XR == 1 ? ~0u : 0u};
  const int xrd = w * G::WB + T * 2048 + xb * 256;

  // Sums of the first operand's products (even and odd halves of a step) and
  // of the others', added once at the end: shorter chains round less.
  f32x4 acc[T][2], acl[T];
  float ss = 0.f;  // squares of this lane's x values (row xb), for the RMSNorm factor
  // One pass of this wave over its columns: rb[2 t + i] is the byte offset of
  // the row that this lane loads for half i of tile t (kOOB: no such row).
  // up(t): tile t comes from W_up.  sq: add up the squares of x.
  auto pass = [&](const uint32_t(&rb)[2 * T], auto up, bool sq) {
    auto issue = [&](uint8_t* s, int ci) {
      const bool on = ci < c1;
      int c = ci + rot;
      if (c >= c1) c -= c1 - c0;
      // out of range by addition, not by a choice of offsets, which the
      // compiler would make a branch with loads on both sides
      const uint32_t out = on ? 0u : kOOB;
      const uint32_t off = out + (uint32_t)(c * kGuCols + lcol) * 2u + (c * kGuCols + lcol < d ? 0u : kOOB);
#pragma unroll
      for (int t = 0; t < T; ++t)
#pragma unroll
        for (int i = 0; i < 2; ++i)
          dma16<STREAM ? 2 /* nt */ : 0>(up(t) ? ru : rg, s + w * G::WB + t * 2048 + i * 1024, rb[2 * t + i] + off);
#pragma unroll
      for (int i = 0; i < G::XI; ++i)
        dma16(rx, s + w * G::WB + T * 2048 + i * 1024,
              out + xoff[i] + (uint32_t)c * (kGuCols * 4u) + (c * kGuCols + xcol[i] < d ? 0u : kOOB));
    };
    // Step c of buffer s, with the loads of LEFT later steps outstanding;
    // MORE: the buffer then takes the loads of step c + BUFS.
    auto step = [&](uint8_t* s, int c, auto left, auto more) {
      wait_vm<decltype(left)::v * G::OPS>();
      gu_bf16x8 av[T][2];
      f32x4 xv[2][2];
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int e = 0; e < 2; ++e)
          xv[h][e] = *reinterpret_cast<const f32x4*>(s + xrd + (((8 * h + 2 * kb + e) ^ (xb & 7)) * 16));
#pragma unroll
      for (int t = 0; t < T; ++t) {
        av[t][0] = *reinterpret_cast<const gu_bf16x8*>(s + t * 2048 + rd0);
        av[t][1] = *reinterpret_cast<const gu_bf16x8*>(s + t * 2048 + rd1);
      }
      // this lane's column of the operands: planes of eight values
      u32x4 bx[2][F];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const float f[8] = {xv[h][0].x, xv[h][0].y, xv[h][0].z, xv[h][0].w, xv[h][1].x, xv[h][1].y, xv[h][1].z, xv[h][1].w};
        if (sq) {
#pragma unroll
          for (int e = 0; e < 8; ++e) ss = fmaf(f[e], f[e], ss);
        }
        if constexpr (NS == 2) {
          uint32_t hi[4], lo[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            hi[e] = pack_nearest(f[2 * e], f[2 * e + 1]);
            lo[e] = pack_nearest(f[2 * e] - __uint_as_float(hi[e] << 16),
                                 f[2 * e + 1] - __uint_as_float(hi[e] & 0xffff0000u));
          }
          if constexpr (F == 1) {
#pragma unroll
            for (int e = 0; e < 4; ++e) bx[h][0][e] = (hi[e] & pm[0]) | (lo[e] & pm[1]);
          } else {
            bx[h][0] = u32x4{hi[0], hi[1], hi[2], hi[3]};
            bx[h][1] = u32x4{lo[0], lo[1], lo[2], lo[3]};
          }
        } else {
          // plane 0 is f cut to 8 bits, plane 1 the rest cut, plane 2 what
          // is left then
          uint32_t p0[4], p1[4], p2[4];
          float zero = 0.f;  // NaN where a value is infinite or NaN
#pragma unroll
          for (int e = 0; e < 8; ++e) zero = fmaf(f[e], 0.f, zero);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float u1 = f[2 * e] - cut(f[2 * e]), v1 = f[2 * e + 1] - cut(f[2 * e + 1]);
            p0[e] = pack_cut(f[2 * e], f[2 * e + 1]);
            p1[e] = pack_cut(u1, v1);
            p2[e] = pack_cut(u1 - cut(u1), v1 - cut(v1));
          }
          if (__any(zero != 0.f)) {  // an infinity or NaN is its first plane alone, a NaN quiet
#pragma unroll
            for (int e = 0; e < 8; ++e) {
              const uint32_t u = __float_as_uint(f[e]), half = e & 1 ? 0xffff0000u : 0x0000ffffu;
              if ((u & 0x7f800000u) == 0x7f800000u) {
                if (u & 0x007fffffu) p0[e / 2] |= 0x00400040u & half;
                p1[e / 2] &= ~half;
                p2[e / 2] &= ~half;
              }
            }
          }
          // (by masks: choices between planes become branches)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            if constexpr (XR == 8) {
              bx[h][0][e] = (p0[e] & pm[0]) | (p1[e] & pm[1]);
              bx[h][1][e] = p2[e] & pm[0];
            } else {
              bx[h][0][e] = p0[e];
              bx[h][1][e] = p1[e];
              bx[h][2][e] = p2[e];
            }
          }
        }
      }
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int f = 0; f < F; ++f)
#pragma unroll
          for (int t = 0; t < T; ++t)
            if (f == 0)
              acc[t][h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[t][h], __builtin_bit_cast(gu_bf16x8, bx[h][f]), acc[t][h], 0, 0, 0);
            else
              acl[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[t][h], __builtin_bit_cast(gu_bf16x8, bx[h][f]), acl[t], 0, 0, 0);
      if constexpr (decltype(more)::v) {
        wait_lds();  // the operand reads are done before the buffer is loaded again
        __builtin_amdgcn_sched_barrier(0);
        issue(s, c + BUFS);
      }
    };
#pragma unroll
    for (int t = 0; t < T; ++t) acc[t][0] = acc[t][1] = acl[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    int c = c0;
    if (c < c1) {
      issue(s0, c);
      issue(s1, c + 1);
      if constexpr (BUFS > 2) issue(s2, c + 2);
      if constexpr (BUFS > 3) issue(s3, c + 3);
      // whole rounds of the buffers in a loop without exits (with one after
      // each step the compiler loses count at the loop's head and waits for
      // every load there), then the last steps: fewer than the buffers, but
      // without the last of these branches, which is never taken, the same
      // loop takes longer (gate/up at 5120 x 13824, 16 rows, 53.0 us, with it 52.6)
      for (; c + BUFS <= c1; c += BUFS) {
        constexpr Const<BUFS - 1> left;
        constexpr Const<1> more;
        step(s0, c, left, more);
        step(s1, c + 1, left, more);
        if constexpr (BUFS > 2) step(s2, c + 2, left, more);
        if constexpr (BUFS > 3) step(s3, c + 3, left, more);
      }
      constexpr Const<0> last;
      if (c < c1) step(s0, c, Const<BUFS - 1>(), last);
      if (c + 1 < c1) step(s1, c + 1, Const<BUFS - 2>(), last);
      if constexpr (BUFS > 2) { if (c + 2 < c1) step(s2, c + 2, Const<BUFS - 3>(), last); }
      if constexpr (BUFS > 3) { if (c + 3 < c1) step(s3, c + 3, Const<BUFS - 4>(), last); }
    }
    wait_vm<0>();  // no load is on its way to LDS any more
    wait_lds();
    __syncthreads();                     // nor any other wave's
    f32x4* red = reinterpret_cast<f32x4*>(s0);
    if constexpr (NS == 3) {
      f32x4 first[T];
#pragma unroll
      for (int t = 0; t < T; ++t) first[t] = acc[t][0] + acc[t][1];
      add_lower_planes(first, acl);
#pragma unroll
      for (int t = 0; t < T; ++t) red[(w * T + t) * kWaveSize + lane] = acl[t];
    } else {
#pragma unroll
      for (int t = 0; t < T; ++t) red[(w * T + t) * kWaveSize + lane] = (acc[t][0] + acc[t][1]) + acl[t];
    }
    if (sq) {
      // the four lanes of a row, then the waves, in a fixed order
      float q = ss + __shfl_xor(ss, 16);
      q = q + __shfl_xor(q, 32);
      if (lane < 16) l_ss[w][lane] = q;
      __syncthreads();
      if (tid < 16) {
        float tot = 0.f;
#pragma unroll
        for (int k = 0; k < W; ++k) tot += l_ss[k][tid];
        l_scale[tid] = 1.f / sqrtf(tot / (float)d + a.eps);
      }
    }
    __syncthreads();
  };
  // Dot product of row i of tile t with row b of x: D[i][j] sits in lane
  // j + 16 (i / 4), register i % 4; the waves' parts in wave order, the
  // columns that hold row b's planes in plane order.
  auto dot = [&](int t, int i, int b) -> float {
    const float* red = reinterpret_cast<const float*>(s0);
    float sum = 0.f, first = 0.f;
#pragma unroll
    for (int p = 0; p < G::COLS; ++p) {
#pragma unroll
      for (int k = 0; k < W; ++k)
        sum += red[((k * T + t) * kWaveSize + p * XR + b + 16 * (i >> 2)) * 4 + (i & 3)];
      if (p == 0) first = sum;
    }
    if (NS == 3 && !is_finite(first)) sum = first;  // as in add_lower_planes
    return a.norm ? sum * l_scale[b] : sum;
  };

  int nact = nb;
  if constexpr (DENSE) {
    const uint32_t all = (1u << B) - 1u;
    for (int r0 = 0; r0 < nb; r0 += 16 * NT) {
      uint32_t rb[2 * T];
#pragma unroll
      for (int t = 0; t < T; ++t)
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const int loc = r0 + 16 * (t % NT) + 8 * i + lr;
          rb[2 * t + i] = loc < nb ? (uint32_t)(n0 + loc) * row_bytes : kOOB;
        }
      pass(rb, [](int t) { return t >= NT; }, a.norm && r0 == 0);
      const int i = tid & 15, b = tid >> 4;
      if (b < B) {
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          const int loc = r0 + 16 * t + i;
          if (loc < nb) {
            const float v = silu(dot(t, i, b));
            a.seg_h[(size_t)b * m + n0 + loc] = v * dot(NT + t, i, b);
          }
        }
      }
      __syncthreads();  // the sums are overwritten by the next round
    }
    if (tid < nb) {
      a.seg_j[n0 + tid] = n0 + tid;
      a.seg_mask[n0 + tid] = all;
    }
  } else {
    for (int r0 = 0; r0 < nb; r0 += 16 * T) {
      uint32_t rb[2 * T];
#pragma unroll
      for (int t = 0; t < T; ++t)
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const int loc = r0 + 16 * t + 8 * i + lr;
          rb[2 * t + i] = loc < nb ? (uint32_t)(n0 + loc) * row_bytes : kOOB;
        }
      pass(rb, [](int) { return false; }, a.norm && r0 == 0);
      const int i = tid >> 4, b = tid & 15;  // (i < 16: the first four waves)
#pragma unroll
      for (int t = 0; t < T; ++t) {
        const int loc = r0 + 16 * t + i;
        bool keep = false;
        if (i < 16 && loc < nb && b < B) {
          const float v = silu(dot(t, i, b));
          l_v[loc][b] = v;
          keep = !(fabsf(v) < a.t);
        }
        const uint64_t bal = __ballot(keep);
        if (b == 0 && i < 16 && loc < nb) l_mask[loc] = (uint32_t)(bal >> (lane & 48)) & 0xffffu;
      }
      __syncthreads();
    }
    // the block's active neurons in order
    const bool on = tid < nb && l_mask[tid] != 0u;
    const uint64_t bal = __ballot(on);
    if (lane == 0) w_cnt[w] = __popcll(bal);
    __syncthreads();
    int pos = __popcll(bal & ((1ull << lane) - 1ull));
    nact = 0;
#pragma unroll
    for (int k = 0; k < W; ++k) {
      if (k < w) pos += w_cnt[k];
      nact += w_cnt[k];
    }
    if (on) {
      l_act[pos] = tid;
      a.seg_j[n0 + pos] = n0 + tid;
      a.seg_mask[n0 + pos] = l_mask[tid];
    }
    __syncthreads();
    for (int r0 = 0; r0 < nact; r0 += 16 * T) {
      uint32_t rb[2 * T];
#pragma unroll
      for (int t = 0; t < T; ++t)
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const int e = r0 + 16 * t + 8 * i + lr;
          rb[2 * t + i] = e < nact ? (uint32_t)(n0 + l_act[e]) * row_bytes : kOOB;
        }
      pass(rb, [](int) { return true; }, false);
      const int i = tid & 15, b = tid >> 4;
      if (b < B) {
#pragma unroll
        for (int t = 0; t < T; ++t) {
          const int e = r0 + 16 * t + i;
          if (e < nact) {
            const int loc = l_act[e];
            const float v = l_v[loc][b];
            a.seg_h[(size_t)b * m + n0 + e] = ((l_mask[loc] >> b) & 1u) ? v * dot(t, i, b) : 0.f;
            if (a.aux) a.seg_v[(size_t)b * m + n0 + e] = v;
          }
        }
      }
      __syncthreads();
    }
    // the rest of the block's segment names no neuron: zero row masks, so a
    // list entry is exactly an entry with its row's bit set
    if (tid >= nact && tid < nb) a.seg_mask[n0 + tid] = 0u;
  }
  if (tid == 0) a.seg_cnt[blk] = nact;
}

template <int T, bool DENSE>
static hipError_t launch_gateup_t(int planes, const GateUpArgs& a, int G, hipStream_t s) {
  KernelTimer timer(DENSE ? "mlp_gateup_dense" : "mlp_gateup_cats", s);
  const dim3 grid(G), block(GuGeom<T, 2, 8>::THREADS);
#define CATS_GU(TT, NS, XR, STREAM) \
  hipExtLaunchKernelGGL((k_mlp_gateup<TT, NS, XR, DENSE, STREAM>), grid, block, 0, s, timer.start(), timer.stop(), 0, a)
  // Non-temporal reads for rows of whole lines in blocks that the 256 MB
  // last-level cache cannot hold two of.  From memory they are 5 to 10%
  // faster (4096 x 11008 dense at 16 rows 37.0 us cached, 32.4 so; 24 blocks of
  // 2048 x 5632 in turn 29.7 / 28.3 a call), from that cache 7% slower (three
  // such blocks in turn 25.5 / 27.9; a larger block called again and again by
  // itself, of which k = 0.9 leaves the cache little to hold: 2048 x 28672 at 9
  // rows 58 / 61); where lines straddle rows and steps they fetch them twice
  // (2856 x 7001 at 11 rows 22.2 / 28.1).
  const bool stream = a.d % 64 == 0 && (uint64_t)a.m * a.d * 6 >= (144ull << 20);
  if (a.B <= 8) {
    if (planes == 2 && stream) CATS_GU(T, 2, 8, true);
    else if (planes == 2) CATS_GU(T, 2, 8, false);
    else if (stream) CATS_GU(T, 3, 8, true);
    else CATS_GU(T, 3, 8, false);
  } else if constexpr (T <= 6) {  // (eight tiles and 16 rows of x leave no room for a second step)
    if (planes == 2 && stream) CATS_GU(T, 2, 16, true);
    else if (planes == 2) CATS_GU(T, 2, 16, false);
    else if (stream) CATS_GU(T, 3, 16, true);
    else CATS_GU(T, 3, 16, false);
  } else {
    return hipErrorInvalidValue;
  }
#undef CATS_GU
  return hipGetLastError();
}

// Tiles of a step: the fewest rounds over the block's neurons that eight (up to
// 8 rows) or six tiles a step allow, and of the steps that need no more rounds
// the smallest, whose pipeline is deeper and which multiplies fewer missing
// tiles.  A dense step holds gate and up tiles.  us a call with steps as large as
// they go / so: 28672 neurons (seven tiles) at 9 rows, k = 0.5: 1024 columns 53 / 47,
// 4096 columns 138 / 123; dense 20000 neurons (five) at 4 rows of 4096 columns
// 96 / 88, 14336 neurons (four) at 9 rows of 5120 columns 92 / 85.
int gateup_tiles(int m, int B, bool dense) {
  const int G = fused_grid(m);
  const int tiles = ((m + G - 1) / G + 15) / 16;  // of the largest block
  const int most = (B > 8 ? 6 : 8) / (dense ? 2 : 1);
  const int rounds = (tiles + most - 1) / most;
  const int per = (tiles + rounds - 1) / rounds;
  if (dense) return 2 * per;
  return per == 5 ? 6 : (per == 7 ? 8 : per);
}

hipError_t launch_gateup(bool dense, int planes, const GateUpArgs& a, int G, hipStream_t s) {
  if (planes == 2 && gateup_narrow(a.d, a.m, dense)) return launch_gateup_narrow(dense, a, G, s);
  const int T = gateup_tiles(a.m, a.B, dense);
  if (dense) {
    if (T == 2) return launch_gateup_t<2, true>(planes, a, G, s);
    if (T == 4) return launch_gateup_t<4, true>(planes, a, G, s);
    if (T == 6) return launch_gateup_t<6, true>(planes, a, G, s);
    return launch_gateup_t<8, true>(planes, a, G, s);
  }
  if (T == 1) return launch_gateup_t<1, false>(planes, a, G, s);
  if (T == 2) return launch_gateup_t<2, false>(planes, a, G, s);
  if (T == 3) return launch_gateup_t<3, false>(planes, a, G, s);
  if (T == 4) return launch_gateup_t<4, false>(planes, a, G, s);
  if (T == 6) return launch_gateup_t<6, false>(planes, a, G, s);
  return launch_gateup_t<8, false>(planes, a, G, s);
}

}  // namespace cats
