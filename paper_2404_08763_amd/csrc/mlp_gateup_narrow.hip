// Gate and up projections of a batch (5..16 rows, bf16 weights) of narrow
// blocks of many neurons (d = 512, 1024 or 2048; gateup_narrow): x stays in
// registers.
//
// What bounds it: latency.  A tile of 16 neurons is 16 to 64 KB of weights,
// and k_mlp_gateup, whose waves stream columns, has one to four steps of 64
// columns per wave and pass there, so it fills and drains its pipeline more
// than it streams.  Here 16 waves hold one sixteenth of the columns each as
// matrix-core operands (x = hi + lo, both bf16: 16 of its 24 significand bits,
// products exact, fp32 accumulation), a tile is KS matrix instructions deep per
// wave and plane, and the next tile's loads are in flight while a tile is
// multiplied and the waves' parts are added in LDS, across the change from gate
// to up tiles as well.
//
// Measured (us a call, k_mlp_gateup / this kernel in front of the same
// down-projection and sum): 512 x 28672 at 9 / 16 rows, k = 0.5, 34.6 / 29.2
// and 35.9 / 30.5; dense at 16 rows 35.4 / 30.6; 1024 x 28672 at 16 rows
// 49.8 / 43.0; 512 x 8000 at 8 rows 19.3 / 18.2.
#include "stream.hpp"
#include "internal.hpp"

namespace cats {

typedef __bf16 gn_bf16x8 __attribute__((ext_vector_type(8)));

// Waves of a block: each holds 1/16 of x's columns.
constexpr int kGnWaves = 16;
constexpr int kGnThreads = kGnWaves * kWaveSize;
constexpr int kGnTile = 16;  // neurons per tile (and batch columns)

// Split 8 fp32 values into bf16 hi and lo parts, packed two per word
// (element 2i in the low half of word i, the order of a 16-byte bf16 load).
// Also adds the squares of the 8 values to ss (for the RMSNorm scale).
__device__ __forceinline__ void split8(const u32x4& a, const u32x4& b, gn_bf16x8& hi, gn_bf16x8& lo, float& ss) {
  const float f[8] = {__uint_as_float(a.x), __uint_as_float(a.y), __uint_as_float(a.z), __uint_as_float(a.w),
                      __uint_as_float(b.x), __uint_as_float(b.y), __uint_as_float(b.z), __uint_as_float(b.w)};
  uint32_t h[8], l[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    ss = fmaf(f[e], f[e], ss);
    h[e] = split2_plane(f[e], 0);
    l[e] = split2_plane(f[e], 1);
  }
  const u32x4 hv = {h[0] | (h[1] << 16), h[2] | (h[3] << 16), h[4] | (h[5] << 16), h[6] | (h[7] << 16)};
  const u32x4 lv = {l[0] | (l[1] << 16), l[2] | (l[3] << 16), l[4] | (l[5] << 16), l[6] | (l[7] << 16)};
  hi = __builtin_bit_cast(gn_bf16x8, hv);
  lo = __builtin_bit_cast(gn_bf16x8, lv);
}

// KS: steps of 32 columns per wave; the kernel covers d = 512 KS columns
// exactly, so no column needs a bounds check.
template <int KS, bool DENSE, bool AUX>
__global__ __launch_bounds__(kGnThreads) void k_mlp_gateup_narrow(GateUpArgs a) {
  constexpr int KW = 32 * KS;  // columns per wave
  constexpr int NBMAX = kFusedMaxNeurons;

  __shared__ f32x4 red[kGnWaves * kWaveSize];   // the waves' partial tiles
  __shared__ float l_v[NBMAX][kGnTile];         // v of each local neuron and row
  __shared__ float l_h[NBMAX][kGnTile];         // h (0 where the row masks it)
  __shared__ uint32_t l_mask[NBMAX];            // bit b: row b keeps the neuron
  __shared__ int w_cnt[kGnWaves + 1];
  __shared__ float l_ss[kGnWaves][kGnTile];     // the waves' sums of squares per row
  __shared__ float l_scale[kGnTile];            // per-row factor on every dot product

  const int tid = threadIdx.x;
  const int lane = tid & (kWaveSize - 1);
  const int w = __builtin_amdgcn_readfirstlane(tid / kWaveSize);
  const int B = a.B, d = a.d, m = a.m;
  const float t = a.t;
  const int G = gridDim.x, blk = blockIdx.x;
  const int n0 = (int)(((int64_t)blk * m) / G);
  const int nb = (int)(((int64_t)(blk + 1) * m) / G) - n0;
  const int T = (nb + kGnTile - 1) / kGnTile;  // tiles (two at least: gateup_narrow)
  const int nops = 2 * T;                      // gate tiles, then up tiles

  const uint32_t row_bytes = (uint32_t)d * 2u;
  const uint32_t mat_bytes = (uint32_t)((uint64_t)m * row_bytes);
  const __amdgpu_buffer_rsrc_t rg = make_rsrc(a.wg, mat_bytes);
  const __amdgpu_buffer_rsrc_t ru = make_rsrc(a.wu, mat_bytes);

  for (int i = tid; i < nb; i += kGnThreads) l_mask[i] = 0u;

  // This lane's operand coordinates: A row (neuron in tile) = lane % 16,
  // B column (batch row) = lane % 16, and 8 consecutive k at 8 * (lane / 16)
  // within each 32-column step.
  const int r16 = lane & 15;
  const int kb = lane >> 4;
  const int cw0 = w * KW + kb * 8;

  const uint32_t colb = (uint32_t)cw0 * 2u;  // this lane's byte offset in a weight row
  __syncthreads();  // l_mask cleared

  // Row base of this lane's neuron in operation `op` (kOOB where the row is
  // not read: past the block's neurons, past the last operation, or an up
  // row no batch row keeps).
  auto row_of = [&](int op) -> uint32_t {
    const bool up = op >= T;
    const int i = (up ? op - T : op) * kGnTile + r16;
    bool ok = op < nops && i < nb;
    if (!DENSE && up && ok) ok = l_mask[i] != 0u;
    return ok ? (uint32_t)(n0 + i) * row_bytes : kOOB;
  };

  // ---- x slice of this wave as hi/lo bf16 fragments (rows past B are zero)
  gn_bf16x8 xh[KS], xl[KS];
  float ss = 0.f;  // sum of squares of this lane's x values (row r16)
  {
    const __amdgpu_buffer_rsrc_t rx = make_rsrc(a.x, (uint32_t)(B * d * sizeof(float)));
    const uint32_t xrow = r16 < B ? (uint32_t)(r16 * d + cw0) * 4u : kOOB;
    u32x4 wa[KS], wb[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      wa[s] = ld_buf16(rx, xrow + s * 128u);
      wb[s] = ld_buf16(rx, xrow + s * 128u + 16u);
    }
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      split8(wa[s], wb[s], xh[s], xl[s], ss);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  // Per-row factor on the gate and up dot products: 1, or the RMSNorm scale
  // 1/sqrt(mean(x^2) + eps) when the block is normalised in front (the sum
  // of squares in a fixed order: lane, then the four lanes of a row in
  // ascending order, then the waves in order).
  if (a.norm) {
    float s4 = ss + __shfl_xor(ss, 16);
    s4 = s4 + __shfl_xor(s4, 32);
    if (lane < kGnTile) l_ss[w][lane] = s4;
    __syncthreads();
    if (tid < kGnTile) {
      float tot = 0.f;
#pragma unroll
      for (int ww = 0; ww < kGnWaves; ++ww) tot += l_ss[ww][tid];
      l_scale[tid] = 1.f / sqrtf(tot / (float)d + a.eps);
    }
  } else if (tid < kGnTile) {
    l_scale[tid] = 1.f;
  }
  // Weight loads here are ordinary cached loads, not the non-temporal ones of
  // the other weight streams: one load instruction reads 64 bytes of each
  // of 16 rows, half of a 128-byte line, and the line's other half comes
  // with the next step; with the non-temporal hint the line was often gone
  // before its second half was asked for.
  // The first gate tile's weights go out only now: issued before the x
  // fragments are built, they would sit in registers the fragments need,
  // and the compiler parks them elsewhere one load round trip at a time.
  // buf[s] holds step s of the current tile, and is loaded with step s of the
  // next one step after its products have read it.
  u32x4 buf[KS];
  {
    const uint32_t rb0 = row_of(0);
#pragma unroll
    for (int s = 0; s < KS; ++s) buf[s] = ld_buf16(rg, rb0 + colb + s * 64u);
  }
  __syncthreads();

  for (int op = 0; op < nops; ++op) {
    // The up tile of neuron tile i needs tile i's masks, known once gate
    // tile i is reduced: with two tiles and more, before this operation.
    const uint32_t rbn = row_of(op + 1);
    const __amdgpu_buffer_rsrc_t rn = (op + 1 < T) ? rg : ru;
    // Four independent accumulators (hi and lo products of even and odd
    // steps) keep the matrix core pipelined instead of waiting on one chain;
    // they are added in a fixed order at the end.
    f32x4 ah0 = {0.f, 0.f, 0.f, 0.f}, ah1 = ah0, al0 = ah0, al1 = ah0;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      const gn_bf16x8 av = __builtin_bit_cast(gn_bf16x8, buf[s]);
      if (s & 1) {
        ah1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, xh[s], ah1, 0, 0, 0);
        al1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, xl[s], al1, 0, 0, 0);
      } else {
        ah0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, xh[s], ah0, 0, 0, 0);
        al0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, xl[s], al0, 0, 0, 0);
      }
      if (s >= 1) buf[s - 1] = ld_buf16(rn, rbn + colb + (s - 1) * 64u);
      __builtin_amdgcn_sched_barrier(0);
    }
    buf[KS - 1] = ld_buf16(rn, rbn + colb + (KS - 1) * 64u);
    const f32x4 acc = (ah0 + ah1) + (al0 + al1);
    red[w * kWaveSize + lane] = acc;
    __syncthreads();
    if (tid < kGnTile * kGnTile) {
      // D[i][j] sits in lane j + 16 (i / 4), register i % 4
      const int i = tid >> 4, jb = tid & 15;
      const int src = jb + 16 * (i >> 2), reg = i & 3;
      float sum = 0.f;
#pragma unroll
      for (int ww = 0; ww < kGnWaves; ++ww) sum += red[ww * kWaveSize + src][reg];
      sum *= l_scale[jb];
      const bool up = op >= T;
      const int li = (up ? op - T : op) * kGnTile + i;
      if (li < nb && jb < B) {
        if (!up) {
          const float v = silu(sum);
          l_v[li][jb] = v;
          if (DENSE || !(fabsf(v) < t)) atomicOr(&l_mask[li], 1u << jb);
        } else {
          l_h[li][jb] = ((l_mask[li] >> jb) & 1u) ? l_v[li][jb] * sum : 0.f;
        }
      }
    }
    __syncthreads();
  }

  // ---- ordered compaction of the block's union-active neurons
  int base = 0;
  for (int p = 0; p * kGnThreads < nb; ++p) {
    const int loc = p * kGnThreads + tid;
    const uint32_t mk = loc < nb ? l_mask[loc] : 0u;
    const uint64_t bal = __ballot(mk != 0u);
    if (lane == 0) w_cnt[w] = __popcll(bal);
    __syncthreads();
    if (tid == 0) {
      int run = 0;
      for (int k = 0; k < kGnWaves; ++k) {
        const int c = w_cnt[k];
        w_cnt[k] = run;
        run += c;
      }
      w_cnt[kGnWaves] = run;
    }
    __syncthreads();
    if (mk) {
      const int pos = base + w_cnt[w] + __popcll(bal & ((1ull << lane) - 1ull));
      const size_t o = (size_t)n0 + pos;
      a.seg_j[o] = n0 + loc;
      a.seg_mask[o] = mk;
      for (int b = 0; b < B; ++b) {
        a.seg_h[(size_t)b * m + o] = l_h[loc][b];
        if constexpr (AUX) a.seg_v[(size_t)b * m + o] = l_v[loc][b];
      }
    }
    base += w_cnt[kGnWaves];
    __syncthreads();
  }
  if (tid == 0) a.seg_cnt[blk] = base;
  // the rest of the block's segment names no neuron: zero row masks, so a
  // list entry is exactly an entry with its row's bit set
  for (int i = base + tid; i < nb; i += kGnThreads) a.seg_mask[n0 + i] = 0u;
}

template <int KS, bool DENSE, bool AUX>
static hipError_t launch_narrow_t(const GateUpArgs& a, int G, hipStream_t s) {
  KernelTimer timer(DENSE ? "mlp_gateup_narrow_dense" : "mlp_gateup_narrow_cats", s);
  hipExtLaunchKernelGGL((k_mlp_gateup_narrow<KS, DENSE, AUX>), dim3(G), dim3(kGnThreads), 0, s, timer.start(),
                        timer.stop(), 0, a);
  return hipGetLastError();
}

// Where it is the faster one of the two (us a call, k_mlp_gateup / this
// kernel).  CATS: 512 x 3000 at 5 rows 15.4 / 15.7, 512 x 5632 at 8 rows
// 18.4 / 17.6; 1024 x 5632 at 5 rows 19.3 / 19.9, 1024 x 8000 at 9 rows
// 23.6 / 22.5; 2048 x 28672 at 5 / 16 rows 67.7 / 70.0 and 72.4 / 74.9, above
// eight tiles of neurons a block 2048 x 34000 at 16 rows, k = 0.9, 86.2 / 80.7.
// Dense, where k_mlp_gateup has no change from gate to up: 512 x 11008 at 8
// rows 19.3 / 19.5, 512 x 13824 at 16 rows 22.8 / 22.7; 1024 x 11008 at 5 rows
// 24.0 / 23.8, 1024 x 18000 at 8 rows 33.0 / 31.0.
bool gateup_narrow(int d, int m, bool dense) {
  if (dense) return (d == 512 || d == 1024) && m > 12288;
  return (d == 512 && m >= 5000) || (d == 1024 && m >= 8000) || (d == 2048 && m > 32768);
}

hipError_t launch_gateup_narrow(bool dense, const GateUpArgs& a, int G, hipStream_t s) {
  if (dense) return a.d == 512 ? launch_narrow_t<1, true, false>(a, G, s) : launch_narrow_t<2, true, false>(a, G, s);
  if (a.d == 512) return a.aux ? launch_narrow_t<1, false, true>(a, G, s) : launch_narrow_t<1, false, false>(a, G, s);
  if (a.d == 1024) return a.aux ? launch_narrow_t<2, false, true>(a, G, s) : launch_narrow_t<2, false, false>(a, G, s);
  return a.aux ? launch_narrow_t<4, false, true>(a, G, s) : launch_narrow_t<4, false, false>(a, G, s);
}

}  // namespace cats
