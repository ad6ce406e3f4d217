// Many-row products on the matrix cores, for the calibration (N vectors at
// once): the gate activations, the gate and up projections of a dense block
// together, and its down-projection.  bf16 weights; the fp32 operand enters
// as NS bf16 planes made once by k_rows_split (NS = 2: hi + lo, 16 of its 24
// significand bits, each product exact; NS = 3: all 24 bits).
//
// What bounds it: the matrix cores.  A product is 2 NS N d m operations on
// operands that fit the caches (C2 with 2048 vectors: 370 GFLOP, 90 MB of
// weights).  A block of four waves owns 256 output rows (neurons or columns)
// x 128 vectors, a wave 128 x 64 of them as 8 x 4 tiles of 16 x 16, so that a
// step of 32 k reads 16 KB of operands from LDS per wave for 64 NS / 2
// products (half of what the LDS delivers in the time the products take;
// 64 x 64 per wave needs three quarters).  Two blocks fit a compute unit, so one
// block's barrier and operand reads run under the other's products.  The
// operands go from memory straight to LDS (no registers, no VALU work), the
// next step's while the current one is multiplied: one barrier per step.
// Splitting x beforehand matters most: split inside the product, every block
// of neurons converts the same vectors again (43 times at C2).
// C2 with 2048 vectors (d = 4096, m = 11008): 310 us, 1.19 PFLOP/s counting both
// planes, where a torch bf16 product of that shape reaches 1.18 and the largest
// 1.46 (the 256 x 128 tiles that split x per block: 618 us).  The order of LDS
// reads and products, wave priority and 512 blocks against 688 tiles were
// within 2%.
#include "stream.hpp"
#include "internal.hpp"

namespace cats {

typedef __bf16 gr_bf16x8 __attribute__((ext_vector_type(8)));
typedef short gr_i16x4 __attribute__((ext_vector_type(4)));

constexpr int kGrN = kRowsTileN;  // vectors per block
constexpr int kGrK = 32;          // depth of a step (one matrix instruction)
constexpr int kGrThreads = 256;
constexpr int kGrXcds = 8;        // block b runs on XCD b mod 8

enum GrMode { kGrActs, kGrGateUp, kGrDown };

template <int NS>
__device__ __forceinline__ void split_planes(float f, uint16_t (&p)[NS]) {
#pragma unroll
  for (int i = 0; i < NS; ++i) p[i] = (uint16_t)(NS == 2 ? split2_plane(f, i) : split3_plane(f, i));
}

// Geometry of a block of TM output rows: its four waves, each wave's tiles
// and the steps whose operands are in LDS at once.  Two blocks fit a compute
// unit's 160 KB in every case.
template <int TM, int NS>
struct GrGeom {
  static constexpr int WM = TM == 64 ? 1 : 2;  // waves along the output rows
  static constexpr int WN = 4 / WM;            // along the vectors
  static constexpr int MI = TM / WM / 16;      // 16-row tiles of a wave
  static constexpr int NB = kGrN / WN / 16;    // 16-vector tiles of a wave
  static constexpr int BUFS = TM == 256 || NS == 3 ? 2 : (TM == 128 ? 3 : 4);
  static constexpr int WQ = TM / 64;           // weight loads of a wave and step
  static constexpr int LOADS = WQ + 2 * NS;    // all its loads of a step
};

template <int MODE, int NS, int TM>
__global__ __launch_bounds__(kGrThreads, 2) void k_rows_gemm(RowsGemmArgs a) {
  typedef GrGeom<TM, NS> G;
  constexpr int MI = G::MI, NB = G::NB;
  static_assert(MODE != kGrDown || TM == 256, "the transposing reads take 512-byte rows");
  constexpr int WB = TM * 64, XB = NS * kGrN * 64;  // LDS bytes of a step
  // one array per step in flight: the compiler then sees that a load into
  // one does not touch the operands read from another
  __shared__ __attribute__((aligned(1024))) uint8_t sw0[WB], sx0[XB], sw1[WB], sx1[XB];
  __shared__ __attribute__((aligned(1024))) uint8_t sw2[G::BUFS > 2 ? WB : 16], sx2[G::BUFS > 2 ? XB : 16];
  __shared__ __attribute__((aligned(1024))) uint8_t sw3[G::BUFS > 3 ? WB : 16], sx3[G::BUFS > 3 ? XB : 16];
  const int tid = threadIdx.x, lane = tid & (kWaveSize - 1);
  const int w = __builtin_amdgcn_readfirstlane(tid / kWaveSize);
  const int wm = w / G::WN, wn = w % G::WN;
  const int r16 = lane & 15, kb = lane >> 4;

  // Tile of this block: each XCD takes a consecutive run of tiles, vectors
  // fastest, so the blocks that share an L2 share rows of both operands.
  const int nt = a.MT * a.NT;  // tiles per part of the reduction
  const int total = nt * a.S;
  const int x = blockIdx.x % kGrXcds, ix = blockIdx.x / kGrXcds;
  const int per = total / kGrXcds, rem = total % kGrXcds;
  const int id = x * per + (x < rem ? x : rem) + ix;
  const int part = id / nt, tile = id - part * nt;
  const int mt = tile / a.NT, v0 = (tile - mt * a.NT) * kGrN;
  const int steps = (a.K + kGrK - 1) / kGrK;
  const int st0 = (int)(((int64_t)part * steps) / a.S), st1 = (int)(((int64_t)(part + 1) * steps) / a.S);

  const uint32_t row_bytes = (uint32_t)a.wcols * 2u;
  const uint32_t mat_bytes = (uint32_t)((uint64_t)a.wrows * row_bytes);
  const __amdgpu_buffer_rsrc_t rw0 = make_rsrc(a.w0, mat_bytes);
  const __amdgpu_buffer_rsrc_t rw1 = make_rsrc(MODE == kGrGateUp ? a.w1 : a.w0, mat_bytes);
  // the block's vectors: at most 128 rows of a plane
  const int nv = min(kGrN, a.N - v0);
  __amdgpu_buffer_rsrc_t rx[NS];
#pragma unroll
  for (int p = 0; p < NS; ++p)
    rx[p] = make_rsrc(a.xs + ((size_t)p * a.N + v0) * a.Kp, (uint32_t)nv * (uint32_t)a.Kp * 2u);

  // ---- loader coordinates.  A row of a step is 64 bytes (four 16-byte
  // pieces; 16 rows per instruction), piece c of row r stored at slot
  // c ^ ((r >> 1) & 3) so that a fragment's eight-lane groups hit distinct
  // banks.  W_down's step is 32 rows of 512 bytes (two per instruction), its
  // 32-byte pieces at slot c ^ (r % 4 + 4 (r / 8)), for the transposing reads.
  // Gate/up: the first half of each wave's rows is gate, the second the
  // same neurons' up rows.
  auto is_up = [&](int i) { return MODE == kGrGateUp && i % MI >= MI / 2; };
  uint32_t woff[G::WQ];
#pragma unroll
  for (int q = 0; q < G::WQ; ++q) {
    const int i = G::WQ * w + q;
    if constexpr (MODE == kGrDown) {
      const int r = 2 * i + (lane >> 5), s = lane & 31;
      const int c = mt * TM + ((((s >> 1) ^ ((r & 3) | ((r >> 3) << 2))) << 1) | (s & 1)) * 8;
      woff[q] = c < a.wcols ? (uint32_t)r * row_bytes + (uint32_t)c * 2u : kOOB;
    } else {
      const int r = lane >> 2;
      const int j = MODE == kGrGateUp ? mt * (TM / 2) + (i / MI) * (8 * MI) + 16 * (i % (MI / 2)) + r
                                      : mt * TM + 16 * i + r;
      woff[q] = j < a.wrows ? (uint32_t)j * row_bytes + (uint32_t)((lane & 3) ^ ((r >> 1) & 3)) * 16u : kOOB;
    }
  }
  uint32_t xoff[2];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int r = 16 * (2 * w + q) + (lane >> 2);
    xoff[q] = r < nv ? (uint32_t)r * (uint32_t)a.Kp * 2u + (uint32_t)((lane & 3) ^ ((r >> 1) & 3)) * 16u : kOOB;
  }
  const int kl = ((lane & 3) ^ (((lane >> 2) >> 1) & 3)) * 8;  // this lane's k within a step (not W_down)
  // With more than two buffers every call issues its LOADS loads (out of
  // range past the part's last step), so that a wait can count them; out of
  // range by addition, which leaves no branch.
  auto issue = [&](uint8_t* sw, uint8_t* sx, int st) {
    const int k0 = st * kGrK;
    const uint32_t out = G::BUFS == 2 || st < st1 ? 0u : kOOB;
#pragma unroll
    for (int q = 0; q < G::WQ; ++q) {
      const int i = G::WQ * w + q;
      if constexpr (MODE == kGrDown) {
        // rows past K lie past the matrix and read as zero
        dma16(rw0, sw + i * 1024, out + woff[q] + (uint32_t)k0 * row_bytes);
      } else {
        dma16(is_up(i) ? rw1 : rw0, sw + i * 1024, out + woff[q] + (uint32_t)k0 * 2u + (k0 + kl < a.K ? 0u : kOOB));
      }
    }
#pragma unroll
    for (int p = 0; p < NS; ++p)
#pragma unroll
      for (int q = 0; q < 2; ++q)
        dma16(rx[p], sx + p * kGrN * 64 + (2 * w + q) * 1024, out + xoff[q] + (uint32_t)k0 * 2u);
  };

  f32x4 acc[MI][NB];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[i][b] = f32x4{0.f, 0.f, 0.f, 0.f};

  const int fslot = (kb ^ ((r16 >> 1) & 3)) * 16;
  auto multiply = [&](const uint8_t* sw, const uint8_t* sx) {
    auto read_a = [&](int i) -> gr_bf16x8 {
      if constexpr (MODE == kGrDown) {
        // lane r of a 16-lane group names four values of row 8 kb + r / 4 and
        // receives column r % 16 of that group's four rows; two such reads
        // give eight rows of one column
        const int ar = 8 * kb + (r16 >> 2);
        const uint8_t* src = sw + ar * 512 + ((8 * wm + i) ^ ((r16 >> 2) | (kb << 2))) * 32 + (r16 & 3) * 8;
        const gr_i16x4 q0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) gr_i16x4*)src);
        const gr_i16x4 q1 =
            __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) gr_i16x4*)(src + 4 * 512));
        const uint2 u0 = __builtin_bit_cast(uint2, q0), u1 = __builtin_bit_cast(uint2, q1);
        return __builtin_bit_cast(gr_bf16x8, u32x4{u0.x, u0.y, u1.x, u1.y});
      } else {
        return *reinterpret_cast<const gr_bf16x8*>(sw + (16 * MI * wm + 16 * i + r16) * 64 + fslot);
      }
    };
    gr_bf16x8 bv[NS][NB], av[MI];
#pragma unroll
    for (int p = 0; p < NS; ++p)
#pragma unroll
      for (int b = 0; b < NB; ++b)
        bv[p][b] = *reinterpret_cast<const gr_bf16x8*>(sx + p * kGrN * 64 + (16 * NB * wn + 16 * b + r16) * 64 + fslot);
#pragma unroll
    for (int i = 0; i < MI; ++i) av[i] = read_a(i);
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int p = 0; p < NS; ++p)
#pragma unroll
        for (int b = 0; b < NB; ++b)
          acc[i][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[i], bv[p][b], acc[i][b], 0, 0, 0);
    // order: the vectors' operands and two rows of tiles, then each row's
    // products with the read of the row after next among them
    constexpr int RA = MODE == kGrDown ? 2 : 1;  // LDS reads per operand row
    __builtin_amdgcn_sched_group_barrier(0x100, NB * NS + 2 * RA, 0);
#pragma unroll
    for (int i = 0; i < MI - 2; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, NB * NS, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, RA, 0);
    }
    __builtin_amdgcn_sched_group_barrier(0x008, 2 * NB * NS, 0);
  };
  // A step: this wave's loads of it have landed (those of the LEFT steps
  // after it may be on their way) and its operand reads of the step before
  // are done; after the barrier that holds for every wave, so the loads of
  // step st + BUFS - 1 may overwrite the buffer of step st - 1.
  auto step = [&](uint8_t* sw, uint8_t* sx, uint8_t* nw, uint8_t* nx, int st, auto left, auto more) {
    wait_vm<decltype(left)::v * G::LOADS>();
    wait_lds();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if (decltype(more)::v && (G::BUFS > 2 || st + 1 < st1)) issue(nw, nx, st + G::BUFS - 1);
    __builtin_amdgcn_sched_barrier(0);  // the loads go out before the products
    multiply(sw, sx);
  };
  issue(sw0, sx0, st0);  // (a part has at least one step)
  if constexpr (G::BUFS > 2) issue(sw1, sx1, st0 + 1);
  if constexpr (G::BUFS > 3) issue(sw2, sx2, st0 + 2);
  // whole rounds of the buffers in a loop without exits (with one after each
  // step the compiler loses count of the loads at the loop's head and waits
  // for all of them there), then the last steps
  constexpr Const<G::BUFS - 2> left;
  constexpr Const<1> more;
  constexpr Const<0> last;
  int st = st0;
  for (; st + G::BUFS <= st1; st += G::BUFS) {
    if constexpr (G::BUFS == 2) {
      step(sw0, sx0, sw1, sx1, st, left, more);
      step(sw1, sx1, sw0, sx0, st + 1, left, more);
    } else if constexpr (G::BUFS == 3) {
      step(sw0, sx0, sw2, sx2, st, left, more);
      step(sw1, sx1, sw0, sx0, st + 1, left, more);
      step(sw2, sx2, sw1, sx1, st + 2, left, more);
    } else {
      step(sw0, sx0, sw3, sx3, st, left, more);
      step(sw1, sx1, sw0, sx0, st + 1, left, more);
      step(sw2, sx2, sw1, sx1, st + 2, left, more);
      step(sw3, sx3, sw2, sx2, st + 3, left, more);
    }
  }
  if (st < st1) step(sw0, sx0, nullptr, nullptr, st, left, last);
  if constexpr (G::BUFS > 2) { if (st + 1 < st1) step(sw1, sx1, nullptr, nullptr, st + 1, Const<G::BUFS - 3>(), last); }
  if constexpr (G::BUFS > 3) { if (st + 2 < st1) step(sw2, sx2, nullptr, nullptr, st + 2, Const<G::BUFS - 4>(), last); }
  wait_vm<0>();  // no load is on its way to LDS when the block ends

  // D[i][j] sits in lane j + 16 (i / 4), register i % 4: a lane holds four
  // consecutive output rows of one vector.
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    const int v = v0 + 16 * NB * wn + 16 * b + r16;
    if (v >= a.N) continue;
    if constexpr (MODE == kGrDown) {
      float* dst = a.out + ((size_t)part * a.N + v) * a.wcols;
#pragma unroll
      for (int i = 0; i < MI; ++i) {
        const int c = mt * TM + 16 * MI * wm + 16 * i + 4 * kb;
        if (c < a.wcols) *reinterpret_cast<f32x4*>(dst + c) = acc[i][b];  // wcols is a multiple of 8
      }
    } else {
      constexpr int NI = MODE == kGrGateUp ? MI / 2 : MI;
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        const int j = mt * (TM / MI) * NI + 16 * NI * wm + 16 * i + 4 * kb;
        float s[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) s[e] = silu(acc[i][b][e]);
        float* dst = a.out + (size_t)v * a.wrows + j;
        if ((a.wrows & 3) == 0) {
          if (j < a.wrows) *reinterpret_cast<f32x4*>(dst) = f32x4{fabsf(s[0]), fabsf(s[1]), fabsf(s[2]), fabsf(s[3])};
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (j + e < a.wrows) dst[e] = fabsf(s[e]);
        }
        if constexpr (MODE == kGrGateUp) {
          // h = v (x W_up) as planes for the down-projection, zero past m
          if (j < a.Kp2) {
            uint16_t pl[4][NS];
#pragma unroll
            for (int e = 0; e < 4; ++e)
              split_planes<NS>(j + e < a.wrows ? s[e] * acc[MI / 2 + i][b][e] : 0.f, pl[e]);
#pragma unroll
            for (int p = 0; p < NS; ++p)
              *reinterpret_cast<uint2*>(a.hs + ((size_t)p * a.N + v) * a.Kp2 + j) =
                  uint2{pl[0][p] | ((uint32_t)pl[1][p] << 16), pl[2][p] | ((uint32_t)pl[3][p] << 16)};
          }
        }
      }
    }
  }
}

// One block per vector: add the S partial down-projections of the layer
// before (part order), write the sum back, normalise (unit-gain RMSNorm) when
// asked, and write the planes, zero from d to Kp.  Bound by its few MB of traffic.
template <int NS>
__global__ __launch_bounds__(256) void k_rows_split(RowsSplitArgs a) {
  __shared__ float red[4];
  const int tid = threadIdx.x;
  const size_t row = blockIdx.x;
  const int d4 = a.d >> 2;  // d is a multiple of 8
  const f32x4* xr = reinterpret_cast<const f32x4*>(a.x + row * a.d);
  f32x4* xw = a.xsum ? reinterpret_cast<f32x4*>(a.xsum + row * a.d) : nullptr;
  if (a.zero)
    for (int i = blockIdx.x * 256 + tid; i < a.nzero; i += gridDim.x * 256) a.zero[i] = 0u;
  float inv = 1.f;
  if (a.norm || a.S > 0 || xw) {
    float ss = 0.f;
    for (int c = tid; c < d4; c += 256) {
      f32x4 v = xr[c];
      if (a.S > 0) {
        f32x4 t = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
        for (int p = 0; p < a.S; ++p) t += reinterpret_cast<const f32x4*>(a.partial + ((size_t)p * a.N + row) * a.d)[c];
        v += t;
      }
      if (xw) xw[c] = v;
      ss = fmaf(v.x, v.x, ss);
      ss = fmaf(v.y, v.y, ss);
      ss = fmaf(v.z, v.z, ss);
      ss = fmaf(v.w, v.w, ss);
    }
    ss = wave_sum(ss);
    if ((tid & (kWaveSize - 1)) == 0) red[tid / kWaveSize] = ss;
    __syncthreads();
    if (a.norm) inv = 1.0f / sqrtf(((red[0] + red[1]) + (red[2] + red[3])) / (float)a.d + a.eps);
  }
  const f32x4* xs = xw ? xw : xr;  // each thread reads back what it wrote itself
  for (int c = tid; c < a.Kp / 4; c += 256) {
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
    if (c < d4) v = xs[c];
    uint16_t pl[4][NS];
#pragma unroll
    for (int e = 0; e < 4; ++e) split_planes<NS>(v[e] * inv, pl[e]);
#pragma unroll
    for (int p = 0; p < NS; ++p)
      *reinterpret_cast<uint2*>(a.xs + ((size_t)p * a.N + row) * a.Kp + 4 * c) =
          uint2{pl[0][p] | ((uint32_t)pl[1][p] << 16), pl[2][p] | ((uint32_t)pl[3][p] << 16)};
  }
}

hipError_t launch_rows_split(int ns, const RowsSplitArgs& a, hipStream_t s) {
  KernelTimer timer("rows_split", s);
  if (ns == 2)
    hipExtLaunchKernelGGL(k_rows_split<2>, dim3(a.N), dim3(256), 0, s, timer.start(), timer.stop(), 0, a);
  else
    hipExtLaunchKernelGGL(k_rows_split<3>, dim3(a.N), dim3(256), 0, s, timer.start(), timer.stop(), 0, a);
  return hipGetLastError();
}

template <int MODE, int TM>
static hipError_t launch_rows_gemm(const char* name, int ns, RowsGemmArgs a, int outs, hipStream_t s) {
  constexpr int rows = MODE == kGrGateUp ? TM / 2 : TM;
  a.MT = (outs + rows - 1) / rows;
  a.NT = (a.N + kGrN - 1) / kGrN;
  const dim3 grid(a.MT * a.NT * a.S);
  KernelTimer timer(name, s);
  if (ns == 2)
    hipExtLaunchKernelGGL((k_rows_gemm<MODE, 2, TM>), grid, dim3(kGrThreads), 0, s, timer.start(), timer.stop(), 0, a);
  else
    hipExtLaunchKernelGGL((k_rows_gemm<MODE, 3, TM>), grid, dim3(kGrThreads), 0, s, timer.start(), timer.stop(), 0, a);
  return hipGetLastError();
}

// Output rows per block.  256 keeps the matrix cores busiest but needs about
// two blocks for every three compute units (4096 x 11008 gate product, us at
// 256 / 128 / 64 rows: 2048 vectors 310 / 386 / 550; 512 vectors, 172 blocks of
// 256, 128 / 126 / 150); below 80 such blocks 64 rows and four steps in flight
// read the weights fastest (64 vectors, 43 blocks: 120 / 82 / 60; 256
// vectors, 86 blocks: 122 / 88 / 100).
template <int MODE>
static hipError_t launch_rows_tiles(const char* name, int ns, const RowsGemmArgs& a, hipStream_t s) {
  const int64_t blocks = (int64_t)((a.wrows * (MODE == kGrGateUp ? 2 : 1) + 255) / 256) * ((a.N + kGrN - 1) / kGrN);
  if (blocks >= 170) return launch_rows_gemm<MODE, 256>(name, ns, a, a.wrows, s);
  if (blocks >= 80) return launch_rows_gemm<MODE, 128>(name, ns, a, a.wrows, s);
  return launch_rows_gemm<MODE, 64>(name, ns, a, a.wrows, s);
}

hipError_t launch_rows_acts(int ns, const RowsGemmArgs& a, hipStream_t s) {
  return launch_rows_tiles<kGrActs>("rows_acts", ns, a, s);
}

hipError_t launch_rows_gateup(int ns, const RowsGemmArgs& a, hipStream_t s) {
  return launch_rows_tiles<kGrGateUp>("rows_gateup", ns, a, s);
}

hipError_t launch_rows_down(int ns, const RowsGemmArgs& a, hipStream_t s) {
  return launch_rows_gemm<kGrDown, 256>("rows_down", ns, a, a.wcols, s);
}

}  // namespace cats
