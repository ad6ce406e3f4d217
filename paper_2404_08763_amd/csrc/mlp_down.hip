// Down-projection of a batch (3..16 rows, bf16 weights) on the matrix cores:
//   partial_q[b][c] = sum over the union-active neurons j of group q of
//                     h[b][j] W_down[j][c]
// from the segment lists of k_mlp_gateup; k_mlp_reduce sums the groups in order.
//
// What bounds it: reading the active rows of W_down, and for narrow layers the
// round trips before the first row is asked for, and the partial sums (written
// here, read by k_mlp_reduce).  So:
//  - Block (ct, q) owns 512 columns and the rows of neuron group q, its eight
//    waves 128 columns of every other 32-row step: half the groups, and half
//    the partial sums, of blocks of 1024 columns (4096 x 11008 at 16 rows:
//    8.4 MB instead of 16.8).
//  - A list entry is known by its row mask, so a block asks for masks,
//    indices and h of its whole range at once and lists the entries in LDS: one
//    round trip, where counts, then indices, then h took three.
//  - A lane's operand is eight rows of one column, which W_down's row-major
//    layout does not hold contiguously: a wave streams its 32-row x 128-column
//    slice of a step (256-byte runs, two steps ahead) into its own LDS region
//    and reads it back column-wise with gfx950's transposing LDS reads.
//  - h enters as NS bf16 planes (as x does in the gate/up kernel; products
//    exact, fp32 accumulation), staged per block as [plane][row][list entry].
// Measured (us, before: 1024-column blocks, three round trips): 4096 x 11008 at
// 8 / 16 rows 18.6 / 20.2 (20.5 / 22.6), 5120 x 13824 at 16 rows 29.2 (33.9),
// 8192 x 28672 at 8 rows 76 (80; 6.2 TB/s), 512 x 1408 at 8 rows 6.3 (8.3).
#include "stream.hpp"
#include "internal.hpp"

namespace cats {

typedef __bf16 dn_bf16x8 __attribute__((ext_vector_type(8)));
typedef short dn_i16x4 __attribute__((ext_vector_type(4)));

constexpr int kDnWaves = 8;
constexpr int kDnThreads = kDnWaves * kWaveSize;
constexpr int kDnRows = 32;                     // rows of a step
constexpr int kDnChunk = kDnThreads;            // segment positions listed at a time, one per thread
constexpr int kDnPitch = 128 * 2 + 8;           // LDS bytes per row of a wave's slice (8 pad: row groups 16 banks apart)
constexpr int kDnHPitch = kDnChunk + 8;         // bf16 per batch row of the staged h
static_assert(kDownCols == 4 * 128, "four waves of 128 columns side by side");

template <int NS>
__global__ __launch_bounds__(kDnThreads) void k_mlp_down(DownArgs a) {
  __shared__ __attribute__((aligned(16))) int s_j[kDnChunk];
  __shared__ __attribute__((aligned(16))) uint16_t s_h[NS][kMaxRows * kDnHPitch];
  __shared__ __attribute__((aligned(16))) uint8_t s_w[kDnWaves * kDnRows * kDnPitch];
  __shared__ int w_cnt[kDnWaves];

  const int tid = threadIdx.x;
  const int lane = tid & (kWaveSize - 1);
  const int w = __builtin_amdgcn_readfirstlane(tid / kWaveSize);
  const int wc = w & 3, wr = w >> 2;  // columns, and which of every two steps
  const int B = a.B, d = a.d, m = a.m;
  const int ct = blockIdx.x % a.CT, q = blockIdx.x / a.CT;
  const int g0 = (int)(((int64_t)q * a.G) / a.NG), g1 = (int)(((int64_t)(q + 1) * a.G) / a.NG);
  const int p0 = (int)(((int64_t)g0 * m) / a.G), p1 = (int)(((int64_t)g1 * m) / a.G);  // segment positions
  const int col0 = ct * kDownCols + wc * 128;  // this wave's first column
  const uint32_t row_bytes = (uint32_t)d * 2u;
  const __amdgpu_buffer_rsrc_t rd = make_rsrc(a.wd, (uint32_t)((uint64_t)m * row_bytes));
  const __amdgpu_buffer_rsrc_t rm = make_rsrc(a.seg_mask, (uint32_t)m * 4u);
  const __amdgpu_buffer_rsrc_t rj = make_rsrc(a.seg_j, (uint32_t)m * 4u);
  const __amdgpu_buffer_rsrc_t rh = make_rsrc(a.seg_h, (uint32_t)((size_t)B * m * sizeof(float)));
  uint8_t* wreg = s_w + (size_t)w * kDnRows * kDnPitch;

  // streaming a step: load p (0..7) covers rows 8 (lane / 16) + p, 16 bytes
  // (8 columns) per lane, one 256-byte run per row
  const int lr = lane >> 4, lc = lane & 15;
  const int lcol = col0 + lc * 8;
  const uint32_t lcolb = lcol < d ? (uint32_t)lcol * 2u : kOOB;
  // operands: A lane = column oi + 16 kq, B lane = batch row oi + 16 kq; both
  // hold the eight rows 8 kq .. 8 kq + 7 of the step
  const int oi = lane & 15, kq = lane >> 4;

  f32x4 acch[8], accl[8];
#pragma unroll
  for (int t = 0; t < 8; ++t) acch[t] = accl[t] = f32x4{0.f, 0.f, 0.f, 0.f};

  // this thread's position of a chunk: mask, index and h of every row
  uint32_t mk, jv, hv[kMaxRows];
  auto fetch = [&](int c0) {
    const int p = c0 + tid;
    const uint32_t off = p < p1 ? (uint32_t)p * 4u : kOOB;
    mk = __builtin_amdgcn_raw_buffer_load_b32(rm, (int)off, 0, 0);
    jv = __builtin_amdgcn_raw_buffer_load_b32(rj, (int)off, 0, 0);
#pragma unroll
    for (int b = 0; b < kMaxRows; ++b)
      hv[b] = __builtin_amdgcn_raw_buffer_load_b32(rh, (int)(b < B ? (uint32_t)b * (uint32_t)m * 4u + off : kOOB), 0, 0);
  };
  fetch(p0);
  for (int c0 = p0; c0 < p1; c0 += kDnChunk) {
    // the chunk's entries in order
    const uint64_t bal = __ballot(mk != 0u);
    if (lane == 0) w_cnt[w] = __popcll(bal);
    __syncthreads();  // (and the chunk before is multiplied)
    int pos = __popcll(bal & ((1ull << lane) - 1ull)), nr = 0;
#pragma unroll
    for (int k = 0; k < kDnWaves; ++k) {
      if (k < w) pos += w_cnt[k];
      nr += w_cnt[k];
    }
    const int nsteps = (nr + kDnRows - 1) / kDnRows;
    if (mk != 0u) {
      s_j[pos] = (int)jv;
#pragma unroll
      for (int b = 0; b < kMaxRows; ++b)
#pragma unroll
        for (int p = 0; p < NS; ++p)
          s_h[p][b * kDnHPitch + pos] =
              (uint16_t)(NS == 2 ? split2_plane(__uint_as_float(hv[b]), p) : split3_plane(__uint_as_float(hv[b]), p));
    }
    // the last step's missing rows are zero
    if (tid < nsteps * kDnRows - nr) {
      s_j[nr + tid] = -1;
#pragma unroll
      for (int b = 0; b < kMaxRows; ++b)
#pragma unroll
        for (int p = 0; p < NS; ++p) s_h[p][b * kDnHPitch + nr + tid] = 0;
    }
    __syncthreads();

    // a lane's rows of a step are 8 lr .. 8 lr + 7, their indices two 16-byte
    // LDS reads
    auto load_step = [&](u32x4(&buf)[8], int st) {
      int jr[8];
      if (st < nsteps) {
        const int4 ja = *reinterpret_cast<const int4*>(s_j + st * kDnRows + 8 * lr);
        const int4 jb = *reinterpret_cast<const int4*>(s_j + st * kDnRows + 8 * lr + 4);
        jr[0] = ja.x; jr[1] = ja.y; jr[2] = ja.z; jr[3] = ja.w;
        jr[4] = jb.x; jr[5] = jb.y; jr[6] = jb.z; jr[7] = jb.w;
      } else {
#pragma unroll
        for (int p = 0; p < 8; ++p) jr[p] = -1;
      }
#pragma unroll
      for (int p = 0; p < 8; ++p)
        buf[p] = ld_buf16_stream(rd, jr[p] >= 0 ? (uint32_t)jr[p] * row_bytes + lcolb : kOOB);
    };
    // this wave's slice of a step into its LDS region (the previous step's
    // reads by this wave come first: LDS operations of a wave run in order)
    auto write_step = [&](const u32x4(&buf)[8]) {
#pragma unroll
      for (int p = 0; p < 8; ++p) {
        uint8_t* dst = wreg + (8 * lr + p) * kDnPitch + lc * 16;
        reinterpret_cast<uint2*>(dst)[0] = uint2{buf[p].x, buf[p].y};
        reinterpret_cast<uint2*>(dst)[1] = uint2{buf[p].z, buf[p].w};
      }
    };
    auto compute_step = [&](int st) {
      const int e0 = st * kDnRows + 8 * kq;
      dn_bf16x8 bv[NS];
#pragma unroll
      for (int p = 0; p < NS; ++p) bv[p] = *reinterpret_cast<const dn_bf16x8*>(s_h[p] + oi * kDnHPitch + e0);
      // A operand by transposing reads: in each 16-lane group, lane r
      // names four consecutive 16-bit values (row 8 kq + r / 4, columns
      // 4 (r % 4) .. + 3 of the tile) and lane i receives value i % 4 of the
      // rows named by lanes i / 4 + 4 k, k = 0..3: column i of four
      // consecutive rows.  Two reads give the eight rows of a step's half.
      const int ar = 8 * kq + (oi >> 2);
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        const uint8_t* src = wreg + ar * kDnPitch + (t * 16 + 4 * (oi & 3)) * 2;
        const dn_i16x4 r0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) dn_i16x4*)src);
        const dn_i16x4 r1 =
            __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) dn_i16x4*)(src + 4 * kDnPitch));
        const uint2 w0 = __builtin_bit_cast(uint2, r0), w1 = __builtin_bit_cast(uint2, r1);
        const dn_bf16x8 av = __builtin_bit_cast(dn_bf16x8, u32x4{w0.x, w0.y, w1.x, w1.y});
        acch[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, bv[0], acch[t], 0, 0, 0);
#pragma unroll
        for (int p = 1; p < NS; ++p) accl[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, bv[p], accl[t], 0, 0, 0);
      }
    };
    // Whole pairs of this half's steps in a loop without a way round either of
    // them, and the next chunk's entries asked for whether there are any or
    // not: with a condition the compiler cannot count the loads in flight and
    // waits for all of them at the loop's head.
    u32x4 rA[8], rB[8];
    load_step(rA, wr);
    load_step(rB, wr + 2);
    fetch(c0 + kDnChunk);
    int st = wr;
    for (; st + 2 < nsteps; st += 4) {
      write_step(rA);
      load_step(rA, st + 4);
      compute_step(st);
      write_step(rB);
      load_step(rB, st + 6);
      compute_step(st + 2);
    }
    if (st < nsteps) {
      write_step(rA);
      compute_step(st);
    }
  }

  // the two halves of the steps, in order
  if constexpr (NS == 3) {
    add_lower_planes(acch, accl);
  } else {
#pragma unroll
    for (int t = 0; t < 8; ++t) accl[t] = acch[t] + accl[t];
  }
  __syncthreads();
  f32x4* red = reinterpret_cast<f32x4*>(s_w);
  if (wr == 1) {
#pragma unroll
    for (int t = 0; t < 8; ++t) red[(wc * 8 + t) * kWaveSize + lane] = accl[t];
  }
  __syncthreads();
  if (wr == 1) return;
  // D[i][j] sits in lane j + 16 (i / 4), register i % 4: batch row
  // jb = lane % 16, columns 4 (lane / 16) .. + 3 of each tile
  const int jb = lane & 15, c4 = (lane >> 4) * 4;
  if (jb < B) {
    float* part = a.partial + ((size_t)q * B + jb) * d;
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const int c = col0 + t * 16 + c4;
      if (c < d) *reinterpret_cast<f32x4*>(part + c) = accl[t] + red[(wc * 8 + t) * kWaveSize + lane];
    }
  }
}

hipError_t launch_down(int planes, const DownArgs& a, hipStream_t s) {
  const dim3 grid(a.CT * a.NG), block(kDnThreads);
  KernelTimer timer("mlp_down", s);
  if (planes == 2)
    hipExtLaunchKernelGGL(k_mlp_down<2>, grid, block, 0, s, timer.start(), timer.stop(), 0, a);
  else
    hipExtLaunchKernelGGL(k_mlp_down<3>, grid, block, 0, s, timer.start(), timer.stop(), 0, a);
  return hipGetLastError();
}

}  // namespace cats
