// Role-routed linear layer (Sec. 3.1: Nexus tokens get their own projection
// matrices W_Q^N, W_K^N, W_V^N, W_O^N and their own MLP branches; every other
// token keeps the model's standard ones):
//     y[t] = W_N x[t]   for Nexus rows,   y[t] = W x[t]   for all other rows,
// x [T][K] bf16, W and W_N [N][K] bf16 (a linear layer's output-by-input
// layout), y [T][N] fp32.
//
// Up to kSkinnyRows rows a weight-streaming kernel does the whole call.  More rows:
// routing, then tiles.
//
// Routing: three small kernels lay the rows out as one permutation: the
// non-Nexus rows in order, then the Nexus rows in order.  The GEMM then runs
// over 128-row tiles of that permutation (a tile never mixes the two groups, so
// each tile reads one weight set), gathering its x rows through the
// permutation and scattering its y rows back.
//
// GEMM: 128 x 256 output tile per workgroup of eight waves, each wave a 64 x 64
// part as 2 x 2 blocks of v_mfma_f32_32x32x16_bf16, K in steps of 64.  Both
// operands are K-contiguous rows (x rows and weight rows), staged straight from
// global memory into LDS (direct-to-LDS loads), double-buffered: step s + 1
// streams in while step s is multiplied.  LDS rows are 128 bytes with an XOR
// swizzle on the 16-byte chunk index, so the fragment reads (32 rows at one
// chunk) are bank-conflict free.  Each fragment read feeds two MFMAs, and the
// reads are scheduled two K sub-steps ahead of the MFMAs that consume them.
// Tiles are laid out so that the workgroups of one XCD share a band of output
// columns and walk the row tiles in order: the x rows a tile needs are also
// needed by the tiles of the other columns of the band, resident on the same
// XCD at the same time, and so is each weight chunk, which keeps both in its L2.
#include "common.h"
#include "scan.h"

namespace sonic {

constexpr int kRouteThreads = 1024;
// 128 x 256 tiles, eight waves as 2 (rows) x 4 (columns), each 64 x 64.  Measured on
// the 8B-shaped QKV product (T = 43392, K = 4096, N = 6144): 128 x 128 with four waves
// 0.80-0.88 PFLOP/s, 256 x 128 0.91, 128 x 256 0.93; 256 x 256 tiles need more than
// 256 registers per lane and spill.
constexpr int kPM = 128, kPN = 256, kPK = 64;    // tile rows, tile columns, K step
constexpr int kPWavesM = 2, kPWavesN = 4;        // waves along rows and columns
constexpr int kPThreads = kPWavesM * kPWavesN * kWave;
constexpr int kPBM = kPM / kPWavesM / 32, kPBN = kPN / kPWavesN / 32;   // 32x32 blocks per wave
constexpr int kPRowChunks = kPK / 8;            // 16-byte chunks per staged row

// Pass 1: Nexus rows per block of 1024 rows.
__global__ __launch_bounds__(kRouteThreads) void route_count_kernel(const uint8_t *__restrict__ role, int T,
                                                                    int32_t *__restrict__ blk_nexus,
                                                                    const int32_t *status) {
  __shared__ int lds[kRouteThreads / kWave + 1];
  __shared__ int s_ok;
  if (!block_status_clear(status, &s_ok)) return;
  const int i = blockIdx.x * kRouteThreads + threadIdx.x;
  int tot;
  block_flag_scan<kRouteThreads>(i < T && role[i] == kNexus, &tot, lds);
  if (threadIdx.x == 0) blk_nexus[blockIdx.x] = tot;
}

// Pass 2 (one workgroup): Nexus rows before each block, in place; counts = (non-Nexus, Nexus).
__global__ __launch_bounds__(kRouteThreads) void route_scan_kernel(int nblk, int T, int32_t *__restrict__ blk_nexus,
                                                                   int32_t *__restrict__ counts,
                                                                   const int32_t *status) {
  __shared__ int lds[kRouteThreads / kWave + 1];
  __shared__ int s_ok;
  const bool ok = block_status_clear(status, &s_ok);
  int carry = 0;
  for (int base = 0; base < nblk; base += kRouteThreads) {
    const int i = base + threadIdx.x;
    const int v = (ok && i < nblk) ? blk_nexus[i] : 0;
    int tot;
    const int off = block_int_scan<kRouteThreads>(v, &tot, lds);
    if (ok && i < nblk) blk_nexus[i] = carry + off;
    carry += tot;
  }
  if (threadIdx.x == 0) {   // no rows at all when the status is set: every GEMM tile exits
    counts[0] = ok ? T - carry : 0;
    counts[1] = ok ? carry : 0;
  }
}

// Pass 3: row i to its slot of the permutation.
__global__ __launch_bounds__(kRouteThreads) void route_fill_kernel(const uint8_t *__restrict__ role, int T,
                                                                   const int32_t *__restrict__ blk_nexus,
                                                                   const int32_t *__restrict__ counts,
                                                                   int32_t *__restrict__ perm,
                                                                   const int32_t *status) {
  __shared__ int lds[kRouteThreads / kWave + 1];
  __shared__ int s_ok;
  if (!block_status_clear(status, &s_ok)) return;
  const int i = blockIdx.x * kRouteThreads + threadIdx.x;
  const bool in = i < T;
  const bool nx = in && role[i] == kNexus;
  int tot;
  const int r = block_flag_scan<kRouteThreads>(nx, &tot, lds);
  const int nexus_before = blk_nexus[blockIdx.x] + r;   // Nexus rows before row i
  if (in) perm[nx ? counts[0] + nexus_before : i - nexus_before] = i;
}

// chunk position of chunk c in staged row r (16 rows hit 16 distinct 4-bank groups)
__device__ __forceinline__ int swz_p(int r) { return (r & 7) ^ ((r >> 3) & 1); }

__global__ __launch_bounds__(kPThreads) void routed_gemm_kernel(
    const uint16_t *__restrict__ x, const uint16_t *__restrict__ w_text, const uint16_t *__restrict__ w_nexus,
    float *__restrict__ y, const int32_t *__restrict__ perm, const int32_t *__restrict__ counts, int K, int N,
    int n_tiles, int band) {
  __shared__ __align__(16) uint16_t a_lds0[kPM * kPK];
  __shared__ __align__(16) uint16_t a_lds1[kPM * kPK];
  __shared__ __align__(16) uint16_t b_lds0[kPN * kPK];
  __shared__ __align__(16) uint16_t b_lds1[kPN * kPK];
  __shared__ int rows_lds[kPM];

  // tile of this workgroup: XCD x takes column tiles [x * band, (x + 1) * band), row tiles in order
  const int xcd = blockIdx.x % kNumXcd;
  const int loc = blockIdx.x / kNumXcd;
  const int m_tile = loc / band;
  const int n_tile = xcd * band + loc % band;
  const int n_text = counts[0], n_nexus = counts[1];
  const int mt_text = (n_text + kPM - 1) / kPM;
  const int mt_all = mt_text + (n_nexus + kPM - 1) / kPM;
  if (n_tile >= n_tiles || m_tile >= mt_all) return;
  const bool nexus = m_tile >= mt_text;
  const int g0 = nexus ? n_text : 0;                           // first slot of the group
  const int row0 = (nexus ? m_tile - mt_text : m_tile) * kPM;  // first row of the tile in the group
  const int nrows = min(kPM, (nexus ? n_nexus : n_text) - row0);
  const int n0 = n_tile * kPN;
  const uint16_t *__restrict__ w = nexus ? w_nexus : w_text;

  for (int r = threadIdx.x; r < kPM; r += kPThreads) rows_lds[r] = perm[g0 + row0 + min(r, nrows - 1)];
  __syncthreads();

  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int lane = threadIdx.x % kWave;
  // staging: instruction i of a tile fills rows 8i .. 8i + 7 (lane L: row 8i + L / 8 at
  // chunk position L % 8); wave w issues instructions w * IA .. of A and w * IB .. of B
  constexpr int kNW = kPThreads / kWave;
  constexpr int IA = kPM / 8 / kNW, IB = kPN / 8 / kNW;   // per wave and step
  static_assert(IA * kNW * 8 == kPM && IB * kNW * 8 == kPN, "whole instructions per wave");
  // per-lane byte offsets from the operand bases (the host checks that both operands
  // lie below 4 GiB), with the K step added to the wave-uniform base
  uint32_t a_off[IA], b_off[IB];
#pragma unroll
  for (int q = 0; q < IA; ++q) {
    const int r = 8 * (wave * IA + q) + lane / 8;
    const int c = (lane % 8) ^ swz_p(r);
    a_off[q] = static_cast<uint32_t>(rows_lds[r]) * static_cast<uint32_t>(K) * 2u + 16u * static_cast<uint32_t>(c);
  }
#pragma unroll
  for (int q = 0; q < IB; ++q) {
    const int r = 8 * (wave * IB + q) + lane / 8;
    const int c = (lane % 8) ^ swz_p(r);
    b_off[q] = static_cast<uint32_t>(min(n0 + r, N - 1)) * static_cast<uint32_t>(K) * 2u +
               16u * static_cast<uint32_t>(c);
  }
  const char *xb = uniform_ptr(reinterpret_cast<const char *>(x));
  const char *wb = uniform_ptr(reinterpret_cast<const char *>(w));
  auto stage = [&](int s, uint16_t *a_buf, uint16_t *b_buf) {
    const size_t koff = static_cast<size_t>(s) * kPK * 2;   // bytes
    const uint32_t la = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(a_buf));
    const uint32_t lb = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(b_buf));
#pragma unroll
    for (int q = 0; q < IA; ++q) dma_row16_s(xb + koff, a_off[q], la + (wave * IA + q) * kWave * 16);
#pragma unroll
    for (int q = 0; q < IB; ++q) dma_row16_s(wb + koff, b_off[q], lb + (wave * IB + q) * kWave * 16);
  };

  // this wave's (32 kPBM) x (32 kPBN) part of the tile
  const int wm = 32 * kPBM * (wave % kPWavesM), wn = 32 * kPBN * (wave / kPWavesM);
  const int li = lane & 31, lg = lane >> 5;
  f32x16 acc[kPBM][kPBN];
#pragma unroll
  for (int bi = 0; bi < kPBM; ++bi)
#pragma unroll
    for (int bj = 0; bj < kPBN; ++bj) acc[bi][bj] = f32x16{};

  // each A fragment feeds kPBN MFMAs, each B fragment kPBM
  auto mult = [&](const uint16_t *a_buf, const uint16_t *b_buf) {
#pragma unroll
    for (int kk = 0; kk < kPK / 16; ++kk) {
      const int c = 2 * kk + lg;
      bf16x8 af[kPBM], bf[kPBN];
#pragma unroll
      for (int t = 0; t < kPBM; ++t) {
        const int ra = wm + 32 * t + li;
        af[t] = *reinterpret_cast<const bf16x8 *>(&a_buf[(ra * kPRowChunks + (c ^ swz_p(ra))) * 8]);
      }
#pragma unroll
      for (int t = 0; t < kPBN; ++t) {
        const int rb = wn + 32 * t + li;
        bf[t] = *reinterpret_cast<const bf16x8 *>(&b_buf[(rb * kPRowChunks + (c ^ swz_p(rb))) * 8]);
      }
#pragma unroll
      for (int bi = 0; bi < kPBM; ++bi)
#pragma unroll
        for (int bj = 0; bj < kPBN; ++bj)
          acc[bi][bj] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[bi], bf[bj], acc[bi][bj], 0, 0, 0);
    }
    // the fragment reads run two K sub-steps (eight reads) ahead of the MFMAs
    order_reads_ahead<(kPK / 16) * kPBM * kPBN, 1, 2 * (kPBM + kPBN)>();
  };

  // double buffer: each wave issues IA + IB loads per step, so "step s has landed"
  // is "all but the IA + IB most recent" while step s + 1 streams
  const int steps = K / kPK;
  stage(0, a_lds0, b_lds0);
  for (int s = 0; s < steps; s += 2) {
    if (s + 1 < steps) {
      stage(s + 1, a_lds1, b_lds1);
      wait_vm<IA + IB>();
    } else {
      wait_vm<0>();
    }
    lds_barrier();            // step s is in buffer 0 for every wave
    mult(a_lds0, b_lds0);
    lds_barrier();            // every wave is done with buffer 0
    if (s + 1 >= steps) break;
    if (s + 2 < steps) {
      stage(s + 2, a_lds0, b_lds0);
      wait_vm<IA + IB>();
    } else {
      wait_vm<0>();
    }
    lds_barrier();            // step s + 1 is in buffer 1
    mult(a_lds1, b_lds1);
    lds_barrier();            // every wave is done with buffer 1
  }

  // lane (j = li, half lg) holds rows 8 (e / 4) + 4 lg + e % 4 of column j of each block
#pragma unroll
  for (int bi = 0; bi < kPBM; ++bi)
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int r = wm + 32 * bi + 8 * (e >> 2) + 4 * lg + (e & 3);
      if (r < nrows) {
        float *yrow = y + static_cast<size_t>(rows_lds[r]) * N;
#pragma unroll
        for (int bj = 0; bj < kPBN; ++bj) {
          const int n = n0 + wn + 32 * bj + li;
          if (n < N) yrow[n] = acc[bi][bj][e];
        }
      }
    }
}

// Few rows (the tokens one generation step adds, a short turn's Nexus rows): the product
// only streams the weights, so the kernel is built around that stream.  A workgroup owns
// 16 NT output columns of one weight set for a block of 16 TT rows, and its NW waves a
// contiguous part of K each.  A wave stages 64-deep slices of its weight and x rows into
// an LDS ring of S slots of its own (direct-to-LDS loads, whole 128-byte row pieces), so
// no barrier stands between the loads and the products.  The rows of a block are all
// multiplied by the workgroup's set and those of its role are stored, so no permutation
// is built and the call is one launch; a set without rows in the block costs its
// workgroup one look at the roles.  The waves' partial sums are added in wave order.
// Bound by the weights' stream: 8 rows of K = 4096, N = 6144 take 10.9 us (50 MB, 4.6 TB/s;
// the tile kernel with its routing launches took 55), 64 rows 13.9 (58), 128 rows 20.8
// (59), weights not in the Infinity Cache.  Loading the operand registers straight from
// memory instead (16 rows per 16 lanes) took 16.7 us for 8 rows and 40 for 64: the address
// path then handles one lane a cycle.
constexpr int kSkinnyRows = 256;

template <int NT, int TT, int NW, int S>
__global__ __launch_bounds__(NW * kWave) void skinny_proj_kernel(
    const uint16_t *__restrict__ x, const uint16_t *__restrict__ w_text, const uint16_t *__restrict__ w_nexus,
    float *__restrict__ y, const uint8_t *__restrict__ role, int T, int K, int N, const int32_t *status) {
  constexpr int C = 16 * NT, R = 16 * TT;         // columns and rows of the workgroup
  constexpr int IN = (C + R) / 8;                 // direct-to-LDS instructions per slot (8 rows each)
  constexpr int SLOT = (C + R) * kPK;             // elements per slot: weight rows, then x rows
  constexpr int RS = C + 1;                       // row stride of the partial sums, in floats
  static_assert((S - 1) * IN < 64, "the wait count fits vmcnt");
  static_assert(NW * R * RS * sizeof(float) <= NW * S * SLOT * sizeof(uint16_t), "the partial sums fit in the ring");
  __shared__ __align__(16) uint16_t ring[NW * S * SLOT];
  const bool nexus = blockIdx.y != 0;
  const int n0 = blockIdx.x * C, r0 = blockIdx.z * R;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int lane = threadIdx.x % kWave;
  // one round trip for the status word and the roles (every wave for itself: the same answer)
  const int32_t pending = __hip_atomic_load(status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  static_assert(R <= 2 * kWave, "two roles per lane");
  const bool m0 = (role[min(r0 + min(lane, R - 1), T - 1)] == kNexus) == nexus;   // rows past the end repeat one
  const bool m1 = R > kWave && (role[min(r0 + min(lane + kWave, R - 1), T - 1)] == kNexus) == nexus;
  if (pending != 0 || !__any(m0 || m1)) return;

  const int nk = K / kPK;
  const int per = (nk + NW - 1) / NW;
  const int k0 = min(nk, wave * per);
  const int steps = min(nk, k0 + per) - k0;
  const char *wb = uniform_ptr(reinterpret_cast<const char *>(nexus ? w_nexus : w_text));
  const char *xb = uniform_ptr(reinterpret_cast<const char *>(x));
  // lane L of instruction i fills row 8 i + L / 8 at chunk position L % 8 (both operands
  // lie below 4 GiB, checked by the host)
  uint32_t off[IN];
#pragma unroll
  for (int i = 0; i < IN; ++i) {
    const int r = 8 * i + lane / 8;
    const int c = (lane % 8) ^ swz_p(r % 16);
    const int row = i < C / 8 ? min(n0 + r, N - 1) : min(r0 + r - C, T - 1);
    off[i] = static_cast<uint32_t>(row) * static_cast<uint32_t>(K) * 2u + 16u * static_cast<uint32_t>(c);
  }
  uint16_t *const my = ring + wave * S * SLOT;
  const uint32_t my0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(my));
  auto issue = [&](int step, int slot) {
    const size_t kb = static_cast<size_t>(k0 + step) * kPK * 2;
#pragma unroll
    for (int i = 0; i < IN; ++i)
      dma_row16_s((i < C / 8 ? wb : xb) + kb, off[i], my0 + slot * (SLOT * 2) + i * kWave * 16);
  };
  const int fr = lane & 15, quarter = lane >> 4;   // fragment row; K chunk of the sub-step
  f32x4 acc[NT][TT];
#pragma unroll
  for (int i = 0; i < NT; ++i)
#pragma unroll
    for (int t = 0; t < TT; ++t) acc[i][t] = f32x4{0.f, 0.f, 0.f, 0.f};

  for (int s = 0; s < min(S, steps); ++s) issue(s, s);
  for (int s = 0, slot = 0; s < steps; ++s, slot = slot + 1 == S ? 0 : slot + 1) {
    if (s + S <= steps) wait_vm<(S - 1) * IN>();   // all but the slots behind this one
    else wait_vm<0>();
    const uint16_t *sl = my + slot * SLOT;
#pragma unroll
    for (int kk = 0; kk < kPK / 32; ++kk) {
      const int p = ((4 * kk + quarter) ^ swz_p(fr)) * 8;
      bf16x8 wf[NT], xf[TT];
#pragma unroll
      for (int i = 0; i < NT; ++i) wf[i] = *reinterpret_cast<const bf16x8 *>(&sl[(16 * i + fr) * kPK + p]);
#pragma unroll
      for (int t = 0; t < TT; ++t) xf[t] = *reinterpret_cast<const bf16x8 *>(&sl[(C + 16 * t + fr) * kPK + p]);
#pragma unroll
      for (int t = 0; t < TT; ++t)
#pragma unroll
        for (int i = 0; i < NT; ++i)
          acc[i][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[i], xf[t], acc[i][t], 0, 0, 0);
    }
    __builtin_amdgcn_s_waitcnt(15 | (3 << 14) | (7 << 4));   // lgkmcnt(0): the slot may be refilled
    if (s + S < steps) issue(s + S, slot);
  }
  __syncthreads();   // every wave is done with its part of the ring (and its loads have landed)
  // lane (fr, quarter) holds columns 16 i + 4 quarter .. + 3 of row 16 t + fr
  float *red = reinterpret_cast<float *>(ring);
#pragma unroll
  for (int i = 0; i < NT; ++i)
#pragma unroll
    for (int t = 0; t < TT; ++t)
#pragma unroll
      for (int e = 0; e < 4; ++e) red[(wave * R + 16 * t + fr) * RS + 16 * i + 4 * quarter + e] = acc[i][t][e];
  __syncthreads();
  for (int u = threadIdx.x; u < R * C; u += NW * kWave) {
    const int r = u / C, c = u % C;
    if (r0 + r < T && n0 + c < N && (role[r0 + r] == kNexus) == nexus) {
      float v = red[r * RS + c];
#pragma unroll
      for (int w = 1; w < NW; ++w) v += red[(w * R + r) * RS + c];
      y[static_cast<size_t>(r0 + r) * N + n0 + c] = v;
    }
  }
}

int routed_gemm_blocks(int T, int N) {
  const int m_tiles = (T + kPM - 1) / kPM + 1;   // the two groups can each end in a partial tile
  const int n_tiles = (N + kPN - 1) / kPN;
  const int band = (n_tiles + kNumXcd - 1) / kNumXcd;
  return kNumXcd * band * m_tiles;
}

hipError_t launch_routed_gemm(int T, int K, int N, const uint8_t *role, const uint16_t *x, const uint16_t *w_text,
                              const uint16_t *w_nexus, float *y, int32_t *blk_nexus, int32_t *counts, int32_t *perm,
                              int32_t *status, hipStream_t stream) {
  if (T <= kSkinnyRows) {
#define SKINNY(NT, TT, NW, S)                                                                               \
  skinny_proj_kernel<NT, TT, NW, S>                                                                         \
      <<<dim3((N + 16 * NT - 1) / (16 * NT), 2, (T + 16 * TT - 1) / (16 * TT)), dim3(NW * kWave), 0, stream>>>( \
          x, w_text, w_nexus, y, role, T, K, N, status)
    // Two column blocks a workgroup halve the x rows it stages per weight row, one keeps
    // more workgroups busy: N = 6144, 64 rows 13.9 us with two and 19.3 with one; N = 4096,
    // 13.0 and 11.6; up to 16 rows one is faster at every size.  More than 128 rows stage
    // enough x to want two everywhere (256 rows, N = 4096: 21 and 32).
    const bool two = (N + 15) / 16 > 256 || T > 128;
    if (T <= 16) SKINNY(1, 1, 8, 2);
    else if (T <= 32) {
      if (two) SKINNY(2, 2, 8, 2);
      else SKINNY(1, 2, 8, 3);
    } else if (T <= 64) {
      if (two) SKINNY(2, 4, 4, 3);
      else SKINNY(1, 4, 4, 3);
    } else {
      if (two) SKINNY(2, 8, 4, 2);
      else SKINNY(1, 8, 4, 2);
    }
#undef SKINNY
    return hipGetLastError();
  }
  const int nblk = (T + kRouteThreads - 1) / kRouteThreads;
  route_count_kernel<<<dim3(nblk), dim3(kRouteThreads), 0, stream>>>(role, T, blk_nexus, status);
  route_scan_kernel<<<dim3(1), dim3(kRouteThreads), 0, stream>>>(nblk, T, blk_nexus, counts, status);
  route_fill_kernel<<<dim3(nblk), dim3(kRouteThreads), 0, stream>>>(role, T, blk_nexus, counts, perm, status);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int n_tiles = (N + kPN - 1) / kPN;
  const int band = (n_tiles + kNumXcd - 1) / kNumXcd;
  routed_gemm_kernel<<<dim3(routed_gemm_blocks(T, N)), dim3(kPThreads), 0, stream>>>(
      x, w_text, w_nexus, y, perm, counts, K, N, n_tiles, band);
  return hipGetLastError();
}

}  // namespace sonic
