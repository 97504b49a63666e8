// Role-routed linear layer (Sec. 3.1: Nexus tokens get their own projection
// matrices W_Q^N, W_K^N, W_V^N, W_O^N and their own MLP branches; every other
// token keeps the model's standard ones):
//     y[t] = W_N x[t]   for Nexus rows,   y[t] = W x[t]   for all other rows,
// x [T][K] bf16, W and W_N [N][K] bf16 (a linear layer's output-by-input
// layout), y [T][N] fp32.
//
// Few rows go to a weight-streaming kernel that does the whole call; more rows are laid
// out as one permutation, the non-Nexus rows in order, then the Nexus rows in order, and
// multiplied in tiles of it (a tile never mixes the two groups, so each tile reads one
// weight set), gathering x rows through the permutation and scattering y rows back.
// Up to kLocalRows rows every tile's workgroup ranks the rows itself; more rows take
// three small routing kernels first.
//
// GEMM: PM x PN output tile per workgroup of eight waves (2 x 4 parts), in blocks of
// v_mfma_f32_16x16x32_bf16, K in steps of 64.  Both operands are K-contiguous rows (x
// rows and weight rows), staged straight from global memory into an LDS ring of S steps
// (direct-to-LDS loads).  LDS rows are 128 bytes with an XOR swizzle on the 16-byte
// chunk index, which spreads 16 rows at one chunk over all banks; a fragment read takes
// four chunks at once, and the counters still show it at two passes instead of one
// (SQ_LDS_BANK_CONFLICT half of SQ_LDS_IDX_ACTIVE).
// Tiles are laid out so that the workgroups of one XCD share a band of output columns
// and walk its row tiles in order: the x rows a tile needs are also needed by the tiles
// of the other columns of the band, resident on the same XCD at the same time, and so is
// each weight chunk, which keeps both in its L2.
#include "common.h"
#include "scan.h"

#include <algorithm>
#include <cmath>
#include <type_traits>

namespace sonic {

constexpr int kRouteThreads = 1024;
constexpr int kPK = 64;                          // K step
constexpr int kPWavesM = 2, kPWavesN = 4;        // waves along rows and columns
constexpr int kPThreads = kPWavesM * kPWavesN * kWave;

// Pass 1: Nexus rows per block of 1024 rows.
__global__ __launch_bounds__(kRouteThreads) void route_count_kernel(const uint8_t *__restrict__ role, int T,
                                                                    int32_t *__restrict__ blk_nexus) {
  __shared__ int lds[kRouteThreads / kWave + 1];
  const int i = blockIdx.x * kRouteThreads + threadIdx.x;
  int tot;
  block_flag_scan<kRouteThreads>(i < T && role[i] == kNexus, &tot, lds);
  if (threadIdx.x == 0) blk_nexus[blockIdx.x] = tot;
}

// Pass 2 (one workgroup): Nexus rows before each block, in place; counts = (non-Nexus, Nexus).
// Its look at the status word decides for the whole call: the word may change at any time,
// and a tile must find either no rows or every slot of the permutation filled.
__global__ __launch_bounds__(kRouteThreads) void route_scan_kernel(int nblk, int T, int32_t *__restrict__ blk_nexus,
                                                                   int32_t *__restrict__ counts,
                                                                   const int32_t *status) {
  __shared__ int lds[kRouteThreads / kWave + 1];
  __shared__ int s_ok;
  const bool ok = block_status_clear(status, &s_ok);
  int carry = 0;
  for (int base = 0; base < nblk; base += kRouteThreads) {
    const int i = base + threadIdx.x;
    const int v = i < nblk ? blk_nexus[i] : 0;
    int tot;
    const int off = block_int_scan<kRouteThreads>(v, &tot, lds);
    if (i < nblk) blk_nexus[i] = carry + off;
    carry += tot;
  }
  if (threadIdx.x == 0) {   // no rows at all when the status is set: every GEMM tile exits
    counts[0] = ok ? T - carry : 0;
    counts[1] = ok ? carry : 0;
  }
}

// Pass 3: row i to its slot of the permutation, unless pass 2 stopped the call.
__global__ __launch_bounds__(kRouteThreads) void route_fill_kernel(const uint8_t *__restrict__ role, int T,
                                                                   const int32_t *__restrict__ blk_nexus,
                                                                   const int32_t *__restrict__ counts,
                                                                   int32_t *__restrict__ perm) {
  __shared__ int lds[kRouteThreads / kWave + 1];
  if (counts[0] + counts[1] != T) return;
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

// Routing inside a tile's workgroup, for up to kLocalRows rows: every workgroup reads all
// roles and ranks the rows itself, which saves the three routing launches.  Bit j of
// flags: row 512 j + thread is a Nexus row; before[j]: Nexus rows before it.
constexpr int kLocalRounds = 16;
constexpr int kLocalRows = kLocalRounds * kPThreads;
__device__ __forceinline__ bool local_routes(const uint8_t *__restrict__ role, int T, const int32_t *status, int &flags,
                                             int (&before)[kLocalRounds], int &total) {
  constexpr int NW = kPThreads / kWave;
  static_assert(kLocalRounds * NW == 2 * kWave, "two counts per lane");
  __shared__ int cnt[2 * kWave];
  __shared__ int s_ok;   // one thread's look at the status word decides for every wave
  if (threadIdx.x == 0) s_ok = __hip_atomic_load(status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0;
  const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  uint8_t mine[kLocalRounds];
#pragma unroll
  for (int j = 0; j < kLocalRounds; ++j) {
    mine[j] = kText;
    if (j * kPThreads < T) mine[j] = role[min(j * kPThreads + static_cast<int>(threadIdx.x), T - 1)];
  }
#pragma unroll
  for (int j = 0; j < kLocalRounds; ++j) {
    const bool nx = j * kPThreads + threadIdx.x < T && mine[j] == kNexus;
    flags |= (nx ? 1 : 0) << j;
    const uint64_t m = __ballot(nx);
    before[j] = lanes_below(m);
    if (lane == 0) cnt[j * NW + wave] = __popcll(m);
  }
  __syncthreads();
  if (!s_ok) return false;
  // every wave scans the 128 counts: lane l holds counts 2l and 2l + 1
  const int c0 = cnt[2 * lane], c1 = cnt[2 * lane + 1];
  int incl = c0 + c1;
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    const int v = __shfl_up(incl, o);
    if (lane >= o) incl += v;
  }
  const int ex = incl - c0 - c1;
#pragma unroll
  for (int j = 0; j < kLocalRounds; ++j) {
    const int i = j * NW + wave;
    before[j] += __shfl(ex, i / 2) + ((i & 1) ? __shfl(c0, i / 2) : 0);
  }
  total = __shfl(incl, kWave - 1);
  return true;
}

// The matrix cores (58 % busy) and the LDS reads with their conflicts bound a large tile
// (T = 43392, K = 4096, N = 6144: 1.83 ms, 1.19 PFLOP/s, where 128 x 256 tiles with two
// barriers a step took 2.19 ms): a 128 x 64 part per wave reads 0.75 KB of fragments per
// 32 Kflop product, a 64 x 64 one 1 KB, which at 128 B a cycle is all the LDS delivers in
// that time even without conflicts.  Blocks of 16 x 16 keep
// the accumulators in four-register groups; 32 x 32 blocks of this part spilled.  A small
// tile is bound by the latency of its steps (about 1.5 us each with one in flight), so
// its ring is deeper.
template <int PM, int PN, int S, bool LOCAL>
__global__ __launch_bounds__(kPThreads, 2) void routed_gemm_kernel(
    const uint16_t *__restrict__ x, const uint16_t *__restrict__ w_text, const uint16_t *__restrict__ w_nexus,
    float *__restrict__ y, const uint8_t *__restrict__ role, const int32_t *__restrict__ perm,
    const int32_t *__restrict__ counts, int T, int K, int N, int n_tiles, int xn, int band, const int32_t *status) {
  constexpr int BM = PM / kPWavesM / 16, BN = PN / kPWavesN / 16;   // 16 x 16 blocks per wave
  __shared__ __align__(16) uint16_t a_lds[S][PM * kPK];
  __shared__ __align__(16) uint16_t b_lds[S][PN * kPK];
  __shared__ int rows_lds[PM];

  // tile of this workgroup: the XCDs form (8 / xn) x xn bands; a band takes `band` column
  // tiles and every (8 / xn)-th row tile, in order
  const int xcd = blockIdx.x % kNumXcd;
  const int loc = blockIdx.x / kNumXcd;
  const int m_tile = loc / band * (kNumXcd / xn) + xcd / xn;
  const int n_tile = xcd % xn * band + loc % band;
  if (n_tile >= n_tiles) return;
  int n_text, n_nexus, flags = 0, before[LOCAL ? kLocalRounds : 1];
  if constexpr (LOCAL) {
    if (!local_routes(role, T, status, flags, before, n_nexus)) return;
    n_text = T - n_nexus;
  } else {
    n_text = counts[0];
    n_nexus = counts[1];
  }
  const int mt_text = (n_text + PM - 1) / PM;
  const int mt_all = mt_text + (n_nexus + PM - 1) / PM;
  if (m_tile >= mt_all) return;
  const bool nexus = m_tile >= mt_text;
  const int g0 = nexus ? n_text : 0;                          // first slot of the group
  const int row0 = (nexus ? m_tile - mt_text : m_tile) * PM;  // first row of the tile in the group
  const int nrows = min(PM, (nexus ? n_nexus : n_text) - row0);
  const int n0 = n_tile * PN;
  const uint16_t *__restrict__ w = nexus ? w_nexus : w_text;

  if constexpr (LOCAL) {
#pragma unroll
    for (int j = 0; j < kLocalRounds; ++j) {
      const int row = j * kPThreads + threadIdx.x;
      const bool nx = (flags >> j) & 1;
      const int slot = (nx ? before[j] : row - before[j]) - row0;
      if (row < T && nx == nexus && slot >= 0 && slot < PM) rows_lds[slot] = row;
    }
  } else {
    for (int r = threadIdx.x; r < nrows; r += kPThreads) rows_lds[r] = perm[g0 + row0 + r];
  }
  __syncthreads();

  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int lane = threadIdx.x % kWave;
  // staging: instruction i of a tile fills rows 8i .. 8i + 7 (lane L: row 8i + L / 8 at
  // chunk position L % 8); wave w issues instructions w * IA .. of A and w * IB .. of B
  constexpr int kNW = kPThreads / kWave;
  constexpr int IA = PM / 8 / kNW, IB = PN / 8 / kNW;   // per wave and step
  static_assert((S - 1) * (IA + IB) < 64, "the wait count fits vmcnt");
  static_assert(IA * kNW * 8 == PM && IB * kNW * 8 == PN, "whole instructions per wave");
  // per-lane byte offsets from the operand bases (the host checks that both operands
  // lie below 4 GiB), with the K step added to the wave-uniform base
  uint32_t a_off[IA], b_off[IB];
#pragma unroll
  for (int q = 0; q < IA; ++q) {
    const int r = 8 * (wave * IA + q) + lane / 8;
    const int c = (lane % 8) ^ swz_p(r);
    a_off[q] = static_cast<uint32_t>(rows_lds[min(r, nrows - 1)]) * static_cast<uint32_t>(K) * 2u + 16u * static_cast<uint32_t>(c);
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

  // this wave's (16 BM) x (16 BN) part of the tile.  The products are W . x^T, so a lane
  // ends up with four consecutive output columns of one row.
  const int wm = 16 * BM * (wave % kPWavesM), wn = 16 * BN * (wave / kPWavesM);
  const int fr = lane & 15, quarter = lane >> 4;   // fragment row; K chunk of the sub-step
  f32x4 acc[BM][BN];
#pragma unroll
  for (int i = 0; i < BM; ++i)
#pragma unroll
    for (int j = 0; j < BN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  // A step of 64 is four phases: K sub-step (32 deep) by half of the wave's rows.  A
  // phase's products run while the next phase's fragments are read into the other set
  // (the weight fragments change every other phase).  Rows 16 apart share their
  // swizzle, so the reads of a phase are one address per operand and immediates.
  constexpr int H = BM / 2;
  bf16x8 af[2][H], bf[2][BN];
  const uint16_t *const a_rd = &a_lds[0][(wm + fr) * kPK];
  const uint16_t *const b_rd = &b_lds[0][(wn + fr) * kPK];
  const int ch[2] = {(quarter ^ swz_p(fr)) * 8, ((4 + quarter) ^ swz_p(fr)) * 8};
  auto read_a = [&](int set, int buf, int kk, int half) {
#pragma unroll
    for (int t = 0; t < H; ++t)
      af[set][t] = *reinterpret_cast<const bf16x8 *>(a_rd + ch[kk] + buf * PM * kPK + 16 * (half * H + t) * kPK);
  };
  auto read_b = [&](int buf, int kk) {
#pragma unroll
    for (int t = 0; t < BN; ++t)
      bf[kk][t] = *reinterpret_cast<const bf16x8 *>(b_rd + ch[kk] + buf * PN * kPK + 16 * t * kPK);
  };
  // (products first: the other wave of the SIMD issues its reads and loads in between; 0.7 %)
  auto mult = [&](int set, int kk, int half) {
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int i = 0; i < H; ++i)
#pragma unroll
      for (int j = 0; j < BN; ++j)
        acc[half * H + i][j] =
            __builtin_amdgcn_mfma_f32_16x16x32_bf16(bf[kk][j], af[set][i], acc[half * H + i][j], 0, 0, 0);
    __builtin_amdgcn_s_setprio(0);
  };
  // Behind the last read of a buffer comes the step's only barrier: every wave has its
  // fragments of this buffer, so it is refilled (step s + S), and step s + 1 has landed
  // in the next one, whose first fragments are read under the last products.
  const int steps = K / kPK;
  auto phase_order = [&](auto reads) {
    __builtin_amdgcn_sched_group_barrier(0x100, decltype(reads)::value, 0);   // DS reads
    __builtin_amdgcn_sched_group_barrier(0x008, H * BN, 0);                   // MFMAs
    __builtin_amdgcn_sched_barrier(0);
  };
  auto step = [&](int s, int buf, int nxt) {
    read_a(1, buf, 0, 1);
    mult(0, 0, 0);
    phase_order(std::integral_constant<int, H>{});
    read_a(0, buf, 1, 0);
    read_b(buf, 1);
    mult(1, 0, 1);
    phase_order(std::integral_constant<int, H + BN>{});
    read_a(1, buf, 1, 1);
    mult(0, 1, 0);
    phase_order(std::integral_constant<int, H>{});
    if (S > 2 && s + S <= steps) wait_vm<(S - 2) * (IA + IB)>();   // all but the steps behind s + 1
    else wait_vm<0>();
    lds_barrier();
    read_a(0, nxt, 0, 0);   // past the last step: stale rows, never multiplied
    read_b(nxt, 0);
    __builtin_amdgcn_sched_barrier(0);
    if (s + S < steps) stage(s + S, &a_lds[0][buf * PM * kPK], &b_lds[0][buf * PN * kPK]);
    mult(1, 1, 1);
    __builtin_amdgcn_sched_barrier(0);
  };
  for (int s = 0; s < min(S, steps); ++s) stage(s, a_lds[s], b_lds[s]);
  if (steps >= S) wait_vm<(S - 1) * (IA + IB)>();
  else wait_vm<0>();
  lds_barrier();
  read_a(0, 0, 0, 0);
  read_b(0, 0);
  // one step per round, the buffer an index: with the steps unrolled by the ring and an
  // exit between them the compiler copies the accumulators and spills
  for (int s = 0, buf = 0; s < steps; ++s) {
    const int nxt = buf + 1 == S ? 0 : buf + 1;
    step(s, buf, nxt);
    buf = nxt;
  }

  // Lane (fr, quarter) holds columns 16 j + 4 quarter .. + 3 of row 16 i + fr.  Two column
  // blocks' lanes fr and fr + 8 change halves, so that a store writes whole 128-byte lines, 32
  // columns of eight rows, instead of half a line of sixteen: with few K steps the stores bound
  // the call (T = 9000, N = 10240, K = 64 95 us, now 90).
  typedef f32x4 f32x4_u __attribute__((aligned(4)));   // y is 4-byte aligned, N any number
  auto store = [&](int r, int n, const f32x4 &v) {
    if (r >= nrows) return;
    float *yr = y + static_cast<size_t>(rows_lds[r]) * N + n;
    if (n + 4 <= N) {
      *reinterpret_cast<f32x4_u *>(yr) = v;
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (n + e < N) yr[e] = v[e];
    }
  };
  const bool low = fr < 8;
#pragma unroll
  for (int i = 0; i < BM; ++i) {
#pragma unroll
    for (int j = 0; j + 1 < BN; j += 2) {
      f32x4 upper, lower;   // rows fr % 8 and fr % 8 + 8 of the block
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float give = low ? acc[i][j + 1][e] : acc[i][j][e];
        const float got = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(give), 0x128, 0xF, 0xF, false));   // row_ror:8
        upper[e] = low ? acc[i][j][e] : got;
        lower[e] = low ? got : acc[i][j + 1][e];
      }
      const int n = n0 + wn + 16 * j + 4 * quarter + (low ? 0 : 16);
      store(wm + 16 * i + (fr & 7), n, upper);
      store(wm + 16 * i + (fr & 7) + 8, n, lower);
    }
    if (BN % 2) store(wm + 16 * i + fr, n0 + wn + 16 * (BN - 1) + 4 * quarter, acc[i][BN - 1]);
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
  constexpr int RING = NW * S * SLOT;
  constexpr bool kRoom = RING * sizeof(uint16_t) + 16 <= 160 * 1024;   // ... for the decision behind the ring
  __shared__ __align__(16) uint16_t ring[RING + (kRoom ? 8 : 0)];
  const bool nexus = blockIdx.y != 0;
  const int n0 = blockIdx.x * C, r0 = blockIdx.z * R;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int lane = threadIdx.x % kWave;
  // One thread's look at the status word decides for every wave: the word may change
  // between two looks, and a wave that left alone would leave its partial sums unwritten.
  // One round trip for it and the roles.
  int *const s_ok = reinterpret_cast<int *>(ring + (kRoom ? RING : 0));
  if (threadIdx.x == 0) *s_ok = __hip_atomic_load(status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0;
  static_assert(R <= 2 * kWave, "two roles per lane");
  const bool m0 = (role[min(r0 + min(lane, R - 1), T - 1)] == kNexus) == nexus;   // rows past the end repeat one
  const bool m1 = R > kWave && (role[min(r0 + min(lane + kWave, R - 1), T - 1)] == kNexus) == nexus;
  __syncthreads();
  if (*s_ok == 0 || !__any(m0 || m1)) return;
  if (!kRoom) __syncthreads();   // the ring is filled over the word

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

template <int PM, int PN, int S, bool LOCAL>
static void launch_tiles(int T, int K, int N, const uint8_t *role, const uint16_t *x, const uint16_t *w_text,
                         const uint16_t *w_nexus, float *y, const int32_t *counts, const int32_t *perm,
                         const int32_t *status, hipStream_t stream) {
  const int m_tiles = (T + PM - 1) / PM + 1;   // the two groups can each end in a partial tile
  const int n_tiles = (N + PN - 1) / PN;
  // column bands: as many XCDs side by side as leave the fewest of them without columns
  int xn = kNumXcd, band = (n_tiles + kNumXcd - 1) / kNumXcd;
  for (int c = kNumXcd / 2; c >= 1; c /= 2) {
    const int w = (n_tiles + c - 1) / c;
    if (c * w < xn * band) xn = c, band = w;
  }
  const int m_per = (m_tiles + kNumXcd / xn - 1) / (kNumXcd / xn);
  routed_gemm_kernel<PM, PN, S, LOCAL><<<dim3(kNumXcd * band * m_per), dim3(kPThreads), 0, stream>>>(
      x, w_text, w_nexus, y, role, perm, counts, T, K, N, n_tiles, xn, band, status);
}

hipError_t launch_routed_gemm(int T, int K, int N, const uint8_t *role, const uint16_t *x, const uint16_t *w_text,
                              const uint16_t *w_nexus, float *y, int32_t *blk_nexus, int32_t *counts, int32_t *perm,
                              int32_t *status, hipStream_t stream) {
  // The weight-streaming kernel stages its block of x rows once per 32 columns and weight
  // set, so the rows it multiplies, in whole blocks, times the columns bound its use: in
  // us, weights not in the Infinity Cache, no Nexus rows / a fifth of them, streamed against
  // tiled, K = 4096: 64 rows of N = 14336 41 / 70 and 42 / 56; of 28672 72 / 125 and 58 / 98;
  // 128 rows of N = 6144 29 / 51 and 33 / 40, of 10240 52 / 76 and 39 / 48, of 14336 55 / 100
  // and 51 / 60.  (128 x 256 tiles behind routing kernels took 72 / 76 and 75 / 85 for the last two.)
  const int blocks = T <= 16 ? 16 : T <= 32 ? 32 : T <= 64 ? 64 : T <= 128 ? 128 : 256;
  if (T <= 16 || (T <= kSkinnyRows && static_cast<int64_t>(blocks) * N <= (1 << 20))) {
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
#define TILES(PM, PN, S)                                                                                        \
  (local ? launch_tiles<PM, PN, S, true>(T, K, N, role, x, w_text, w_nexus, y, counts, perm, status, stream)    \
         : launch_tiles<PM, PN, S, false>(T, K, N, role, x, w_text, w_nexus, y, counts, perm, status, stream))
  // Tile shape: large tiles read less per product, small ones keep 256 CUs busy and end
  // with less waste.  A shape's cost is its time for one tile per CU (measured, K = 4096:
  // 256 x 256 93 us, 128 x 256 58, 128 x 128 36, 64 x 128 43 for two, 64 x 64 29 for two
  // and 20 alone) times the rounds it takes; a last, partial round runs faster than a
  // full one and counts half its missing part.  Over 950 sizes (130 .. 9,000 rows, K = 256 ..
  // 14336, N = 200 .. 28672) the shape so chosen takes 3 % more than the best one on average
  // and up to a half more where the estimate of the last round is off.  Best against 256 x 256, K = 4096: T = 512,
  // N = 6144 37.9 us (128 x 128) and 94.6; T = 1024, N = 1024 21.5 (64 x 64) and 91.0;
  // T = 4096, N = 6144 256 x 256 itself, 207 against 245 for 128 x 256.
  const struct { int pm, pn, cost, least; } shapes[] = {
      {256, 256, 100, 100}, {128, 256, 60, 60}, {128, 128, 39, 39}, {64, 128, 24, 24}, {64, 64, 15, 20}};
  int best = 0;
  double best_cost = 0, best_rounds = 0;
  for (int i = 0; i < 5; ++i) {
    const double tiles = ((T + shapes[i].pm - 1) / shapes[i].pm + 1.0) * ((N + shapes[i].pn - 1) / shapes[i].pn);
    const double rounds = std::max(1.0, tiles / 256);
    const double cost = std::max<double>(shapes[i].least, 0.5 * (rounds + std::ceil(rounds)) * shapes[i].cost);
    if (i == 0 || cost < best_cost) best = i, best_cost = cost, best_rounds = rounds;
  }
  // Routing inside the tiles costs each of the tiles a CU does in turn about 0.7 us and 0.3 per
  // 1,024 rows (the two smallest shapes are two at a time), the routing kernels 4 to 5 us:
  // T = 5000, N = 28672, K = 64 146 us inside and 135 by kernels, T = 4000, N = 8192, K = 4096 285
  // and 271; T = 700, N = 28672, K = 64 27.9 and 29.4, T = 4000, N = 1024, K = 256 13.4 and 17.6.
  const bool local = T <= kLocalRows && best_rounds / (best >= 3 ? 2 : 1) * (0.7 + T * 0.0003) <= 4.5;
  if (!local) {
    const int nblk = (T + kRouteThreads - 1) / kRouteThreads;
    route_count_kernel<<<dim3(nblk), dim3(kRouteThreads), 0, stream>>>(role, T, blk_nexus);
    route_scan_kernel<<<dim3(1), dim3(kRouteThreads), 0, stream>>>(nblk, T, blk_nexus, counts, status);
    route_fill_kernel<<<dim3(nblk), dim3(kRouteThreads), 0, stream>>>(role, T, blk_nexus, counts, perm);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  switch (best) {
    case 0: TILES(256, 256, 2); break;
    case 1: TILES(128, 256, 3); break;
    case 2: TILES(128, 128, 4); break;
    case 3: TILES(64, 128, 3); break;
    default: TILES(64, 64, 4); break;
  }
#undef TILES
  return hipGetLastError();
}

}  // namespace sonic
