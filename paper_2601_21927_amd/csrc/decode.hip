// Decode over the retained context {I_sys, N, Q_n} (problem statement).
//
// decode_kernel: grid (split, kv-head, request), four or eight waves.  A split owns a
// contiguous range of the request's context rows 0..len (row len is the token
// being generated: it is read from k_new/v_new, and split 0 of each kv-head also
// appends it to the cache).  The range is cut into 16-row groups, dealt to the
// waves round-robin; per group a wave computes
//   scores   S^T (16 rows x 16 cols) = K . Q^T   v_mfma_f32_16x16x32_bf16;
//            column c < G is q-head kvh*G + c;
//   softmax  per q-head, online, fp32, exp2 with log2(e) folded into the scale;
//            a column's statistics live in the four lanes that hold it;
//   values   O^T (d x 16 cols) += V^T . P^T   v_mfma_f32_16x16x32_bf16, V read
//            back transposed (ds_read_b64_tr_b16); P^T is the score accumulator
//            itself (its lane layout is the operand layout) as the sum of two bf16
//            values, the 16 rows' first and second parts in one product against
//            the rows of V twice, and the softmax sum adds those values.
// K and V rows go straight from global memory to a two-slot LDS ring of the
// wave's own (direct-to-LDS loads), so a wave keeps its next group in flight
// while it computes one.  The waves then merge through LDS.
//
// With one split the workgroup writes the output.  With several, each split
// stores its partial (max, sum, acc) and counts itself done with an atomic; the
// split that arrives last merges the partials by log-sum-exp and writes the
// output.  The eight XCDs' L2 caches are not coherent with each other, so the
// hand-off does not go through them: the partials are stored write-through at
// system scope and read back with loads that bypass the caches, which needs no
// L2 writeback or invalidate (either would evict the K/V other workgroups are
// streaming).  Every split of a pair counts itself once per call, splits
// without rows included, so the last to count knows that every workgroup of
// the pair has read cache_len; it counts the pair for its request while it
// loads the partials, and the last pair of a request advances cache_len.
//
// BAL (many pairs, long contexts): the rows of the whole batch are shared evenly
// among the workgroups instead of each request's among its own.  Every workgroup
// works the shares out from all lengths, so no length may advance while another
// workgroup has yet to read it: pairs (and workgroups left without rows) count for
// their request, requests for the call, and the last one advances every length.
#include "common.h"
#include "scan.h"

#include <algorithm>
#include <type_traits>

namespace sonic {

constexpr int kGroupRows = 16;
// In a completion counter: a workgroup that counted found an error on the status word.  The
// word may change while a call runs, so the workgroups (and waves) of one call may see
// different values; each counts all the same, which leaves the counters at zero for the
// next call, and what such a workgroup had a part in is not merged and not advanced.
constexpr int kStopBit = 1 << 30;
// Shared rows, bytes of a cache row (all kv-heads) from which the workgroups of the kv-heads
// alternate.  With all those of one head before the next, the resident ones read a part of
// each row, and of long rows that is a part of the memory channels: 16 / 16 heads of 128, 32
// contexts of 3,000 .. 8,000 rows, 326 us so and 264 alternating.  Shorter rows are better
// off with a head at a time (32 / 8, 64 contexts of 100 .. 4,000, 52.6 and 55.5).
constexpr int kLongRow = 4096;
constexpr int kMaxSplits = 16;   // of a (request, kv-head): the merge loads all its partials in one round trip

typedef short v4i16 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) v4i16 lds_v4i16_t;
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));

// The K/V loads of the pipeline go straight to LDS and are written as inline
// assembly, so the compiler does not count them (it would otherwise wait for the
// prefetched group as well before reading the current one); their completion is
// waited for explicitly (wait_vm).
// 16 bytes per lane into LDS at dst + 16 * lane (dst wave-uniform, passed in M0)
__device__ __forceinline__ void dma16(const void *src, const uint16_t *dst) {
  // C-style cast: converting the LDS pointer to its 32-bit address
  const uint32_t lds = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(
      reinterpret_cast<uintptr_t>((const __attribute__((address_space(3))) uint16_t *)dst)));
  asm volatile("s_mov_b32 m0, %1\n\tglobal_load_lds_dwordx4 %0, off" : : "v"(src), "s"(lds) : "memory", "m0");
}
// Accesses that bypass the (non-coherent) caches, for partials handed from one XCD to
// another: buffer operations with the system-scope bits (sc0, sc1), 16 bytes a lane.  Each
// instruction is a request of its own to memory, so their number counts: the merge of 16
// splits of 7 heads took 1.2 us longer with 8 bytes a lane, 2.9 with 4.
constexpr int kSystemScope = 1 | 16;
typedef __amdgpu_buffer_rsrc_t rsrc_t;
__device__ __forceinline__ rsrc_t partial_rsrc(float *p) {   // p wave-uniform
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(uniform_ptr(reinterpret_cast<const char *>(p))), 0, -1, 0x00027000);
}

// The value of the lane N places on in the row of 16 lanes (cyclic).
template <int N> __device__ __forceinline__ float row_rotate(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x120 | N, 0xF, 0xF, false));
}

__device__ __forceinline__ bool stops(int32_t pending) {
  pending = __builtin_amdgcn_readfirstlane(pending);
  return pending != 0 && pending != SONIC_ERR_CAPACITY;
}

template <int D, int G, bool MASKED, int NW, bool BAL>
__global__ __launch_bounds__(NW * kWave, 2) void decode_kernel(
    uint16_t *__restrict__ kc, uint16_t *__restrict__ vc, const int64_t *__restrict__ row_off,
    const int32_t *__restrict__ row_cap, int32_t *__restrict__ cache_len, const uint8_t *__restrict__ row_role,
    const uint16_t *__restrict__ q, const uint16_t *__restrict__ k_new, const uint16_t *__restrict__ v_new,
    float *__restrict__ out, DecodeWs ws, int32_t *status, int Hkv, int nsplit_max, int max_ctx, int batch,
    int target, float scale_log2) {
  constexpr int KS = D / 32;                   // k steps of the 16x16x32 score product
  constexpr int DB = D / 16;                   // 16-wide d blocks of the value product
  constexpr int DC = D / 8;                    // 16-byte chunks per row
  constexpr int NI = kGroupRows * DC / kWave;  // direct-to-LDS instructions per tensor and group
  constexpr int NG = 2 * NI;                   // loads per lane per group
  constexpr int DP = D + 16;                   // row stride of the merge in LDS: heads 16 banks apart
  constexpr int SLOT = kGroupRows * D;         // elements of one tensor's slot
  constexpr int KSWZ = DC - 1;                 // K: 16-byte chunk p of row r at p ^ (r & KSWZ)
  constexpr int VSWZ = DC / 2 - 1;             // V: 32-byte segment s of row r at s ^ (r & VSWZ)
  static_assert(NI * kWave == kGroupRows * DC, "a group's rows are whole DMA instructions");
  // ring: [wave][slot 0/1][K, V][16 rows][D] with the swizzles above (K for the
  // row-fragment reads of the scores, V for the transposing reads); reused for the
  // merge of the waves at the end
  __shared__ __align__(16) uint16_t ring[NW * 2 * 2 * SLOT];
  // each wave's copy of the G query rows (direct-to-LDS, so that no load the
  // compiler counts precedes the pipeline's)
  constexpr int NQ = (G * D * 2 + 1023) / 1024;   // direct-to-LDS instructions for Q
  __shared__ __align__(16) uint16_t q_lds[NW][NQ * 512];
  // split 0: the new token's k and v rows, fetched at the start and appended at the end
  __shared__ __align__(16) uint16_t app_lds[kWave * 8];
  static_assert(2 * DC <= kWave, "one direct-to-LDS instruction holds the new k and v rows");
  __shared__ float m_lds[NW][16];
  __shared__ float l_lds[NW][16];
  __shared__ int s_last;
  __shared__ int s_stop[NW];   // each wave's look at the status word
  static_assert(sizeof(float) * NW * G * DP <= sizeof(uint16_t) * NW * 4 * SLOT,
                "the merge fits in the ring");

  // BAL: blockIdx.z == 0, the grid is (workgroups, kv-heads) or, with long rows, (kv-heads, workgroups)
  const bool heads_first = BAL && Hkv * D * 2 >= kLongRow;
  const int kvh = heads_first ? blockIdx.x : blockIdx.y;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int lane = threadIdx.x % kWave;
  const int Hq = Hkv * G;
  const int nsplit = heads_first ? gridDim.y : gridDim.x;   // BAL: workgroups of a kv-head
  int split, b, nsp, R, len;
  int64_t base;
  // A pending error other than a capacity error (a layout error of an earlier call) stops
  // the whole call: nothing is appended, written or advanced.  A wave that sees one loads
  // no rows and goes on to the workgroup's count (see kStopBit).
  bool stop;
  // BAL: the workgroup's plan.  Lane l looks at request l (at most 64): its length,
  // capacity and first row, all requested together with the status word.  A split is R
  // rows, the same for every request, and request l takes ceil(rows / R) consecutive
  // workgroups of each kv-head.  R is about the smallest with which these are
  // `target` (whole rounds of resident workgroups; a few more are launched, which the short
  // last splits make room for), no fewer than 256 rows and no less than a sixteenth of the
  // longest request.
  int first = 0, lane_ctx = 0, used = 0;
  bool flat = false;
  int counts = 0, call_counts = 0;   // of the request (or, flat, of the call at once), of the call
  if constexpr (BAL) {
    const int l = threadIdx.x % kWave, lb = min(l, batch - 1);
    const int32_t pending = __hip_atomic_load(status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const int ll = cache_len[lb], lc = row_cap[lb];
    const int64_t lo = row_off[lb];
    stop = stops(pending);
    const bool fits = ll >= 0 && ll < lc && ll < max_ctx;   // (behind an error a length may be anything)
    if (__any(!fits) && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) raise_status(status, SONIC_ERR_CAPACITY);
    lane_ctx = l < batch && fits ? ll + 1 : 0;
    const int groups = (lane_ctx + kGroupRows - 1) / kGroupRows;
    const int total = __builtin_amdgcn_readlane(wave_scan(groups), kWave - 1);
    int longest = groups;
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) longest = max(longest, __shfl_xor(longest, o));
    longest = max(max(__builtin_amdgcn_readlane(longest, 0), __builtin_amdgcn_readlane(longest, 16)),
                  max(__builtin_amdgcn_readlane(longest, 32), __builtin_amdgcn_readlane(longest, 48)));
    const unsigned ug = groups;
    const int active = __popcll(__ballot(lane_ctx > 0));
    int rg = max(max(256 / kGroupRows, (longest + kMaxSplits - 1) / kMaxSplits), (total + target - 1) / target);
    int mine, upto;
    auto cut = [&](int groups_each) {
      rg = groups_each;
      mine = (ug + rg - 1) / static_cast<unsigned>(rg);
      upto = wave_scan(mine);
      used = __builtin_amdgcn_readlane(upto, kWave - 1);
    };
    cut(rg);
    if (used > nsplit) {
      // a request's last split is half full on average: go on there, and end where every
      // request may have an empty one
      const int half = max(rg, (2 * total - 1) / (2 * target - active) + 1);
      int most = longest;
      if (nsplit > active) most = min(most, (total + nsplit - active - 1) / (nsplit - active));
#pragma unroll 1
      for (int i = 0; used > nsplit; ++i) cut(i < 4 ? min(most, half + half * i / 32) : most);
    }
    const int w = heads_first ? blockIdx.y : blockIdx.x;
    b = __popcll(__ballot(upto <= w));
    R = rg * kGroupRows;
    // The workgroups left without rows count for the active requests in turn, or, where there
    // are few of them, everything counts for the call at once: one level of counts less at
    // the call's end (0.8 us of 30), but a thousand in one word take 10 us.
    const unsigned spare = nsplit - used;
    flat = spare * Hkv <= 128;
    if (active == 0) return;   // no request has room: nothing to count or advance
    counts = Hkv * (active + static_cast<int>(spare));
    int rank = 0, expect = 0;
    if (!flat) {
      const unsigned each = spare / active, more = spare - each * active;
      rank = lanes_below(__ballot(lane_ctx > 0));
      expect = Hkv * (1 + each + (rank < more ? 1 : 0));
    }
    if (w < used) {
      nsp = __builtin_amdgcn_readlane(mine, b);
      first = __builtin_amdgcn_readlane(upto, b) - nsp;
      len = __builtin_amdgcn_readlane(ll, b);
      const uint32_t lo32 = __builtin_amdgcn_readlane(static_cast<int>(lo), b);
      const uint32_t hi32 = __builtin_amdgcn_readlane(static_cast<int>(lo >> 32), b);
      base = static_cast<int64_t>((static_cast<uint64_t>(hi32) << 32) | lo32);
    } else {
      b = 0;
      if (!flat) {
        const int nth = (w - used) % active;
        b = __builtin_ctzll(__ballot(lane_ctx > 0 && rank == nth));
      }
      nsp = 0, first = w, len = 0, base = 0;
    }
    split = w - first;
    if (!flat) counts = __builtin_amdgcn_readlane(expect, b);
    call_counts = active;
  } else {
    split = blockIdx.x;
    b = blockIdx.z;
    // the status word, the length and the request's first cache row are requested
    // together (one round trip for all three)
    const int32_t pending = __hip_atomic_load(status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    len = cache_len[b];
    const int cap = row_cap[b];
    base = row_off[b];
    asm volatile("" ::"s"(len), "s"(cap), "s"(base));
    __builtin_amdgcn_sched_barrier(0);   // none of the three is looked at before all are requested
    stop = stops(pending);
    if (len < 0 || len >= cap || len >= max_ctx) {   // uniform over the request: no append, no output, no count
      if (split == 0 && kvh == 0 && threadIdx.x == 0) raise_status(status, SONIC_ERR_CAPACITY);
      return;
    }
    // split ranges: R rows each, a multiple of the group size
    R = ((len + nsplit_max) / nsplit_max + kGroupRows - 1) / kGroupRows * kGroupRows;
    nsp = (len + R) / R;   // splits that hold rows; the others have nothing to do
  }
  const int n_ctx = len + 1;
  const int pair = b * Hkv + kvh;
  float *orow = out + (static_cast<size_t>(b) * Hq + kvh * G) * D;
  // the pair's partials: [split][G][D] values, then, behind every pair's, [split][G] (max, sum)
  const size_t slot0 = BAL ? static_cast<size_t>(kvh) * nsplit + first : static_cast<size_t>(pair) * nsplit_max;
  float *const acc_rec = ws.part + slot0 * (G * D);
  float *const stat_rec = ws.part + static_cast<size_t>(gridDim.x) * gridDim.y * gridDim.z * (G * D) + slot0 * (2 * G);
  // A pair's last workgroup counts the pair for its request in done[b]; the last pair of a
  // request advances its length.  BAL: a workgroup without rows counts for a request as well,
  // and a request's last count is one count of the call in the upper bits of done[0]; the
  // last of the call advances every length.  A workgroup has read the lengths before it
  // counts, so none can still see an advanced one.
  constexpr int kCallOne = 1 << 16, kLowBits = kCallOne - 1;
  auto add = [&](int32_t *counter, int n, bool stopped) {
    if (stopped) __hip_atomic_fetch_or(counter, kStopBit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return __hip_atomic_fetch_add(counter, n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  };
  auto count = [&](bool stopped) { return add(&ws.done[BAL && flat ? 0 : b], 1, stopped); };
  auto advance = [&](int old) {   // the first wave; `old` is its first lane's
    old = __builtin_amdgcn_readfirstlane(old);
    if constexpr (BAL) {
      if ((old & kLowBits) != counts - 1) return;
      if (!flat) {
        if (threadIdx.x == 0) old = add(&ws.done[0], kCallOne, (old & kStopBit) != 0);
        old = __builtin_amdgcn_readfirstlane(old);
        if ((old & ~kStopBit) >> 16 != call_counts - 1) return;
      }
      if ((old & kStopBit) == 0 && lane_ctx > 0) cache_len[threadIdx.x] = lane_ctx;
      if (threadIdx.x < batch) ws.done[threadIdx.x] = 0;
    } else {
      if ((old & ~kStopBit) != Hkv - 1) return;
      if (threadIdx.x == 0) {
        if ((old & kStopBit) == 0) cache_len[b] = n_ctx;
        ws.done[b] = 0;
      }
    }
  };
  if (lane == 0) s_stop[wave] = stop;
  auto any_stop = [&]() {   // behind a barrier
    int any = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) any |= s_stop[w];
    return __builtin_amdgcn_readfirstlane(any) != 0;
  };

  // Behind the store of outputs 4u .. 4u + 3 of the pair (o, normalised by L).  An infinite V
  // comes out of the sums as NaN (a probability's second part is zero or negative for half of
  // the rows, a row past a range's end is a copy of its first one times zero, and so is a
  // split past the last one): where the scores were numbers, the V column is read again, and
  // one whose only values that are none are infinities of one sign gives that infinity.
  auto settle_infinities = [&](int u, f32x4 o, float L) {
    const float all_of = (o[0] + o[1]) + (o[2] + o[3]);
    if (__builtin_expect(__any(all_of != all_of && L == L), 0)) {
      const int dd = 4 * (u % (D / 4));
      const uint16_t *col = vc + (static_cast<size_t>(base) * Hkv + kvh) * D + dd;
      const uint16_t *last = v_new + static_cast<size_t>(pair) * D + dd;
      int found[4] = {0, 0, 0, 0};   // 1: +inf, 2: -inf, 4: NaN
#pragma unroll 4
      for (int r = 0; r < n_ctx; ++r) {
        if (MASKED && r < len && row_role[base + r] == kText) continue;
        const uint16_t *x = r < len ? col + static_cast<size_t>(r) * Hkv * D : last;
#pragma unroll
        for (int e = 0; e < 4; ++e) found[e] |= x[e] == 0x7F80 ? 1 : x[e] == 0xFF80 ? 2 : (x[e] & 0x7FFF) > 0x7F80 ? 4 : 0;
      }
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (o[e] != o[e] && L == L && (found[e] == 1 || found[e] == 2)) orow[4 * u + e] = found[e] == 1 ? INFINITY : -INFINITY;
    }
  };

  // Every split counts itself once, after its partial (if any) is stored.  The last
  // to count merges the partials of the nsp splits with rows by log-sum-exp, all of them
  // in one memory round trip, writes the output, and counts the pair for its request
  // while the partials load; the last pair of a request advances the length.
  auto finish_pair = [&](bool stopped) {
    if (threadIdx.x == 0) {
      const int old = add(&ws.arrive[pair], 1, stopped);
      s_last = (old & ~kStopBit) == (BAL ? nsp : nsplit) - 1 ? ((old & kStopBit) != 0 ? 2 : 1) : 0;
    }
    __syncthreads();
    if (!s_last) return;
    if (__builtin_expect(s_last == 2, 0)) {   // a split of the pair was stopped: nothing to merge
      if (threadIdx.x < kWave) {
        int old_done = 0;
        if (threadIdx.x == 0) {
          ws.arrive[pair] = 0;
          old_done = count(true);
        }
        advance(old_done);
      }
      return;
    }
    // Thread u merges values 4u .. 4u + 3 (of q-head u / (D / 4)).  For the weights, lane
    // 16 j + i of a wave takes split i of the wave's j-th q-head.
    static_assert(G * D / 4 <= NW * kWave && kMaxSplits == 16, "one pass; a row of lanes holds a head's splits");
    if (wave * kWave >= G * D / 4) return;
    constexpr int LH = D / 4;   // lanes per q-head
    const int u = min(static_cast<int>(threadIdx.x), G * D / 4 - 1);
    const rsrc_t ra = partial_rsrc(acc_rec), rs = partial_rsrc(stat_rec);
    const int head = min(wave * (kWave / LH) + lane / 16, G - 1), sp = lane % 16;
    const auto ml = __builtin_amdgcn_raw_buffer_load_b64(rs, (min(sp, nsp - 1) * G + head) * 8, 0, kSystemScope);
    f32x4 a[kMaxSplits];
    auto load = [&](auto n) {
#pragma unroll
      for (int i = 0; i < decltype(n)::value; ++i)
        a[i] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(ra, u * 16, min(i, nsp - 1) * (G * D * 4), kSystemScope));
    };
    if (nsp <= 4) load(std::integral_constant<int, 4>{});
    else load(std::integral_constant<int, kMaxSplits>{});
    __builtin_amdgcn_sched_barrier(0);
    // behind the loads, so that the round trips pass together (the compiler waits for an
    // atomic's result on the spot)
    int old_done = 0;
    if (threadIdx.x == 0) old_done = count(false);
    const float m = sp < nsp ? __uint_as_float(ml[0]) : -INFINITY;
    float top = m;
    top = fmaxf(top, row_rotate<8>(top));
    top = fmaxf(top, row_rotate<4>(top));
    top = fmaxf(top, row_rotate<2>(top));
    top = fmaxf(top, row_rotate<1>(top));
    const float w = m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m - top);
    float sum = w == 0.f ? 0.f : w * __uint_as_float(ml[1]);
    sum += row_rotate<8>(sum);
    sum += row_rotate<4>(sum);
    sum += row_rotate<2>(sum);
    sum += row_rotate<1>(sum);
    const int from = lane / LH * 16;
    f32x4 A = {0.f, 0.f, 0.f, 0.f};
    auto fold = [&](auto n) {
#pragma unroll
      for (int i = 0; i < decltype(n)::value; ++i) {
        const float wi = __shfl(w, from + i);   // 0 past the splits
#pragma unroll
        for (int e = 0; e < 4; ++e) A[e] = fmaf(wi, a[i][e], A[e]);
      }
    };
    if (nsp <= 4) fold(std::integral_constant<int, 4>{});
    else fold(std::integral_constant<int, kMaxSplits>{});
    const float L = __shfl(sum, from);
    const f32x4 o = {A[0] / L, A[1] / L, A[2] / L, A[3] / L};
    if (threadIdx.x < G * D / 4) *reinterpret_cast<f32x4 *>(orow + 4 * u) = o;
    if (threadIdx.x == 0) ws.arrive[pair] = 0;
    if (threadIdx.x < kWave) advance(old_done);
    settle_infinities(u, o, L);
  };
  if (split >= nsp) {   // no rows (only when nsplit > 1)
    __syncthreads();    // every wave has read the lengths: the workgroup may count
    const bool stopped = any_stop();
    if (!BAL) {
      finish_pair(stopped);
    } else if (threadIdx.x < kWave) {
      int old = 0;
      if (threadIdx.x == 0) old = count(stopped);
      advance(old);
    }
    return;
  }
  const bool whole = BAL ? nsp == 1 : nsplit == 1;   // the split is all of the pair's context
  const int r_begin = split * R;
  const int r_end = min(n_ctx, r_begin + R);
  const int ngroups = stop ? 0 : (r_end - r_begin + kGroupRows - 1) / kGroupRows;
  const int col = lane & 15;       // score column (q-head) / value-product column
  const int quarter = lane >> 4;   // score rows 4*quarter .. +3
  const size_t row_stride = static_cast<size_t>(Hkv) * D;
  const uint16_t *knew = k_new + (static_cast<size_t>(b) * Hkv + kvh) * D;
  const uint16_t *vnew = v_new + (static_cast<size_t>(b) * Hkv + kvh) * D;
  uint16_t *kbase = kc + static_cast<size_t>(base) * row_stride + static_cast<size_t>(kvh) * D;
  uint16_t *vbase = vc + static_cast<size_t>(base) * row_stride + static_cast<size_t>(kvh) * D;

  // Split 0 appends the new token at row len.  Its rows go to LDS ahead of every other
  // load of wave 0 (so the first wait covers them, and no wave waits for a load of its
  // own before the pipeline starts); the stores happen after the streaming.  Rows of
  // this call read the new token from k_new / v_new, so nothing here depends on them.
  const bool appender = split == 0 && wave == 0;
  if (appender && !stop) {
    const int c = lane < 2 * DC ? lane % DC : 0;
    dma16((lane >= DC && lane < 2 * DC ? vnew : knew) + c * 8, app_lds);
  }

  // The wave's Q rows go to q_lds (lanes past the G rows fetch row 0 again); the
  // Q^T fragments (B operand of the scores) are read from there once the first wait
  // has passed: lane (col, quarter) takes d = 32*ks + 8*quarter .. +7 of q-head
  // kvh*G + col (columns col >= G take head kvh*G and are never read back).
  if (!stop) {
    const uint16_t *q0 = q + (static_cast<size_t>(b) * Hq + kvh * G) * D;
#pragma unroll
    for (int i = 0; i < NQ; ++i) {
      const int e = (i * kWave + lane) * 8;   // element of the [G][D] block
      dma16(q0 + (e < G * D ? e : e % D), &q_lds[wave][i * 512]);
    }
  }
  bf16x8 qf[KS];
  auto read_q = [&]() {
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
      qf[ks] = *reinterpret_cast<const bf16x8 *>(&q_lds[wave][(col < G ? col : 0) * D + 32 * ks + 8 * quarter]);
  };

  // Row r of the context: the cache below len, the new token at len.  Rows past the
  // split's end load row r_begin instead (and are masked), so every group issues the
  // same loads and the waits can be counted.
  auto row_of = [&](int r) { return r < r_end ? r : r_begin; };
  auto kptr = [&](int r) { return r < len ? kbase + static_cast<size_t>(r) * row_stride : knew; };
  auto vptr = [&](int r) { return r < len ? vbase + static_cast<size_t>(r) * row_stride : vnew; };
  uint16_t *my_ring = ring + wave * 4 * SLOT;

  // Group g of the split covers rows r_begin + 16 g ...; wave w takes groups w, w + NW,
  // w + 2 NW, ... (a fixed order, so the result does not depend on timing).
  auto group_row0 = [&](int g) { return r_begin + kGroupRows * g; };
  // issue the loads of group g into ring slot s: lane -> (row, 16-byte position) of
  // each instruction's rows; the position holds the row's swizzled chunk
  auto issue = [&](int g, int s) {
    const int r0 = group_row0(g);
    uint16_t *kslot = my_ring + s * 2 * SLOT;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int rl = (i * kWave + lane) / DC;
      const int pos = (i * kWave + lane) % DC;
      const int r = row_of(r0 + rl);
      dma16(kptr(r) + (pos ^ (rl & KSWZ)) * 8, kslot + i * kWave * 8);
      dma16(vptr(r) + (pos ^ (2 * (rl & VSWZ))) * 8, kslot + SLOT + i * kWave * 8);
    }
  };
  // masked full-cache mode: the role bytes of this lane's four score rows
  auto load_roles = [&](int r0) {
    uint32_t roles = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      // the clamped index keeps the load inside the request's rows; rows at or past
      // len are the new token, whose role is CURRENT (see the mask below)
      const int r = r0 + 4 * quarter + i;
      roles |= static_cast<uint32_t>(row_role[base + max(0, min(r, len - 1))]) << (8 * i);
    }
    return roles;
  };

  f32x4 oacc[DB];
#pragma unroll
  for (int i = 0; i < DB; ++i) oacc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m_run = -INFINITY;   // running max (log2 domain) of column col, lagging by at most 8
  float l_run = 0.f;         // this lane's share of the column's sum

  // score fragments: lane (col, quarter) reads row col, d = 32*ks + 8*quarter (chunk 4*ks + quarter)
  const int k_off = col * D;
  // transposed-read geometry (value product): 16-lane group kq reads rows 4*kq + (t >> 2)
  // at d = 16*db + 4*(t & 3), t = lane % 16; lane t then holds V[4*kq .. +3][16*db + t]
  const int tr_row = 4 * quarter + (col >> 2);
  const int tr_off = tr_row * D + 4 * (col & 3);
  const int tr_swz = tr_row & VSWZ;

  auto process = [&](int g, int s) {
    const int r0 = group_row0(g);
    const uint16_t *kslot = my_ring + s * 2 * SLOT;
    const uint32_t roles = MASKED ? load_roles(r0) : 0u;
    f32x4 sacc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const bf16x8 a = *reinterpret_cast<const bf16x8 *>(kslot + k_off + (((4 * ks + quarter) ^ (col & KSWZ)) * 8));
      sacc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, qf[ks], sacc, 0, 0, 0);
    }
    // lane (col, quarter) holds rows r0 + 4*quarter + i of column col
    float x[4];
    float mloc = -INFINITY;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = r0 + 4 * quarter + i;
      bool vis = r < r_end;
      if (MASKED) vis = vis && (r >= len || ((roles >> (8 * i)) & 0xFF) != kText);
      x[i] = vis ? sacc[i] * scale_log2 : -INFINITY;
      mloc = fmaxf(mloc, x[i]);
    }
    mloc = pair32_max(pair16_max(mloc));
    if (__any(mloc > m_run + 8.f)) {   // rescale only when the max grows by more than 2^8
      const float m_new = fmaxf(m_run, mloc);
      const float corr = (m_run == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(m_run - m_new);
      m_run = m_new;
      l_run *= corr;
#pragma unroll
      for (int i = 0; i < DB; ++i) oacc[i] *= corr;
    }
    f32x4 p;
#pragma unroll
    for (int i = 0; i < 4; ++i) p[i] = (x[i] == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(x[i] - m_run);
    // Each probability goes into the product as the sum of two bf16 values, its rounding and
    // the rounding of what that left (2^-17 of it at most): a single one left the output
    // 1.2e-3 to 1.6e-3 from 64 bits, more the fewer ranges a context is cut into (the top key
    // of a range rounds to exactly 1).  The sum is taken over the same rounded values, so
    // the output stays a convex combination of the V rows (see the prefill).  Both values
    // of a lane's four rows share one product of depth 32, whose V operand holds the rows
    // twice: as fast as the one of depth 16 with the single values.
    const bf16x4 pr = __builtin_convertvector(p, bf16x4);
    const f32x4 left = p - __builtin_convertvector(pr, f32x4);
    const bf16x4 pl = __builtin_convertvector(left, bf16x4);
    const bf16x8 pp = __builtin_shufflevector(pr, pl, 0, 1, 2, 3, 4, 5, 6, 7);
    {
      const bf16x2 ones = __builtin_bit_cast(bf16x2, 0x3F803F80u);
      l_run = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pr, pr, 0, 1), ones, l_run, false);
      l_run = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pr, pr, 2, 3), ones, l_run, false);
      l_run = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pl, pl, 0, 1), ones, l_run, false);
      l_run = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pl, pl, 2, 3), ones, l_run, false);
    }
    const uint16_t *vslot = kslot + SLOT;
#pragma unroll
    for (int db = 0; db < DB; ++db) {
      const uint16_t *pa = vslot + tr_off + ((db ^ tr_swz) * 16);
      // C-style cast: the transposing read takes an LDS-qualified pointer
      const v4i16 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16_t *)pa);
      const bf16x8 aa = __builtin_bit_cast(bf16x8, __builtin_shufflevector(a, a, 0, 1, 2, 3, 0, 1, 2, 3));
      oacc[db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aa, pp, oacc[db], 0, 0, 0);
    }
    __builtin_amdgcn_s_waitcnt(15 | (3 << 14) | (7 << 4));   // lgkmcnt(0): slot s may be refilled
  };

  // two-deep pipeline: a slot is refilled as soon as its group has been processed
  int ga = wave, gb = wave + NW;   // the groups in ring slots 0 and 1
  if (!stop) {
    issue(ga, 0);
    issue(gb, 1);
  }
  wait_vm<NG>();                          // Q and slot 0 have landed (slot 1 may not have)
  read_q();
  while (ga < ngroups) {
    process(ga, 0);
    ga += 2 * NW;
    issue(ga, 0);
    wait_vm<NG>();                        // slot 1 has landed (slot 0 may not have)
    if (gb >= ngroups) break;
    process(gb, 1);
    gb += 2 * NW;
    issue(gb, 1);
    wait_vm<NG>();
  }
  wait_vm<0>();   // the trailing (unused) loads, before the ring is reused
  if (appender && !stop && lane < 2 * DC) {
    const size_t dst = static_cast<size_t>(len) * row_stride + (lane % DC) * 8;
    *reinterpret_cast<u32x4 *>((lane < DC ? kbase : vbase) + dst) = *reinterpret_cast<const u32x4 *>(&app_lds[lane * 8]);
  }

  // ---- merge: columns across the four quarters, then the waves through LDS ----
  l_run = pair32_add(pair16_add(l_run));
  if (quarter == 0) {
    m_lds[wave][col] = m_run;
    l_lds[wave][col] = l_run;
  }
  __syncthreads();   // every wave is done with the ring
  const bool stopped = any_stop();
  // [wave][G][DP]: a lane's four values are consecutive d, written at once; with rows of D
  // floats the G heads of a column block all met in one bank
  float *acc_lds = reinterpret_cast<float *>(ring);
  if (col < G) {
#pragma unroll
    for (int db = 0; db < DB; ++db)
      *reinterpret_cast<f32x4 *>(&acc_lds[(wave * G + col) * DP + 16 * db + 4 * quarter]) = oacc[db];
  }
  __syncthreads();

  for (int u = threadIdx.x; u < G * D / 4; u += NW * kWave) {
    const int hh = u / (D / 4), dd = 4 * (u % (D / 4));
    float M = -INFINITY;
#pragma unroll
    for (int w = 0; w < NW; ++w) M = fmaxf(M, m_lds[w][hh]);
    float L = 0.f;
    f32x4 A = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float sc = (m_lds[w][hh] == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(m_lds[w][hh] - M);
      L = fmaf(sc, l_lds[w][hh], L);
      const f32x4 a = *reinterpret_cast<const f32x4 *>(&acc_lds[(w * G + hh) * DP + dd]);
#pragma unroll
      for (int e = 0; e < 4; ++e) A[e] = fmaf(sc, a[e], A[e]);
    }
    if (stopped) break;
    if (whole) {
      const f32x4 o = {A[0] / L, A[1] / L, A[2] / L, A[3] / L};
      *reinterpret_cast<f32x4 *>(orow + 4 * u) = o;
      settle_infinities(u, o, L);
    } else {   // write-through at system scope (see the top of the file)
      __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, A), partial_rsrc(acc_rec), u * 16, split * (G * D * 4),
                                             kSystemScope);
      if (dd == 0) {
        const u32x2 ml = {__float_as_uint(M), __float_as_uint(L)};
        __builtin_amdgcn_raw_buffer_store_b64(ml, partial_rsrc(stat_rec), (split * G + hh) * 8, 0, kSystemScope);
      }
    }
  }
  if (!whole) {
    wait_vm<0>();      // this thread's partial is stored
    __syncthreads();   // ... and every thread's
    finish_pair(stopped);
  } else if (threadIdx.x < kWave) {
    int old = 0;
    if (threadIdx.x == 0) old = count(stopped);
    advance(old);
  }
}

// Splits per (request, kv-head).  With fewer than 256 pairs the grid takes as many splits
// as give every CU a workgroup (64 pairs of 1.3k rows: 4 splits took 13.7 us per call and 5
// took 18.3, with eight waves a workgroup), each of at least 256 rows, and at most 16 (the
// merging split loads sixteen partials per memory round trip; 16 pairs of ~8k rows: 8 splits
// took 19.0 us per call and 16 took 18.5, 22.6 against 24.6 us with the caches cold).  With
// 256 pairs or more, unless the rows are shared (see decode_shape), one split, or three when
// the longest context reaches 2048 rows, so that the longest pairs do not outlast the rest
// of the call when lengths are uneven (512 pairs of 180 .. 4,300 rows: 1 split took 127.7
// us, 2 117.1, 3 111.4, 4 121.3 per call).
static int decode_splits(int batch, int Hkv, int max_ctx) {
  const long pairs = static_cast<long>(batch) * Hkv;
  if (pairs >= 256) return max_ctx >= 2048 ? 3 : 1;
  long s = 256 / pairs;
  const long by_rows = (static_cast<long>(max_ctx) + 255) / 256;
  if (s > by_rows) s = by_rows;
  if (s > kMaxSplits) s = kMaxSplits;
  return static_cast<int>(s < 1 ? 1 : s);
}

// How a call is cut into workgroups.
DecodeShape decode_shape(int batch, int Hkv, int G, int D, int max_ctx, bool masked, size_t part_bytes) {
  DecodeShape sh{decode_splits(batch, Hkv, max_ctx), 0, 8, 0};
  const long pairs = static_cast<long>(batch) * Hkv;
  auto part = [&](long slots) { return static_cast<size_t>(slots) * G * (D + 2) * sizeof(float); };
  // what a call needs, however it is cut: a smaller workspace is refused
  const size_t least = sh.splits > 1 ? part(pairs * sh.splits) : 0;
  // Evenly shared rows (see the kernel) where a call fills the GPU several times over and
  // contexts may be long and uneven.  512 four-wave workgroups are resident, `target` is whole
  // rounds of them: two for 256 pairs, a round more for every 256 pairs (half as many again
  // where contexts may pass 6k rows: a finer cut costs 2 us of 14 with short ranges and gains
  // 10 of 260 with long ones).  Measured against three splits a pair, 32 / 8 heads: 64 contexts
  // of 100 .. 4,000 rows 51.8 us and 58.7, 32 of 100 .. 8,000 47.3 and 51.7, 64 of 4,000 195
  // and 197, 64 of 100 (under a bound of 8,192) 17.2 and 20.5.  From 1,024 pairs on three
  // splits do as well or better (16 / 16 heads, 64 of 100 .. 4,000 rows 117 and, shared, 145).
  // Fewer than 256 pairs keep a split per pair and range: there the plan and the count over
  // the whole call cost 2.4 us of 12 and evenness gains less.
  if (!masked && batch <= kWave && pairs >= 256 && pairs < 1024 && max_ctx >= 2048) {
    const long rounds = std::max(2L, max_ctx < 6144 ? (pairs + 255) / 256 : (3 * pairs + 511) / 512);
    const long target = 512 * rounds / Hkv, launched = target + (batch + 15) / 16;
    if (std::max(least, part(launched * Hkv)) <= part_bytes) {
      sh.target = static_cast<int>(target);
      sh.splits = static_cast<int>(launched);
    }
  }
  const long slots = sh.target > 0 ? static_cast<long>(sh.splits) * Hkv : pairs * sh.splits;
  sh.part_bytes = std::max(least, sh.target > 0 ? part(slots) : 0);
  // Four waves, two workgroups per CU, or eight, one per CU.  Of two workgroups one starts and
  // merges while the other streams; eight waves keep more loads in flight where a CU has one
  // workgroup, and even out contexts of uneven length.  D = 128, 32 / 8 heads, four and eight
  // waves: 512 pairs of 200 rows 13.7 and 18.1 us, 64 of 1.3k rows in four ranges each 12.1 and
  // 13.0, 64 of 64 rows 5.1 and 5.5; 8 pairs of 8k rows 13.0 and 11.8, 400 of 80 .. 1,900 rows
  // 33.0 and 28.0.  Between 256 and 768 workgroups equal contexts would gain from four (400
  // pairs of 500 rows 21.7 and 24.6, 576 of 1,000 55.1 and 60.6) what uneven ones lose, so
  // four are taken there only for short ranges and where one round of 512 is nearly full.
  // D = 64 fits twice on a CU with eight (64 pairs of 4k rows 13.0, with four 13.4).
  const bool tiny = max_ctx <= 256L * sh.splits;
  const bool two = (slots >= 480 && slots <= 512) || slots > 768;
  const bool brief = slots >= 256 && slots < 480 && max_ctx <= 512L * sh.splits;
  if (sh.target > 0 || (!masked && (tiny || (D == 128 && (two || brief))))) sh.waves = 4;
  return sh;
}

// Fixed layout of a scratch array shared by calls of different shapes: the counters
// sit at the same offsets for every call (each call leaves them at zero), the partial
// records after them.  Returns the bytes a call needs, or 0 when its requests or
// (request, kv-head) pairs exceed the fixed counter regions.
size_t decode_scratch_layout(int batch, int Hkv, size_t part_bytes, DecodeWs *ws, char *base) {
  if (batch > kScratchMaxRequests || static_cast<long>(batch) * Hkv > kScratchMaxPairs) return 0;
  if (ws) {
    ws->done = reinterpret_cast<int32_t *>(base);
    ws->arrive = reinterpret_cast<int32_t *>(base + kScratchMaxRequests * sizeof(int32_t));
    ws->part = reinterpret_cast<float *>(base + kScratchCounterBytes);
  }
  return kScratchCounterBytes + part_bytes;
}

size_t decode_ws_layout(int batch, int Hkv, size_t part_bytes, DecodeWs *ws, char *base) {
  const size_t dbytes = (static_cast<size_t>(batch) * sizeof(int32_t) + 255) / 256 * 256;
  const size_t abytes = (static_cast<size_t>(batch) * Hkv * sizeof(int32_t) + 255) / 256 * 256;
  if (ws) {
    ws->done = reinterpret_cast<int32_t *>(base);
    ws->arrive = reinterpret_cast<int32_t *>(base + dbytes);
    ws->part = reinterpret_cast<float *>(base + dbytes + abytes);
  }
  return dbytes + abytes + part_bytes;
}

template <int D, int G>
static void launch_decode_dg(int batch, int Hkv, int max_ctx, const DecodeShape &sh, uint16_t *kc, uint16_t *vc,
                             const int64_t *row_off, const int32_t *row_cap, int32_t *cache_len,
                             const uint8_t *row_role, const uint16_t *q, const uint16_t *k_new, const uint16_t *v_new,
                             float scale_log2, float *out, DecodeWs ws, int32_t *status, hipStream_t stream) {
  const dim3 grid = sh.target > 0 && Hkv * D * 2 >= kLongRow ? dim3(Hkv, sh.splits) : dim3(sh.splits, Hkv, sh.target > 0 ? 1 : batch);
#define GO(MASKED, NW, BAL)                                                                                  \
  decode_kernel<D, G, MASKED, NW, BAL><<<grid, dim3(NW * kWave), 0, stream>>>(                               \
      kc, vc, row_off, row_cap, cache_len, row_role, q, k_new, v_new, out, ws, status, Hkv, sh.splits, max_ctx, \
      batch, sh.target, scale_log2)
  if (row_role != nullptr) GO(true, 8, false);
  else if (sh.target > 0) GO(false, 4, true);
  else if (sh.waves == 4) GO(false, 4, false);
  else GO(false, 8, false);
#undef GO
}

hipError_t launch_decode(int batch, int Hq, int Hkv, int D, int max_ctx, const DecodeShape &sh, uint16_t *kc,
                         uint16_t *vc, const int64_t *row_off, const int32_t *row_cap, int32_t *cache_len,
                         const uint8_t *row_role, const uint16_t *q, const uint16_t *k_new, const uint16_t *v_new,
                         float scale_log2, float *out, const DecodeWs &ws, int32_t *status, hipStream_t stream) {
  const int G = Hq / Hkv;
#define DEC(DD, GG)                                                                                               \
  case GG:                                                                                                        \
    launch_decode_dg<DD, GG>(batch, Hkv, max_ctx, sh, kc, vc, row_off, row_cap, cache_len, row_role, q, \
                             k_new, v_new, scale_log2, out, ws, status, stream);                                  \
    break;
#define DEC_ALL_G(DD)                     \
  switch (G) {                            \
    DEC(DD, 1)                            \
    DEC(DD, 2)                            \
    DEC(DD, 3)                            \
    DEC(DD, 4)                            \
    DEC(DD, 5)                            \
    DEC(DD, 6)                            \
    DEC(DD, 7)                            \
    DEC(DD, 8)                            \
    default: return hipErrorInvalidValue; \
  }
  if (D == 64) {
    DEC_ALL_G(64)
  } else if (D == 128) {
    DEC_ALL_G(128)
  } else {
    return hipErrorInvalidValue;
  }
#undef DEC_ALL_G
#undef DEC
  return hipGetLastError();
}

}  // namespace sonic
