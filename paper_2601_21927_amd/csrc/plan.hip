// Prefill planner: layout grammar, segment table and visible-key descriptors.
//
// The mask of Sec. 3.2 depends only on (role, segment) runs, so the planner
// works run by run instead of materialising an L x L mask:
//   * a system row sees the system rows before it (Eq.(3));
//   * a body row of segment i sees the system prompt, every Nexus token of the
//     earlier segments (causal; A1), and its own body up to itself; earlier
//     bodies are removed because the row lies after their segment (Eq.(4));
//   * a Nexus row of segment i sees the system prompt, its own body (it is not
//     after max(N_i)) and every Nexus token of the request (Eq.(5)), or, with the
//     narrower Nexus scope, those of segments 1..i only: a shorter leading part
//     of the same prefix;
//   * a current-query row sees the system prompt, every Nexus token and the
//     current query up to itself; all bodies are removed (Eq.(4)).
// Every block of at most 32 rows of one run therefore sees the same key list
// apart from its own causal diagonal.  With the request's system and Nexus rows
// copied, in order, into one contiguous "prefix" (system prompt first, then the
// Nexus tokens segment by segment), that list is "a leading part of the prefix,
// then one contiguous range of the request ending in the block's own rows".
// One TileDesc per block encodes it; masked key blocks are never enumerated.
//
// Work order: requests by decreasing total cost, and inside a request its blocks
// by decreasing cost.  Blocks of one request run close together in time, so the
// K/V rows they share (system prompt, Nexus tokens, bodies) stay in the L2 of
// the XCD that serves them.
#include "common.h"
#include "scan.h"

namespace sonic {

constexpr int kPlanThreads = 1024;
constexpr int kPlanTok = 8;        // tokens per thread in the run kernel's pass 1
constexpr int kCostBuckets = 1024;

// One step of the grammar SYSTEM* (TEXT+ NEXUS*)* CURRENT* of Eq.(1): may a token
// with role r and segment id t follow one with role rp and id tp (rp = -1 at the
// first token of a request)?  Segment ids are constant within a segment and
// strictly increase between segments.  Per pair of roles, which orders of the ids are
// allowed (1: t < tp, 2: equal, 4: t > tp), packed in one word: as branches for each of a
// thread's eight tokens the grammar was most of the kernel's code.
constexpr uint64_t allow(int rp, int r, int orders) { return static_cast<uint64_t>(orders) << (3 * (4 * (rp + 1) + r)); }
constexpr uint64_t kGrammar =
    allow(-1, kSystem, 7) | allow(-1, kText, 7) | allow(-1, kCurrent, 7) |
    allow(kSystem, kSystem, 7) | allow(kSystem, kText, 7) | allow(kSystem, kCurrent, 7) |
    allow(kText, kText, 6) | allow(kText, kNexus, 2) | allow(kText, kCurrent, 7) |
    allow(kNexus, kNexus, 2) | allow(kNexus, kText, 4) | allow(kNexus, kCurrent, 7) |
    allow(kCurrent, kCurrent, 7);
static_assert(kSystem == 0 && kText == 1 && kNexus == 2 && kCurrent == 3, "roles index the grammar");
__device__ __forceinline__ bool legal_step(int rp, int tp, int r, int t) {
  const int order = t < tp ? 1 : (t == tp ? 2 : 4);
  const int i = 4 * (rp + 1) + r;
  return r <= kCurrent && rp <= kCurrent && ((kGrammar >> (3 * (i & 31) & 63)) & order) != 0;
}

// One workgroup per request: validate, list the Nexus positions and the runs,
// then emit one descriptor per block of up to tile_rows rows of a run.
__global__ __launch_bounds__(kPlanThreads) void plan_runs_kernel(const int32_t *__restrict__ cu,
                                                                 const uint8_t *__restrict__ role,
                                                                 const int32_t *__restrict__ turn, PrefillWs ws,
                                                                 int total_tokens, int nexus_scope, int tile_rows,
                                                                 int32_t *status) {
  __shared__ int lds[kPlanThreads / kWave];
  __shared__ int lds4[4 * (kPlanThreads / kWave)];
  __shared__ int4 s_run[kPlanThreads];
  __shared__ int s_first[kPlanThreads];
  __shared__ unsigned long long s_cost;
  const int b = blockIdx.x;
  if (threadIdx.x == 0) s_cost = 0ull;
  const int s = cu[b];
  const int e = cu[b + 1];
  // cu_seqlens itself is malformed: requests may overlap, in the caller's arrays and in the
  // workspace, so none of them is planned (every wave looks at all of it)
  int malformed = 0;
  for (int i = threadIdx.x % kWave; i < static_cast<int>(gridDim.x); i += kWave) {
    const int si = cu[i], ei = cu[i + 1];
    malformed |= si < 0 || ei < si || ei > total_tokens;
  }
  if (__any(malformed)) {
    if (threadIdx.x == 0) {
      raise_status(status, SONIC_ERR_BAD_LAYOUT);
      ws.req[b] = ReqInfo{0, 0, 0, 0, 0, 0};
    }
    return;
  }
  const int L = e - s;

  // Pass 1: grammar, prefix rows (system and Nexus positions, in order), run starts
  // with the number of prefix rows before each.  In a well-formed request the
  // system rows come first, so the prefix is the system prompt followed by the
  // Nexus tokens.  Each thread takes kPlanTok consecutive tokens (one chunk of
  // kPlanThreads * kPlanTok tokens covers most requests): it counts them, one
  // block scan places its entries, and a second walk over its registers writes
  // them.  A token's predecessor is the thread's previous token, or the lower
  // lane's last one (lane 0 loads its own).
  // (Requesting the next chunk's tokens ahead spilled 48 registers, 14 with the tokens as loaded:
  // a request of 88k tokens took 248 us of prefill, then 236, and takes 226 without.)
  int pre_carry = 0, run_carry = 0, nexus_count = 0, bad_count = 0;
  const int lane = threadIdx.x % kWave;
  struct Tokens {   // as loaded
    uint64_t r;     // eight roles (0xFF past the end)
    u32x4 ta, tb;   // eight ids
    int rp, tp;     // role and id before the first (lane 0)
  };
  auto load = [&](int base, Tokens &k) {
    const int i0 = base + threadIdx.x * kPlanTok;
    static_assert(kPlanTok == 8, "one 8-byte and two 16-byte loads");
    if (i0 + kPlanTok <= L) {
      __builtin_memcpy(&k.r, role + s + i0, 8);
      __builtin_memcpy(&k.ta, turn + s + i0, 16);
      __builtin_memcpy(&k.tb, turn + s + i0 + 4, 16);
    } else {
      k.r = ~0ull;
      k.ta = k.tb = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
      for (int j = 0; j < kPlanTok; ++j) {
        if (i0 + j < L) {
          k.r = (k.r & ~(0xFFull << (8 * j))) | (static_cast<uint64_t>(role[s + i0 + j]) << (8 * j));
          (j < 4 ? k.ta : k.tb)[j & 3] = static_cast<uint32_t>(turn[s + i0 + j]);
        }
      }
    }
    k.rp = -1;
    k.tp = 0;
    if (lane == 0 && i0 > 0 && i0 <= L) {
      k.rp = role[s + i0 - 1];
      k.tp = turn[s + i0 - 1];
    }
  };
  Tokens cur;
  constexpr int kChunk = kPlanThreads * kPlanTok;
  for (int base = 0; base < L; base += kChunk) {
    load(base, cur);
    const int i0 = base + threadIdx.x * kPlanTok;
    int r[kPlanTok], t[kPlanTok];
#pragma unroll
    for (int j = 0; j < kPlanTok; ++j) {
      r[j] = static_cast<int>((cur.r >> (8 * j)) & 0xFF);
      t[j] = static_cast<int>(j < 4 ? cur.ta[j & 3] : cur.tb[j & 3]);
    }
    int rp = __shfl_up(r[kPlanTok - 1], 1), tp = __shfl_up(t[kPlanTok - 1], 1);
    if (lane == 0) {
      rp = cur.rp;
      tp = cur.tp;
    }
    // bit j: token j is a prefix row, starts a run, is a Nexus token, breaks the grammar
    uint32_t pre = 0, start = 0, nexus = 0, bad = 0;
#pragma unroll
    for (int j = 0; j < kPlanTok; ++j) {
      const uint32_t in = i0 + j < L ? 1u << j : 0u;
      pre |= (r[j] == kSystem || r[j] == kNexus) ? in : 0u;
      start |= (i0 + j == 0 || r[j] != rp || (r[j] == kText && t[j] != tp)) ? in : 0u;
      nexus |= r[j] == kNexus ? in : 0u;
      bad |= legal_step(rp, tp, r[j], t[j]) ? 0u : in;
      rp = r[j];
      tp = t[j];
    }
    const int cnt[4] = {static_cast<int>(__popc(pre)), static_cast<int>(__popc(start)), static_cast<int>(__popc(nexus)),
                        static_cast<int>(__popc(bad))};
    int below[4], tot[4];
    block_int_scan_n<kPlanThreads, 4>(cnt, below, tot, lds4);
    const int pc0 = pre_carry + below[0], rc0 = run_carry + below[1];
#pragma unroll
    for (int j = 0; j < kPlanTok; ++j) {
      const uint32_t lower = (1u << j) - 1u;
      const int pc = pc0 + __popc(pre & lower);
      if ((start >> j) & 1) {
        const int rc = rc0 + __popc(start & lower);
        ws.runs[s + rc] = make_int2(i0 + j, pc);
        if (rc < kPlanThreads) s_run[rc] = make_int4(i0 + j, pc, r[j], 0);
      }
      if ((pre >> j) & 1) ws.prefix_pos[s + pc] = i0 + j;
    }
    pre_carry += tot[0];
    run_carry += tot[1];
    nexus_count += tot[2];
    bad_count += tot[3];
  }
  __syncthreads();
  if (bad_count) {
    if (threadIdx.x == 0) {
      raise_status(status, SONIC_ERR_BAD_LAYOUT);
      ws.req[b] = ReqInfo{0, 0, 0, 0, 0, 0};
    }
    return;
  }
  const int nruns = run_carry;
  const int k_tot = nexus_count;
  // run i: start, prefix rows before it, role; the first kPlanThreads runs are in LDS
  auto run_at = [&](int i) {
    if (i < kPlanThreads) return s_run[i];
    const int2 x = ws.runs[s + i];
    return make_int4(x.x, x.y, role[s + x.x], 0);
  };
  int S = 0;
  if (L > 0 && s_run[0].z == kSystem) S = nruns > 1 ? s_run[1].x : L;
  const int npre_all = S + k_tot;

  // Pass 2: descriptors.  A thread sizes one run, then the threads share the blocks of
  // these runs and find each one's run in the list of first blocks.
  int tile_carry = 0;
  int64_t cost = 0;
  for (int rb = 0; rb < nruns; rb += kPlanThreads) {
    const int cnt = min(kPlanThreads, nruns - rb);
    int nt = 0;
    if (threadIdx.x < cnt) {
      const int r = rb + threadIdx.x;
      nt = ((r + 1 < nruns ? run_at(r + 1).x : L) - run_at(r).x + tile_rows - 1) / tile_rows;
    }
    int ttot;
    s_first[threadIdx.x] = block_int_scan<kPlanThreads>(nt, &ttot, lds);
    __syncthreads();
    for (int i = threadIdx.x; i < ttot; i += kPlanThreads) {
      int lo = 0, hi = cnt;   // s_first[lo] <= i < s_first[hi]; every run has a block
      while (hi - lo > 1) {
        const int mid = (lo + hi) / 2;
        if (s_first[mid] <= i) lo = mid;
        else hi = mid;
      }
      const int r = rb + lo;
      const int4 run = run_at(r);
      const int start = run.x, pre_before = run.y, kind = run.z;
      const int end = r + 1 < nruns ? run_at(r + 1).x : L;
      TileDesc d;
      d.req = b;
      d.p0 = start + (i - s_first[lo]) * tile_rows;
      d.nrows = min(tile_rows, end - d.p0);
      d.pad = 0;
      if (kind == kSystem) {          // system rows before the block, then the block
        d.npre = d.p0;
        d.seg_start = d.p0;
        d.seg_len = d.nrows;
        d.ndiag = d.nrows;
      } else if (kind == kText) {     // system + earlier Nexus, own body up to the block
        d.npre = pre_before;
        d.seg_start = start;
        d.seg_len = d.p0 + d.nrows - start;
        d.ndiag = d.nrows;
      } else if (kind == kNexus) {    // system + every Nexus (or up to its own), the owning body:
        const int body = run_at(r - 1).x;   // the grammar puts its run right before
        d.npre = nexus_scope == SONIC_NEXUS_ALL ? npre_all : pre_before + (end - start);
        d.seg_start = body;
        d.seg_len = start - body;
        d.ndiag = 0;
      } else {                        // system + every Nexus, current query up to the block
        d.npre = npre_all;
        d.seg_start = start;
        d.seg_len = d.p0 + d.nrows - start;
        d.ndiag = d.nrows;
      }
      ws.tiles[s + tile_carry + i] = d;
      cost += tile_cost(d);
    }
    tile_carry += ttot;
    __syncthreads();   // s_first is rewritten
  }
  if (cost > 0) atomicAdd(&s_cost, static_cast<unsigned long long>(cost));
  __syncthreads();
  if (threadIdx.x == 0) ws.req[b] = ReqInfo{tile_carry, S, k_tot, nruns, static_cast<int64_t>(s_cost), 0};
}

// One workgroup per request: its descriptors by decreasing cost (a histogram
// sort over kCostBuckets cost values, larger costs share the last bucket), from
// its first slot in `order`.  Requests run by decreasing total cost (ties by
// index), so that first slot is the number of descriptors of the requests ranked
// before it: a workgroup sum over the batch, no global sort.  Workgroup 0 also
// writes the descriptor count (`ok`: 0 where it found an error pending) and resets the queues.
__device__ __forceinline__ void plan_order(int b, bool ok, int batch, const int32_t *__restrict__ cu, const PrefillWs &ws,
                                           int *hist, int *lds) {
  static_assert(kCostBuckets == kPlanThreads, "one histogram bucket per thread");
  hist[threadIdx.x] = 0;
  if (b == 0 && threadIdx.x < kNumXcd) ws.ctrl[8 + threadIdx.x] = 0;
  const int64_t cb = ws.req[b].cost;
  int before = 0, all = 0;
  for (int j0 = 0; j0 < batch; j0 += kPlanThreads) {
    const int j = j0 + threadIdx.x;
    int nt_j = 0, nb = 0;
    if (j < batch) {
      const ReqInfo rj = ws.req[j];
      nt_j = rj.ntiles;
      nb = (rj.cost > cb || (rj.cost == cb && j < b)) ? nt_j : 0;
    }
    const int x[2] = {nb, nt_j};
    int below[2], total[2];
    block_int_scan_n<kPlanThreads, 2>(x, below, total, lds);
    before += total[0];
    all += total[1];
  }
  if (b == 0 && threadIdx.x == 0) ws.ctrl[0] = ok ? all : 0;
  const int nt = ws.req[b].ntiles;
  const int base = cu[b];
  const int dst = before;
  __syncthreads();   // hist is clear
  for (int j = threadIdx.x; j < nt; j += kPlanThreads) {
    const int c = min(tile_cost(ws.tiles[base + j]), kCostBuckets - 1);
    atomicAdd(&hist[kCostBuckets - 1 - c], 1);
  }
  __syncthreads();
  int total;
  const int off = block_int_scan<kPlanThreads>(hist[threadIdx.x], &total, lds);
  hist[threadIdx.x] = off;
  __syncthreads();
  for (int j = threadIdx.x; j < nt; j += kPlanThreads) {
    const int c = min(tile_cost(ws.tiles[base + j]), kCostBuckets - 1);
    const int pos = atomicAdd(&hist[kCostBuckets - 1 - c], 1);
    ws.order[dst + pos] = base + j;
  }
}

// Prefix copies: row j < S + K_tot of request b's prefix gets the K and V rows
// of position prefix_pos[cu[b] + j].  Workgroups gx*b .. gx*b + gx-1 copy request
// b's prefix, one wave per kGatherRows consecutive rows, waves striding over the
// prefix.  The wave's first lanes read the rows' positions, then every
// lane has all of its 16-byte pieces of those rows in flight before it stores
// (kGatherPieces per row and tensor at a time).
constexpr int kGatherWaves = kPlanThreads / kWave;
constexpr int kGatherRows = 4;
constexpr int kGatherPieces = 2;

__device__ __forceinline__ void gather_prefix(int b, int bx, int gx, const int32_t *__restrict__ cu,
                                              const uint16_t *__restrict__ k, const uint16_t *__restrict__ v,
                                              const PrefillWs &ws, int row_pieces) {
  const int s0 = cu[b];
  const ReqInfo ri = ws.req[b];
  const int npre = ri.system + ri.nexus_total;
  const int lane = threadIdx.x % kWave;
  const int wave = threadIdx.x / kWave;
  const u32x4 *__restrict__ k4 = reinterpret_cast<const u32x4 *>(k);
  const u32x4 *__restrict__ v4 = reinterpret_cast<const u32x4 *>(v);
  u32x4 *__restrict__ kd = reinterpret_cast<u32x4 *>(ws.k_pre);
  u32x4 *__restrict__ vd = reinterpret_cast<u32x4 *>(ws.v_pre);
  const int stride = gx * kGatherWaves * kGatherRows;
  for (int j0 = (bx * kGatherWaves + wave) * kGatherRows; j0 < npre; j0 += stride) {
    int src = -1;   // lane u < kGatherRows: source row of copy row j0 + u, or -1 past the prefix
    if (lane < kGatherRows && j0 + lane < npre) src = s0 + ws.prefix_pos[s0 + j0 + lane];
    int sr[kGatherRows];
#pragma unroll
    for (int u = 0; u < kGatherRows; ++u) sr[u] = __builtin_amdgcn_readlane(src, u);
    for (int c0 = 0; c0 < row_pieces; c0 += kGatherPieces * kWave) {
      u32x4 kr[kGatherRows][kGatherPieces], vr[kGatherRows][kGatherPieces];
#pragma unroll
      for (int u = 0; u < kGatherRows; ++u)
#pragma unroll
        for (int p = 0; p < kGatherPieces; ++p) {
          const int c = c0 + p * kWave + lane;
          if (sr[u] >= 0 && c < row_pieces) {
            kr[u][p] = k4[static_cast<size_t>(sr[u]) * row_pieces + c];
            vr[u][p] = v4[static_cast<size_t>(sr[u]) * row_pieces + c];
          }
        }
#pragma unroll
      for (int u = 0; u < kGatherRows; ++u)
#pragma unroll
        for (int p = 0; p < kGatherPieces; ++p) {
          const int c = c0 + p * kWave + lane;
          if (sr[u] >= 0 && c < row_pieces) {
            const size_t dst = static_cast<size_t>(s0 + j0 + u) * row_pieces + c;
            kd[dst] = kr[u][p];
            vd[dst] = vr[u][p];
          }
        }
    }
  }
}

// Both need only the run kernel's results: workgroups [0, batch) order a request's
// descriptors, the others copy prefixes (one launch after the other, the order took 6 us
// of its own before a copy of 19).  Only workgroup 0 looks at the status word, which may change
// at any time: where it gives a descriptor count, every slot below it has to be filled.
__global__ __launch_bounds__(kPlanThreads) void plan_finish_kernel(int batch, const int32_t *__restrict__ cu,
                                                                   const uint16_t *__restrict__ k,
                                                                   const uint16_t *__restrict__ v, PrefillWs ws,
                                                                   int row_pieces, int gx, const int32_t *status) {
  __shared__ int hist[kCostBuckets];
  __shared__ int lds[2 * (kPlanThreads / kWave)];
  __shared__ int s_ok;
  const bool ok = blockIdx.x != 0 || block_status_clear(status, &s_ok);
  const int w = static_cast<int>(blockIdx.x) - batch;
  if (w < 0) plan_order(blockIdx.x, ok, batch, cu, ws, hist, lds);
  else gather_prefix(w / gx, w % gx, gx, cu, k, v, ws, row_pieces);
}

// Grammar check and run table only (ws.req, ws.prefix_pos, ws.runs; ws.tiles is
// written as scratch), for callers that need the segment structure but no prefill.
hipError_t launch_plan_runs(int batch, int total_tokens, const int32_t *cu, const uint8_t *role, const int32_t *turn,
                            PrefillWs ws, int32_t *status, hipStream_t stream) {
  plan_runs_kernel<<<dim3(batch), dim3(kPlanThreads), 0, stream>>>(cu, role, turn, ws, total_tokens,
                                                                    SONIC_NEXUS_ALL, kTileRows, status);
  return hipGetLastError();
}

hipError_t launch_plan(int batch, int total_tokens, int Hkv, int D, int nexus_scope, int tile_rows, const int32_t *cu,
                       const uint8_t *role, const int32_t *turn, const uint16_t *k, const uint16_t *v, PrefillWs ws,
                       int32_t *status, hipStream_t stream) {
  plan_runs_kernel<<<dim3(batch), dim3(kPlanThreads), 0, stream>>>(cu, role, turn, ws, total_tokens, nexus_scope,
                                                                    tile_rows, status);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int row_pieces = Hkv * D / 8;
  // about two workgroups per CU over the batch, none with nothing but rows past every prefix
  constexpr int rows_per_block = kGatherWaves * kGatherRows;
  const int by_rows = (total_tokens + rows_per_block - 1) / rows_per_block;
  const int gx = max(1, min((512 + batch - 1) / batch, by_rows));
  plan_finish_kernel<<<dim3(batch + gx * batch), dim3(kPlanThreads), 0, stream>>>(batch, cu, k, v, ws, row_pieces, gx,
                                                                                  status);
  return hipGetLastError();
}

}  // namespace sonic
