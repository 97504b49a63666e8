// One work item of prefill_kernel, included where it runs: in the kernel's loop, or, for the
// variant that may do an item again, in a function that the loop calls.  (A function for both
// is compiled into other code: 2.7 % slower with the statistics, 1.3 % with the key split.)
//   item       the work item
//   ST         write the statistics
//   alone      RB > 1: a single block of the item's, with the rows and keys up to its end; -1: all
//   ITEM_DONE  leaves the item
const int slot = ws.order[item / Hkv];
const int kvh = item % Hkv;
TileDesc t = ws.tiles[slot];
t.req = __builtin_amdgcn_readfirstlane(t.req);       // uniform: scalar branches and bases
t.p0 = __builtin_amdgcn_readfirstlane(t.p0);
t.nrows = __builtin_amdgcn_readfirstlane(t.nrows);
t.npre = __builtin_amdgcn_readfirstlane(t.npre);
t.seg_start = __builtin_amdgcn_readfirstlane(t.seg_start);
t.seg_len = __builtin_amdgcn_readfirstlane(t.seg_len);
t.ndiag = __builtin_amdgcn_readfirstlane(t.ndiag);
if (RB > 1 && alone >= 0) {
  const int past = max(0, t.nrows - 32 * (alone + 1));
  t.nrows -= past;
  t.seg_len -= past;
  t.ndiag -= past;
}
const int base = rows.seg_row0[t.req];
const int64_t pbase = rows.pre_row0 != nullptr ? rows.pre_row0[t.req] : static_cast<int64_t>(base);
const int h = kvh * G + head;
const int nv = tile_key_count(t);
const int nF = nv - t.ndiag;
const int npre = t.npre;
const int seg_shift = t.seg_start - npre;    // request position of virtual key vk >= npre
const size_t tok_stride = static_cast<size_t>(Hkv) * D;
const size_t head0 = static_cast<size_t>(base) * tok_stride + static_cast<size_t>(kvh) * D;
const size_t phead0 = static_cast<size_t>(pbase) * tok_stride + static_cast<size_t>(kvh) * D;
// row 0 of the request (and of its prefix rows) for this kv-head; rows are
// row_bytes apart, and every row of a request lies below 4 GiB from its row 0
const char *kreq = uniform_ptr(reinterpret_cast<const char *>(rows.seg_k + head0));
const char *vreq = uniform_ptr(reinterpret_cast<const char *>(rows.seg_v + head0));
const char *kpre = uniform_ptr(reinterpret_cast<const char *>(rows.pre_k + phead0));
const char *vpre = uniform_ptr(reinterpret_cast<const char *>(rows.pre_v + phead0));

// RB > 1: a wave whose block lies past the end of a short run only stages, which leaves the LDS
// and the matrix cores to the others (8,000 runs of 3 rows, one q-head of 64: 1,385 us without)
const bool rowless = RB > 1 && row_blk >= t.nrows;

const int nchunks = (nv + kKeyChunk - 1) / kKeyChunk;
// this group's steps: [c_first, c_first + nloc); loads for steps past them
// (the pipeline runs two ahead) fetch a step past the list end instead
const int nloc = KS == 1 ? nchunks : (nchunks + 1) / 2;
const int c_first = grp * nloc;
const int c_stop = c_first + nloc;
auto stage_step = [&](int c) { return (KS == 1 || c < c_stop) ? c : max(c, nchunks); };
auto stage_k = [&](int c, uint16_t *buf) {
  stage_tensor<D, NW, false>(buf, kpre, kreq, row_bytes, koff_lane, wave, lane, stage_step(c), nv, npre,
                            seg_shift);
};
auto stage_v = [&](int c, uint16_t *buf) {
  stage_tensor<D, NW, true>(buf, vpre, vreq, row_bytes, voff_lane, wave, lane, stage_step(c), nv, npre,
                           seg_shift);
};

// Q^T fragments (B operand of S): lane (row n, half g) holds d = 16*ds + 8*g .. +7.
bf16x8 qf[DS];
{
  const bool ok = row_blk + n < t.nrows;
  const uint16_t *qrow = q + (static_cast<size_t>(base + t.p0 + row_blk + n) * Hq + h) * D;
#pragma unroll
  for (int ds = 0; ds < DS; ++ds) {
    u32x4 w = {0u, 0u, 0u, 0u};
    if (ok) w = *reinterpret_cast<const u32x4 *>(qrow + 16 * ds + 8 * g);
    qf[ds] = __builtin_bit_cast(bf16x8, w);
  }
}

f32x16 oacc[DB];
#pragma unroll
for (int i = 0; i < DB; ++i) oacc[i] = f32x16{};
float m_run = -INFINITY;   // running max in the log2 domain (lags by at most kLazy)
float l_run = 0.f;         // sum of the bf16-rounded probabilities the P.V product uses
float l_ex = 0.f;          // STATS: the same sum before rounding (normaliser, Nexus mass)
float l_nex = 0.f;         // STATS: the part of l_ex from Nexus keys
// STATS: Nexus keys are the virtual keys [nex_lo, npre) (the prefix past the system rows)
const int nex_lo = ST ? min(ws.req[t.req].system, npre) : npre;

// One 64-key step: compute on (kc_lds, vc_lds) while step c + 1 streams into
// (kn_lds, vn_lds).
// Pipeline, per wave: K of step c + 2 is requested as soon as every wave has
// finished S(c), V of step c + 1 as soon as every wave has finished P.V(c - 1).
// Each wave issues exactly NJ direct-to-LDS instructions per tensor and step,
// in the order K(0) V(0) K(1) | V(1) K(2) | V(2) K(3) | ..., also for steps past
// the end of the key list (those load key 0 and are never read).  So at the start
// of step c the loads newer than K(c) are V(c) and K(c+1), and in its middle the
// loads newer than V(c) are K(c+1) and V(c+1): both waits are "all but the 2 * NJ
// most recent", the same at every step.
constexpr int NJ = ((kKeyChunk / (kWave / (D / 8))) + NW - 1) / NW;
static_assert(2 * NJ < 64, "the wait count fits vmcnt");
__builtin_assume(wave < NW);
auto step = [&](int c, uint16_t *kc_lds, const uint16_t *vc_lds, uint16_t *vn_lds) {
  wait_vm<2 * NJ>();
  lds_barrier();                                   // K(c) in LDS; every wave is past P.V(c - 1)
  stage_v(c + 1, vn_lds);
  const int vk0 = c * kKeyChunk;
  if (rowless) {
    wait_vm<2 * NJ>();
    lds_barrier();
    stage_k(c + 2, kc_lds);
    return;
  }

  // ---- S^T = K . Q^T for two 32-key blocks ----
  f32x16 sacc[2];
#pragma unroll
  for (int kb = 0; kb < 2; ++kb) {
    sacc[kb] = f32x16{};
    const int m = kb * 32 + n;
#pragma unroll
    for (int ds = 0; ds < DS; ++ds) {
      const bf16x8 a =
          *reinterpret_cast<const bf16x8 *>(&kc_lds[(m * DC + ((2 * ds + g) ^ swz_k<D>(m))) * 8]);
      sacc[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qf[ds], sacc[kb], 0, 0, 0);
    }
  }
  order_reads_ahead<2 * DS, 1, kAheadS>();

  wait_vm<2 * NJ>();
  lds_barrier();                                   // V(c) in LDS; every wave is past S(c)
  stage_k(c + 2, kc_lds);
  // ---- mask (ragged end / causal diagonal only), online softmax ----
  if (vk0 + kKeyChunk > nF) {
    // Row n sees every key before the diagonal block and diagonal keys j <= n:
    // virtual key vk is visible iff vk < min(nv, nF + n + 1) (n counted in the item).  One compare and a
    // select per element, no divergent branches.
    const int lim_g = min(nv, nF + row_blk + n + 1) - vk0 - 8 * g;   // bound on acc_key0
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int e = 0; e < 16; ++e)
        sacc[kb][e] = (kb * 32 + acc_key0(e) < lim_g) ? sacc[kb][e] : -INFINITY;
  }
  float mloc = -INFINITY;
#pragma unroll
  for (int kb = 0; kb < 2; ++kb)
#pragma unroll
    for (int e = 0; e < 16; ++e) mloc = fmaxf(mloc, sacc[kb][e]);
  mloc = pair32_max(mloc) * scale_log2;
  if (__any(mloc > m_run + kLazy)) {
    const float m_new = fmaxf(m_run, mloc);
    const float corr = __builtin_amdgcn_exp2f(m_run - m_new);
    m_run = m_new;
    l_run *= corr;
    if (ST) {
      l_ex *= corr;
      l_nex *= corr;
    }
#pragma unroll
    for (int db = 0; db < DB; ++db) oacc[db] *= corr;
  }
  // STATS: this step's Nexus keys are step-local keys [nx0, nx1)
  const int nx0 = max(nex_lo - vk0, 0), nx1 = min(npre - vk0, kKeyChunk);
  const bool nex_all = ST && nx0 == 0 && nx1 == kKeyChunk;
  const bool nex_some = ST && nx0 < nx1 && !nex_all;
  const int nx0_g = nx0 - 8 * g, nx1_g = nx1 - 8 * g;   // the same range on acc_key0
  float lsum = 0.f, nsum = 0.f;
  bf16x8 pb[4];
#pragma unroll
  for (int kb = 0; kb < 2; ++kb) {
    f32x8 lo, hi;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      lo[e] = __builtin_amdgcn_exp2f(fmaf(sacc[kb][e], scale_log2, -m_run));
      hi[e] = __builtin_amdgcn_exp2f(fmaf(sacc[kb][8 + e], scale_log2, -m_run));
      if (ST) lsum += lo[e] + hi[e];
      if (nex_some) {
        const int klo = kb * 32 + acc_key0(e), khi = kb * 32 + acc_key0(8 + e);
        nsum += ((klo >= nx0_g && klo < nx1_g) ? lo[e] : 0.f) + ((khi >= nx0_g && khi < nx1_g) ? hi[e] : 0.f);
      }
    }
    pb[2 * kb] = __builtin_convertvector(lo, bf16x8);
    pb[2 * kb + 1] = __builtin_convertvector(hi, bf16x8);
  }
  // The output is normalised by the sum of the rounded probabilities themselves, so
  // that it stays a convex combination of the V rows: a row dominated by one key then
  // loses nothing to the rounding of that key's probability (which the lagging max
  // leaves anywhere in [1, 2^8), not exactly 1).  v_dot2c_f32_bf16 against (1, 1)
  // adds a packed pair of them in one instruction.
  l_run += rounded_sum(pb);
  if (ST) l_ex += lsum;
  if (nex_all) l_nex += lsum;
  if (nex_some) l_nex += nsum;

  // ---- O^T += V^T . P^T, V^T operands read transposed from row-major V ----
#pragma unroll
  for (int db = 0; db < DB; ++db) {
    const int dd = db * 32 + v_d_off;     // this lane's 4 d-values, a 4-aligned start
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      v4i16 part[2];
#pragma unroll
      for (int hh = 0; hh < 2; ++hh) {
        const int r = 16 * ks + 4 * hh + v_row_off;
        const int chunk = (dd >> 3) ^ swz_v<D>(r);
        const uint16_t *pa = &vc_lds[r * D + chunk * 8 + (dd & 4)];
        part[hh] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16_t *)pa);
      }
      const u32x4 w = {__builtin_bit_cast(uint2, part[0]).x, __builtin_bit_cast(uint2, part[0]).y,
                       __builtin_bit_cast(uint2, part[1]).x, __builtin_bit_cast(uint2, part[1]).y};
      oacc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, w), pb[ks], oacc[db], 0,
                                                         0, 0);
    }
  }
  order_reads_ahead<4 * DB, 2, kAheadPV>();
};

stage_k(c_first, kbuf0);
stage_v(c_first, vbuf0);
stage_k(c_first + 1, kbuf1);
step(c_first, kbuf0, vbuf0, vbuf1);
for (int c = 1; c < nloc; c += 2) {
  step(c_first + c, kbuf1, vbuf1, vbuf0);
  if (c + 1 >= nloc) break;
  step(c_first + c + 1, kbuf0, vbuf0, vbuf1);
}

if constexpr (KS == 2) {
  // the second group hands its partial to the first: wave w's O into buffer w
  // (lane-minor, so both sides touch consecutive words), max and sum into ml_lds
  wait_vm<0>();
  __syncthreads();                 // every wave past its last step's LDS reads and loads
  uint16_t *const ob = wave < 4 ? (wave < 2 ? k_lds0[wave & 1] : k_lds1[wave & 1])
                                : (wave < 6 ? v_lds0[wave & 1] : v_lds1[wave & 1]);
  float *const xo = reinterpret_cast<float *>(ob);
  if (grp == 1) {
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int e = 0; e < 16; ++e) xo[(db * 16 + e) * kWave + lane] = oacc[db][e];
    ml_lds[(2 * wave) * kWave + lane] = m_run;
    ml_lds[(2 * wave + 1) * kWave + lane] = l_run;
  }
  __syncthreads();
  if (grp == 1) ITEM_DONE;         // the loop head's barrier waits for the first group
  const float m1 = ml_lds[(2 * wave) * kWave + lane];
  const float l1 = ml_lds[(2 * wave + 1) * kWave + lane];
  // A group that saw no key of this row (its steps were past the list end) kept
  // the max at -inf, and its sum and O are NaN (-inf - -inf in the exponent):
  // select them away rather than scale them by zero.
  const bool has0 = m_run != -INFINITY, has1 = m1 != -INFINITY;
  const float mm = fmaxf(m_run, m1);
  const float c0 = has0 ? __builtin_amdgcn_exp2f(m_run - mm) : 0.f;
  const float c1 = has1 ? __builtin_amdgcn_exp2f(m1 - mm) : 0.f;
  l_run = (has0 ? l_run * c0 : 0.f) + (has1 ? l1 * c1 : 0.f);
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const float x = xo[(db * 16 + e) * kWave + lane];
      oacc[db][e] = (has0 ? oacc[db][e] * c0 : 0.f) + (has1 ? x * c1 : 0.f);
    }
}

// ---- normalise and store: lane (n, g) holds d = 32*db + 8*i + 4*g + (0..3) ----
const float l_tot = pair32_add(l_run);
const float inv = 1.f / l_tot;
if constexpr (RB > 1) {
  if (alone >= 0) {
    if (row_blk != 32 * alone) ITEM_DONE;
  } else if (t.ndiag > 0) {
    float sum = 0.f;
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int e = 0; e < 16; ++e) sum += oacc[db][e];
    if (__any(sum != sum && row_blk + n < t.nrows) && lane == 0) s_again = 1;
  }
}
if (ST) {
  const float n_tot = pair32_add(l_nex);
  const float x_tot = pair32_add(l_ex);
  if (row_blk + n < t.nrows && g == 0) {
    const size_t idx = static_cast<size_t>(base + t.p0 + row_blk + n) * Hq + h;
    if (rows.nexus_mass != nullptr) rows.nexus_mass[idx] = n_tot / x_tot;
    rows.lse[idx] = m_run + __builtin_amdgcn_logf(x_tot);
  }
}
if (row_blk + n < t.nrows) {
  float *orow = out + (static_cast<size_t>(base + t.p0 + row_blk + n) * Hq + h) * D;
#pragma unroll
  for (int db = 0; db < DB; ++db) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      f32x4 o = {oacc[db][4 * i] * inv, oacc[db][4 * i + 1] * inv, oacc[db][4 * i + 2] * inv,
                 oacc[db][4 * i + 3] * inv};
      *reinterpret_cast<f32x4 *>(orow + db * 32 + 8 * i + 4 * g) = o;
    }
  }
}
