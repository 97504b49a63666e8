"""Decode over the compacted cache on the GPU against the fp64 oracle."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import decode as OD
from paper_2601_21927_amd import sonic
from paper_2601_21927_amd.runner import bf16_to_device, bf16_to_host
from tests import gpu_helpers as H

pytestmark = pytest.mark.gpu


def compacted(batch, extra_rows):
    """Compact the batch on the GPU (its bit-exactness is tested elsewhere) and check it here too."""
    db = H.device_batch(batch)
    kept = H.kept_counts(batch)
    cache = db.alloc_cache(kept + extra_rows)
    assert db.compact() == sonic.OK
    torch.cuda.synchronize()
    assert db.read_status() == 0
    kc, vc, ki, n, off = H.oracle_compact(batch, kept + extra_rows)
    assert np.array_equal(cache.length.cpu().numpy(), n)
    return db, cache, (kc, vc, n, off)


def run_steps(batch, db, cache, steps, check_steps, row_role=None, oracle_ctx=None):
    """Run `steps` decode steps; compare the outputs of `check_steps` with the oracle.
    oracle_ctx(b, t) -> (k_ctx, v_ctx) bits for request b before step t."""
    B, Hq, d = batch.batch, batch.num_q_heads, batch.head_dim
    max_ctx = int(cache.row_cap_host.max())
    out = torch.empty((B, Hq, d), dtype=torch.float32, device="cuda")
    qs = bf16_to_device(batch.dec_q[:steps])
    ks = bf16_to_device(batch.dec_k[:steps])
    vs = bf16_to_device(batch.dec_v[:steps])
    errs = []
    for t in range(steps):
        st = cache.decode(qs[t], ks[t], vs[t], out, db.status, max_ctx, row_role=row_role)
        assert st == sonic.OK, sonic.status_string(st)
        if t in check_steps:
            torch.cuda.synchronize()
            assert db.read_status() == 0, sonic.status_string(db.read_status())
            got = out.cpu().numpy()
            for b in range(B):
                kc, vc = oracle_ctx(b, t)
                want = OD.decode_step(batch.dec_q[t, b], kc, vc, batch.dec_k[t, b], batch.dec_v[t, b])
                errs.append(np.abs(got[b] - want))
                H.assert_close(got[b], want, f"{batch.name} step {t} request {b}")
    torch.cuda.synchronize()
    return np.concatenate([e.ravel() for e in errs]) if errs else np.zeros(0)


def compact_ctx_fn(batch, ref):
    kc, vc, n, off = ref

    def ctx(b, t):
        base, ln = int(off[b]), int(n[b])
        k = np.concatenate([kc[base:base + ln], batch.dec_k[:t, b]])
        v = np.concatenate([vc[base:base + ln], batch.dec_v[:t, b]])
        return k, v
    return ctx


@pytest.mark.parametrize("Hq,Hkv,d", [(4, 2, 64), (32, 8, 128), (28, 4, 128), (8, 8, 128), (8, 1, 64)])
def test_decode_random_layouts(Hq, Hkv, d):
    H.need_gpu()
    rng = np.random.default_rng(200 + Hq + Hkv + d)
    lays = [W.random_layout(rng, max_h=4, max_b=400, max_k=150, max_s=300, max_c=200) for _ in range(5)]
    lays.append(W.RequestLayout(0, [], [], 1))     # a context of one row
    steps = 6
    batch = W.make_batch("rand", lays, Hq, Hkv, d, seed=int(rng.integers(1 << 30)), decode_steps=steps)
    db, cache, ref = compacted(batch, steps)
    run_steps(batch, db, cache, steps, set(range(steps)), oracle_ctx=compact_ctx_fn(batch, ref))
    # lengths advanced on the device and appended rows are in the cache, bit for bit
    kc, vc, n, off = ref
    assert np.array_equal(cache.length.cpu().numpy(), n + steps)
    k = bf16_to_host(cache.k)
    for b in range(batch.batch):
        base = int(off[b]) + int(n[b])
        assert np.array_equal(k[base:base + steps], batch.dec_k[:steps, b])


def test_masked_full_cache_decode_equals_compact():
    """Full-cache mode (history rows masked by role) against the oracle's masked decode."""
    H.need_gpu()
    rng = np.random.default_rng(77)
    lays = [W.random_layout(rng, max_h=4, max_b=300, max_k=100, max_s=200, max_c=100) for _ in range(4)]
    steps = 4
    batch = W.make_batch("full", lays, 32, 8, 128, seed=77, decode_steps=steps)
    db = H.device_batch(batch)
    # the full cache is the uncompacted augmented K/V, with room for the steps
    lens = np.array([l.length for l in lays], np.int64)
    cache = db.alloc_cache(lens + steps)
    kf = bf16_to_host(cache.k)
    vf = bf16_to_host(cache.v)
    roles = np.full(int((lens + steps).sum()), sonic.ROLE_CURRENT, np.uint8)
    for b in range(batch.batch):
        s, e = int(batch.cu_seqlens[b]), int(batch.cu_seqlens[b + 1])
        o = int(cache.row_off_host[b])
        kf[o:o + e - s] = batch.k[s:e]
        vf[o:o + e - s] = batch.v[s:e]
        roles[o:o + e - s] = batch.role[s:e]
    cache.k.copy_(bf16_to_device(kf))
    cache.v.copy_(bf16_to_device(vf))
    cache.length.copy_(torch.from_numpy(lens.astype(np.int32)))
    row_role = torch.from_numpy(roles).cuda()

    def ctx_masked(b, t):
        raise AssertionError("unused")

    B, Hq, d = batch.batch, batch.num_q_heads, batch.head_dim
    out = torch.empty((B, Hq, d), dtype=torch.float32, device="cuda")
    max_ctx = int(cache.row_cap_host.max())
    for t in range(steps):
        st = cache.decode(bf16_to_device(batch.dec_q[t]), bf16_to_device(batch.dec_k[t]),
                          bf16_to_device(batch.dec_v[t]), out, db.status, max_ctx, row_role=row_role)
        assert st == sonic.OK
        torch.cuda.synchronize()
        assert db.read_status() == 0
        got = out.cpu().numpy()
        for b in range(B):
            s, e = int(batch.cu_seqlens[b]), int(batch.cu_seqlens[b + 1])
            kfull = np.concatenate([batch.k[s:e], batch.dec_k[:t, b]])
            vfull = np.concatenate([batch.v[s:e], batch.dec_v[:t, b]])
            rfull = np.concatenate([batch.role[s:e], np.full(t, sonic.ROLE_CURRENT, np.uint8)])
            want = OD.masked_decode_step(batch.dec_q[t, b], kfull, vfull, rfull, batch.dec_k[t, b],
                                         batch.dec_v[t, b])
            H.assert_close(got[b], want, f"masked full decode step {t} request {b}")


@pytest.mark.parametrize("idx,check", [(1, None), (2, (0, 1, 100, 255)), (3, (0, 255)), (4, (0, 511)),
                                       (5, (0, 1, 1023))])
def test_decode_workloads(idx, check):
    H.need_gpu()
    batch = W.workload(idx)
    steps = batch.decode_steps
    check = set(range(steps)) if check is None else set(check)
    H.note(f"decode workload {idx}: B={batch.batch} steps={steps}")
    db, cache, ref = compacted(batch, steps)
    errs = run_steps(batch, db, cache, steps, check, oracle_ctx=compact_ctx_fn(batch, ref))
    H.note(f"  workload {idx} decode overall: max_abs={errs.max():.3e} mean_abs={errs.mean():.3e}")
    kc, vc, n, off = ref
    assert np.array_equal(cache.length.cpu().numpy(), n + steps)


def test_decode_capacity_overflow():
    """A request whose append would overflow is left unchanged; the others proceed."""
    H.need_gpu()
    lays = [W.RequestLayout(4, [10], [3], 2), W.RequestLayout(2, [5], [1], 1)]
    batch = W.make_batch("cap", lays, 4, 2, 64, seed=3, decode_steps=3)
    db, cache, ref = compacted(batch, np.array([1, 3]))
    kc, vc, n, off = ref
    out = torch.full((2, 4, 64), 5.0, dtype=torch.float32, device="cuda")
    max_ctx = int(cache.row_cap_host.max())
    q, kn, vn = (bf16_to_device(x) for x in (batch.dec_q, batch.dec_k, batch.dec_v))
    assert cache.decode(q[0], kn[0], vn[0], out, db.status, max_ctx) == sonic.OK
    torch.cuda.synchronize()
    assert db.read_status() == 0
    assert np.array_equal(cache.length.cpu().numpy(), n + 1)
    out.fill_(5.0)
    assert cache.decode(q[1], kn[1], vn[1], out, db.status, max_ctx) == sonic.OK   # request 0 is full now
    torch.cuda.synchronize()
    assert db.read_status() == sonic.ERR_CAPACITY
    assert np.array_equal(cache.length.cpu().numpy(), n + np.array([1, 2]))
    got = out.cpu().numpy()
    assert np.all(got[0] == 5.0)
    o, ln = int(off[1]), int(n[1])
    want = OD.decode_step(batch.dec_q[1, 1], np.concatenate([kc[o:o + ln], batch.dec_k[:1, 1]]),
                          np.concatenate([vc[o:o + ln], batch.dec_v[:1, 1]]), batch.dec_k[1, 1], batch.dec_v[1, 1])
    H.assert_close(got[1], want, "request 1 after request 0 overflowed")


def test_decode_honours_pending_layout_error():
    """A layout error left by an earlier call stops decode (no append, no output, no length change);
    a pending capacity error does not (capacity is per request); afterwards decode still matches the
    oracle, so the split counters were left consistent."""
    H.need_gpu()
    # long enough contexts for several splits per (request, kv-head) pair
    lays = [W.RequestLayout(700, [30], [12], 9), W.RequestLayout(650, [20], [4], 3)]
    steps = 2
    batch = W.make_batch("pending", lays, 8, 2, 128, seed=4, decode_steps=steps)
    db, cache, ref = compacted(batch, steps)
    kc, vc, n, off = ref
    max_ctx = int(cache.row_cap_host.max())
    out = torch.full((2, 8, 128), 5.0, dtype=torch.float32, device="cuda")
    q, kn, vn = (bf16_to_device(x) for x in (batch.dec_q, batch.dec_k, batch.dec_v))
    k_before, v_before = bf16_to_host(cache.k).copy(), bf16_to_host(cache.v).copy()
    db.status.fill_(sonic.ERR_BAD_LAYOUT)
    assert cache.decode(q[0], kn[0], vn[0], out, db.status, max_ctx) == sonic.OK
    torch.cuda.synchronize()
    assert db.read_status() == sonic.ERR_BAD_LAYOUT
    assert np.array_equal(cache.length.cpu().numpy(), n)
    assert torch.all(out == 5.0)
    assert np.array_equal(bf16_to_host(cache.k), k_before) and np.array_equal(bf16_to_host(cache.v), v_before)
    ctx = compact_ctx_fn(batch, ref)
    db.status.fill_(sonic.ERR_CAPACITY)
    for t in range(steps):
        assert cache.decode(q[t], kn[t], vn[t], out, db.status, max_ctx) == sonic.OK
        torch.cuda.synchronize()
        assert db.read_status() == (sonic.ERR_CAPACITY if t == 0 else 0)
        got = out.cpu().numpy()
        for b in range(2):
            kk, vv = ctx(b, t)
            want = OD.decode_step(batch.dec_q[t, b], kk, vv, batch.dec_k[t, b], batch.dec_v[t, b])
            H.assert_close(got[b], want, f"step {t} request {b} after a pending status")
        db.clear_status()
    assert np.array_equal(cache.length.cpu().numpy(), n + steps)


def test_decode_default_scale_is_one_over_sqrt_d():
    """softmax_scale = 0 (the binding's default) gives bit for bit the output of an explicit 1/sqrt(d)."""
    H.need_gpu()
    lays = [W.RequestLayout(40, [30], [12], 9), W.RequestLayout(3, [20], [4], 3)]
    batch = W.make_batch("scale", lays, 8, 2, 64, seed=5, decode_steps=1)
    outs = []
    for scale in (None, 1.0 / np.sqrt(64.0)):
        db, cache, ref = compacted(batch, 1)
        out = torch.empty((2, 8, 64), dtype=torch.float32, device="cuda")
        st = sonic.compressed_decode(cache.k, cache.v, cache.row_off, cache.row_cap, cache.length,
                                     bf16_to_device(batch.dec_q[0]), bf16_to_device(batch.dec_k[0]),
                                     bf16_to_device(batch.dec_v[0]), out,
                                     torch.zeros(sonic.decode_workspace_bytes(2, 8, 64, 64), dtype=torch.uint8,
                                                 device="cuda"), db.status, 64, softmax_scale=scale)
        assert st == sonic.OK
        torch.cuda.synchronize()
        outs.append(out.cpu().numpy())
    assert np.array_equal(outs[0], outs[1])


def plain_caches(rng, lens, room, Hkv, d):
    """Caches of the given lengths with `room` rows to spare: (cache, k bits, v bits)."""
    from paper_2601_21927_amd.runner import CompactCache
    cap = np.asarray(lens, np.int64) + room
    off = np.concatenate([[0], np.cumsum(cap)[:-1]])
    cache = CompactCache(int(cap.sum()), Hkv, d, off, cap, "cuda")
    k, v = (W.f32_to_bf16_bits(rng.standard_normal((int(cap.sum()), Hkv, d)).astype(np.float32)) for _ in range(2))
    cache.k.copy_(bf16_to_device(k))
    cache.v.copy_(bf16_to_device(v))
    cache.length.copy_(torch.from_numpy(np.asarray(lens, np.int32)))
    return cache, k, v


@pytest.mark.parametrize("B,Hq,Hkv,d,lens,max_ctx", [
    (64, 16, 4, 128, (0, 1, 15, 16, 255, 256, 257, 700), 2048),     # shared evenly, 64 requests
    (37, 56, 7, 64, (3, 300, 511, 512, 513), 4096),                  # ... odd counts, eight heads a group
    (32, 8, 8, 128, (2500, 40), 2600),                               # ... a request of many splits, one head a group
    (64, 28, 4, 128, (5, 60, 200), 256),                             # a split per pair, four waves
    (12, 8, 8, 128, (100, 700), 1024),                               # fewer workgroups than CUs: eight waves
    (8, 32, 8, 128, (900, 37), 1000),                                # four splits, four waves
    (65, 16, 4, 64, (90, 300), 2048)])                               # more requests than a wave has lanes
def test_decode_work_split(B, Hq, Hkv, d, lens, max_ctx):
    """Every way a call is cut into workgroups, over uneven lengths with a request at its
    capacity among them: outputs, appended rows, lengths, two calls in a row."""
    H.need_gpu()
    rng = np.random.default_rng(B + Hq + d)
    lens = np.array([lens[b % len(lens)] for b in range(B)], np.int64)
    cache, k, v = plain_caches(rng, lens, 2, Hkv, d)
    full = B // 2                                  # this request has no room left
    cache.row_cap[full] = int(lens[full])
    off = cache.row_off_host
    status = torch.zeros(1, dtype=torch.int32, device="cuda")
    out = torch.full((B, Hq, d), 7.0, dtype=torch.float32, device="cuda")
    for t in range(2):
        q, kn, vn = (W.f32_to_bf16_bits(rng.standard_normal((B, h, d)).astype(np.float32)) for h in (Hq, Hkv, Hkv))
        assert cache.decode(bf16_to_device(q), bf16_to_device(kn), bf16_to_device(vn), out, status, max_ctx) == sonic.OK
        torch.cuda.synchronize()
        assert int(status.item()) == sonic.ERR_CAPACITY
        got, gk, gv = out.cpu().numpy(), bf16_to_host(cache.k), bf16_to_host(cache.v)
        for b in range(B):
            o, n = int(off[b]), int(lens[b])
            if b == full:
                assert (got[b] == 7.0).all() and np.array_equal(gk[o:o + n + 2], k[o:o + n + 2])
                continue
            if b < 8 or b % 7 == 0 or b == B - 1:
                want = OD.decode_step(q[b], k[o:o + n], v[o:o + n], kn[b], vn[b])
                err = np.abs(got[b] - want).max()
                # probabilities carry 16 bits: 2^-16 of the largest value, and the fp32 sums
                assert err <= 1e-4, f"request {b} step {t}: {err:.2e}"
            k[o + n], v[o + n] = kn[b], vn[b]
            assert np.array_equal(gk[o:o + n + 1], k[o:o + n + 1]) and np.array_equal(gv[o:o + n + 1], v[o:o + n + 1])
            lens[b] += 1
        assert np.array_equal(cache.length.cpu().numpy(), lens)


@pytest.mark.parametrize("B,Hq,Hkv,d,lens,max_ctx", [
    (64, 16, 4, 128, (5, 300, 700), 2048),       # rows shared over the batch
    (8, 32, 8, 128, (900, 37), 1000),            # four splits per pair
    (64, 28, 4, 128, (5, 60, 200), 256)])        # one split per pair
def test_decode_status_changes_while_it_runs(B, Hq, Hkv, d, lens, max_ctx):
    """Another stream raises and clears a layout error while calls run: a pair's output is
    untouched or the one of a call left alone, a length is advanced or not, and the counters
    in the workspace are at zero again, so that the next call is right."""
    H.need_gpu()
    rng = np.random.default_rng(B + Hq)
    lens = np.array([lens[b % len(lens)] for b in range(B)], np.int64)
    cache, _, _ = plain_caches(rng, lens, 2, Hkv, d)
    q, kn, vn = (bf16_to_device(W.f32_to_bf16_bits(rng.standard_normal((B, h, d)).astype(np.float32)))
                 for h in (Hq, Hkv, Hkv))
    len0 = torch.from_numpy(lens.astype(np.int32)).cuda()
    status = torch.zeros(1, dtype=torch.int32, device="cuda")
    ws = torch.zeros(sonic.decode_workspace_bytes(B, Hq, d, max_ctx), dtype=torch.uint8, device="cuda")
    counters = ws[:(4 * B + 255) // 256 * 256 + 4 * B * Hkv]

    def call(out):
        cache.length.copy_(len0)
        assert sonic.compressed_decode(cache.k, cache.v, cache.row_off, cache.row_cap, cache.length, q, kn, vn, out,
                                       ws, status, max_ctx) == sonic.OK
    want = torch.empty((B, Hq, d), dtype=torch.float32, device="cuda")
    call(want)
    outs = torch.full((32, B, Hq, d), float("nan"), dtype=torch.float32, device="cuda")
    got_len = torch.empty((32, B), dtype=torch.int32, device="cuda")
    flips = H.Flips(status, sonic.ERR_BAD_LAYOUT)
    for i, (out, gl) in enumerate(zip(outs, got_len)):
        if i % 8 == 0:
            flips.start()
        call(out)
        gl.copy_(cache.length)
    torch.cuda.synchronize()
    assert not bool(counters.any())
    left = torch.isnan(outs)
    assert bool((left | (outs == want)).all())
    per_pair = left.view(32, B, Hkv, -1)
    assert bool((per_pair.all(-1) | ~per_pair.any(-1)).all())
    assert bool(((got_len == len0) | (got_len == len0 + 1)).all())
    # a request whose length was advanced has all its outputs
    assert not bool((left.view(32, B, -1).any(-1) & (got_len == len0 + 1)).any())
    H.note(f"  outputs left out: {float(left.float().mean()):.2f}")
    again = torch.full_like(want, float("nan"))
    call(again)
    torch.cuda.synchronize()
    assert torch.equal(again, want) and bool((cache.length == len0 + 1).all())


@pytest.mark.parametrize("B,Hq,Hkv,d,lens,max_ctx", [
    (64, 8, 4, 128, (3, 300, 700), 2048),     # rows shared over the batch
    (8, 32, 8, 128, (900, 37, 640), 1000),    # four splits per pair
    (64, 28, 4, 128, (5, 60, 200), 256),      # one split per pair, four waves
    (3, 8, 8, 64, (100, 33, 900), 1000)])     # several splits, eight waves
def test_decode_infinite_values(B, Hq, Hkv, d, lens, max_ctx):
    """One V row per column of d is infinite (the first row of every 16-row group among
    them, so also the one that stands in for the rows past a range's end): that column of the
    output is that infinity, every other one is what the oracle says."""
    H.need_gpu()
    rng = np.random.default_rng(B + d)
    lens = np.array([lens[b % len(lens)] for b in range(B)], np.int64)
    cache, k, v = plain_caches(rng, lens, 2, Hkv, d)
    off = cache.row_off_host
    rows = [np.unique(np.concatenate([np.arange(0, n, 16), [n // 2, n - 1]]))[:d - 8] for n in lens]
    signs = np.where(np.arange(d) % 3 == 0, 0xFF80, 0x7F80).astype(np.uint16)
    finite = v.copy()
    for b, rs in enumerate(rows):
        for j, r in enumerate(rs):
            v[off[b] + r, :, j] = signs[j]
    cache.v.copy_(bf16_to_device(v))
    status = torch.zeros(1, dtype=torch.int32, device="cuda")
    out = torch.empty((B, Hq, d), dtype=torch.float32, device="cuda")
    q, kn, vn = (W.f32_to_bf16_bits(rng.standard_normal((B, h, d)).astype(np.float32)) for h in (Hq, Hkv, Hkv))
    fin_new = vn.copy()
    vn[:, :, d - 1] = 0x7F80
    assert cache.decode(bf16_to_device(q), bf16_to_device(kn), bf16_to_device(vn), out, status, max_ctx) == sonic.OK
    torch.cuda.synchronize()
    assert int(status.item()) == 0
    got = out.cpu().numpy()
    for b in range(B):
        o, n = int(off[b]), int(lens[b])
        if b >= 6 and b != B - 1:
            continue
        want = OD.decode_step(q[b], k[o:o + n], finite[o:o + n], kn[b], fin_new[b])
        m = len(rows[b])
        inf = np.where(signs == 0x7F80, np.inf, -np.inf)
        want[:, :m] = inf[:m]
        want[:, d - 1] = np.inf
        assert np.array_equal(np.isfinite(got[b]), np.isfinite(want)), f"request {b}"
        ok = np.isfinite(want)
        assert np.array_equal(got[b][~ok], want[~ok]), f"request {b}"
        assert np.abs(got[b][ok] - want[ok]).max() <= 1e-4, f"request {b}"   # as in test_decode_work_split


@pytest.mark.parametrize("B,Hq,Hkv,d,lens,max_ctx", [
    (64, 8, 4, 64, (100, 3, 40), 8192),              # far more workgroups launched than have rows
    (16, 16, 16, 128, (2500, 40, 3000, 700), 3600),  # long cache rows: the kv-heads alternate
    (8, 64, 64, 64, (17, 1500, 300), 2048),
    (64, 32, 8, 64, (1900, 60, 500, 1300), 2048),    # more requests' remainders than workgroups to spare
    (33, 24, 8, 128, (4096, 16, 2), 4200),
    (64, 16, 16, 64, (30, 2100), 2200)])             # 1,024 pairs: three splits each
@pytest.mark.parametrize("how", ["workspace", "smallest workspace", "no workspace", "all full"])
def test_decode_shared_rows(B, Hq, Hkv, d, lens, max_ctx, how):
    """256 pairs and more: rows shared over the batch, or, in a workspace that has no room for
    that, three splits a pair; on the library's own array; and with no request that has room."""
    H.need_gpu()
    rng = np.random.default_rng(B + Hq + d)
    lens = np.array([lens[b % len(lens)] for b in range(B)], np.int64)
    cache, k, v = plain_caches(rng, lens, 2, Hkv, d)
    if how == "all full":
        cache.row_cap.copy_(cache.length)
    off = cache.row_off_host
    status = torch.zeros(1, dtype=torch.int32, device="cuda")
    counters = -(-B * 4 // 256) * 256 + -(-B * Hq * 4 // 256) * 256
    n = counters + B * Hq * 3 * (d + 2) * 4 if how == "smallest workspace" else sonic.decode_workspace_bytes(B, Hq, d, max_ctx)
    ws = torch.zeros(n, dtype=torch.uint8, device="cuda")
    out = torch.full((B, Hq, d), 7.0, dtype=torch.float32, device="cuda")
    check = sorted({0, 1, 2, 3, B - 1})
    for t in range(2):
        q, kn, vn = (W.f32_to_bf16_bits(rng.standard_normal((B, h, d)).astype(np.float32)) for h in (Hq, Hkv, Hkv))
        args = (cache.k, cache.v, cache.row_off, cache.row_cap, cache.length, bf16_to_device(q), bf16_to_device(kn),
                bf16_to_device(vn), out)
        st = (sonic.compressed_decode_noalloc(*args, status, max_ctx) if how == "no workspace" else
              sonic.compressed_decode(*args, ws, status, max_ctx))
        assert st == sonic.OK
        torch.cuda.synchronize()
        assert not bool(ws[:-(-B * 4 // 256) * 256 + 4 * B * Hkv].any())   # the counters
        if how == "all full":
            assert int(status.item()) == sonic.ERR_CAPACITY and bool((out == 7.0).all())
            assert np.array_equal(cache.length.cpu().numpy(), lens)
            continue
        assert int(status.item()) == 0
        got, gk = out.cpu().numpy(), bf16_to_host(cache.k)
        for b in range(B):
            o, ln = int(off[b]), int(lens[b])
            if b in check:
                want = OD.decode_step(q[b], k[o:o + ln], v[o:o + ln], kn[b], vn[b])
                assert np.abs(got[b] - want).max() <= 1e-4, f"request {b} step {t}"   # as in test_decode_work_split
            k[o + ln], v[o + ln] = kn[b], vn[b]
            assert np.array_equal(gk[o + ln], kn[b])
            lens[b] += 1
        assert np.array_equal(cache.length.cpu().numpy(), lens)
