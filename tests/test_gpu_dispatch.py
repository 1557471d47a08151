"""The sizes, placements and shapes where a launch rule changes from one form of a kernel to another: the forms must
agree bit for bit with each other or with the oracle on both sides of the line."""
import ctypes

import numpy as np
import pytest
import torch

import synth_inputs as S

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2507_19823_amd import binding
    assert torch.cuda.is_available(), "GPU tests need the MI355X"
    binding.lib()
    return binding


def _layer(w, k_max, cap=None, m_max=1):
    from paper_2507_19823_amd.session import LayerState
    return LayerState(w.batch, w.n_q_heads, w.n_kv_heads, cap or w.n, w.bits, w.group, k_max=k_max, m_max=m_max)


@pytest.mark.parametrize("k", [1, 63, 64, 65, 257, 1000])
def test_value_rows_are_the_same_wherever_they_live(B, k):
    """hca_gather_values stages the same rows with all of the store in host memory (one small persistent grid), all of it
    in HBM (one sweep), and shared between the two (both kinds of workgroups, or one where the HBM slice is short)."""
    w = S.Workload("gather", 81, 2, 8, 2, 1200, 4, 32, k)
    d = S.make_layer(w)
    st = _layer(w, k)
    st.quantize(d["keys"].cuda())
    st.n = [1200, min(1200, k + 3)]                       # the second row selects nearly everything it has
    q, values = d["q"].cuda(), d["values"]
    st.score_topk(q, k)
    side = torch.cuda.Stream()
    out = []
    for n_host in (1200, 0, 600, 1150, 1):                # 1150: the HBM slice is short, 1: nearly nothing on the host
        vh = values[:, :, :n_host].contiguous().pin_memory() if n_host else None
        vd = values[:, :, n_host:].contiguous().cuda() if n_host < 1200 else None
        for gather in (side, None):                       # a stream of its own: through the gather; else read where they live
            st.y.fill_(-1.0)
            st.acc.zero_()
            torch.cuda.synchronize()
            st.attend(q, vh, n_host, vd, gather_stream=gather)
            torch.cuda.synchronize()
            out.append((n_host, gather is None, st.y.clone(), st.acc.clone()))
    assert torch.isfinite(out[0][2]).all() and (out[0][3] > 0).any()
    for n_host, direct, y, acc in out[1:]:
        assert torch.equal(y, out[0][2]) and torch.equal(acc, out[0][3]), f"n_host_rows = {n_host}, direct {direct}"


@pytest.mark.parametrize("batch,n_host,k,wgs", [(4, 0, 300, 19), (8, 0, 500, 8), (16, 0, 1100, 18), (4, 600, 300, 7), (4, 600, 64, 2),
                                                (1, 600, 400, 8)])
def test_gather_stamps_time_the_launch_that_runs(B, batch, n_host, k, wgs):
    """A timed step gathers with the workgroups of an untimed one - per row: 16 or 64 rows each where the store is in HBM, host
    and HBM kinds where it is shared and the launch is large, else the host kind alone -, and their stamps say so: one start per
    workgroup up to 1024, no end before its start."""
    n, hkv = 1200, 8
    w = S.Workload("stamps", 83, batch, 32, hkv, n, 4, 32, k)
    d = S.make_layer(w)
    st = _layer(w, k, cap=n + 4)
    st.quantize(d["keys"].cuda())
    q, values = d["q"].cuda(), d["values"]
    vh = values[:, :, :n_host].contiguous().pin_memory() if n_host else None
    vd = torch.zeros(batch, hkv, n + 4 - n_host, 128, dtype=torch.float16, device="cuda")
    vd[:, :, :n - n_host] = values[:, :, n_host:].cuda()
    keep = [torch.zeros(batch, hkv, 1, 128, dtype=torch.float16, device="cuda"), torch.zeros(1, 1, 1024, 2, dtype=torch.int64, device="cuda")]

    def buf(*shape, dtype=torch.uint8):
        keep.append(torch.zeros(shape, dtype=dtype, device="cuda"))
        return keep[-1].data_ptr()
    p = B.hca_pipeline_desc()
    cur = torch.cuda.current_stream().cuda_stream
    p.stream_scan = p.stream_topk = p.stream_gather = p.stream_attend = cur
    p.n_sel, p.n_pipe = 3, 4
    for i in range(3):
        p.sel[i] = buf(batch, hkv, n + 4, dtype=torch.float32)
    wsb = B.hca_workspace_bytes(st.shape, k, 1)
    for i in range(4):
        p.idx[i], p.count[i] = buf(batch, hkv, k, dtype=torch.int32), buf(batch, hkv, dtype=torch.int32)
        p.ws_attend[i] = buf(wsb)
    p.ws_topk = buf(wsb)
    pairs = B.hca_scan_stamp_pairs(st.shape, n + 4)
    p.scan_stamps, p.scan_stamp_pairs = buf(1, 1, pairs, 2, dtype=torch.int64), pairs
    p.gather_stamps = keep[1].data_ptr()
    ly = (B.hca_layer * 1)()
    ly[0].kcache, ly[0].acc, ly[0].pos = st.kcache.data_ptr(), st.acc.data_ptr(), st.pos.data_ptr()
    ly[0].k_new, ly[0].q, ly[0].y = keep[0].data_ptr(), q.data_ptr(), st.y.data_ptr()
    ly[0].v_host, ly[0].v_hbm = vh.data_ptr() if n_host else None, vd.data_ptr()
    nres = (ctypes.c_int64 * batch)(*[n] * batch)
    pl = B.hca_pipeline_create(st.shape, 1, p, 1)
    B.hca_pipeline_step(pl, ly, nres, n, k, n_host, n_host, vd.shape[2], st.sm_scale, timing_slot=0)
    torch.cuda.synchronize()
    B.hca_pipeline_destroy(pl)
    stamps = keep[1].cpu().numpy()[0, 0]
    used = min(1024, wgs * batch * hkv)
    assert (stamps[:used, 0] > 0).all() and (stamps[used:] == 0).all()
    assert (stamps[:used, 1] >= stamps[:used, 0]).all()
    assert torch.isfinite(st.y).all()


def _one_stream_attend(B, n, k):
    """A call of hca_sparse_attend on one stream, 8 KV heads, every value in host memory; stream -> None."""
    w = S.Workload("hostvals", 82, 1, 32, 8, n, 4, 32, k)
    d = S.make_layer(w)
    st = _layer(w, k)
    st.quantize(d["keys"].cuda())
    q, values = d["q"].cuda(), d["values"].contiguous().pin_memory()
    st.score_topk(q, k)
    torch.cuda.synchronize()
    return lambda stream=None: B.hca_sparse_attend(st.shape, st.kcache, q, st.idx, st.count, k, st.pos, values, n, n, None, 0,
                                                   st.sm_scale, st.y, None, st.ws, stream=stream, gather_stream=stream)


def test_host_values_on_one_stream_leave_the_others_their_memory(B):
    """2048 x 8 values from host memory on one stream, a scan of 8 x 512 Ki keys on another: a read per thread across the host
    link would double the scan's time.  Allowed: 1.4 times the scan alone."""
    attend = _one_stream_attend(B, 4096, 2048)
    n = 524288
    shape = B.make_shape(1, 32, 8, n)
    kc = torch.zeros(B.hca_kcache_bytes(shape), dtype=torch.uint8, device="cuda")
    q = torch.randn(1, 32, 128, device="cuda").half()
    sel = torch.zeros(1, 8, n, device="cuda")
    ws = torch.empty(B.hca_workspace_bytes(shape, 64, 1), dtype=torch.uint8, device="cuda")
    side, took = torch.cuda.Stream(), []
    for beside in (0, 1, 0, 1, 0, 1):
        torch.cuda.synchronize()
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        torch.cuda._sleep(3000000)
        side.wait_stream(torch.cuda.current_stream())
        a.record()
        for _ in range(12):
            B.hca_score_qkeys(shape, kc, q, [n], sel, None, ws)
        b.record()
        for _ in range(16 * beside):
            attend(side)
        torch.cuda.synchronize()
        took.append((beside, a.elapsed_time(b) * 1000 / 12))
    alone, both = (min(t for x, t in took if x == y) for y in (0, 1))
    assert both < 1.4 * alone, f"{alone:.0f} us alone, {both:.0f} us beside the attends"


def test_a_shaped_gather_is_used(B):
    """hca_tune("gather_wgs") reaches one-stream attends of few host values too: one workgroup per row is slower."""
    attend = _one_stream_attend(B, 4096, 512)
    try:
        own = _passes_us(attend)
        B.hca_tune("gather_wgs", 1)
        one = _passes_us(attend)
    finally:
        B.hca_tune("gather_wgs", 0)
    assert one > 1.2 * own, f"{own:.1f} us, {one:.1f} us with one workgroup"


@pytest.mark.parametrize("bits,gs", [(4, 32), (2, 64)])
@pytest.mark.parametrize("G,n_sel", [(4, 256), (4, 1), (2, 129), (1, 255)])
@pytest.mark.parametrize("use_lse", [False, True])
def test_rows_of_one_chunk_need_no_merge(B, bits, gs, G, n_sel, use_lse):
    """k <= 256: the only chunk of a row writes y and the accumulated scores itself; the same selection with a larger k goes
    through the chunk partials and the merge.  A row with nothing selected gives zeros both ways."""
    w = S.Workload("one", 84, 3, 2 * G, 2, 700, bits, gs, n_sel)
    d = S.make_layer(w)
    st = _layer(w, 600)
    st.quantize(d["keys"].cuda())
    st.n = [700, max(1, n_sel // 2), 0]
    q, vd = d["q"].cuda(), d["values"].cuda()
    st.score(q)
    st.topk(n_sel)
    small = st.idx.reshape(6, n_sel).clone()
    count = st.count.clone()
    wide = torch.zeros(6, 600, dtype=torch.int32, device="cuda")
    wide[:, :n_sel] = small
    lse = torch.randn(3, 2 * G, device="cuda") + 30 if use_lse else None
    out = []
    for idx, k in ((small, n_sel), (wide, 600)):
        st.y.fill_(-1.0)
        st.acc.zero_()
        B.hca_gather_values(st.shape, idx, count, k, st.pos, None, 0, 0, vd, 700, st.ws)
        if use_lse:
            B.hca_attend_gathered_global(st.shape, st.kcache, q, idx, count, k, st.sm_scale, lse, st.y, st.acc, st.ws)
        else:
            B.hca_attend_gathered(st.shape, st.kcache, q, idx, count, k, st.sm_scale, st.y, st.acc, st.ws)
        torch.cuda.synchronize()
        out.append((st.y.clone(), st.acc.clone()))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
    assert (out[0][0][2] == 0).all() and (out[0][0][0] != 0).any()


def _order_key(x):
    u = x.view(np.uint32).copy()
    u[(u << np.uint32(1)) == 0] = 0
    return np.where(u >> np.uint32(31), ~u, u | np.uint32(0x80000000)).astype(np.uint32)


def _scores(kind, n, rng):
    x = rng.standard_normal(n).astype(np.float32)
    if kind == "outlier":                                   # one value far above: nearly all others share a bin
        x[n // 2] = 1e30
    elif kind == "ties":                                    # a few values, thousands of slots each
        x = rng.integers(-2, 3, n).astype(np.float32)
    elif kind == "close":                                   # distinct keys that differ in their last bits, both signs of zero
        x = (np.float32(7) + rng.integers(0, 4096, n).astype(np.float32) * np.float32(4.7683716e-07)).astype(np.float32)
        x[:: 97] = 0.0
        x[1:: 97] = -0.0
    elif kind == "masked":                                  # infinities and the type's lowest value among the scores
        x[rng.random(n) < 0.4] = np.finfo(np.float32).min
        x[rng.random(n) < 0.4] = -np.inf
        x[rng.random(n) < 0.01] = np.inf
    elif kind == "nan":                                     # NaNs order by their bits, like every other value
        x[rng.random(n) < 0.02] = np.nan
        x[rng.random(n) < 0.02] = -np.nan
    elif kind == "tiny":
        x = (x * np.float32(1e-42)).astype(np.float32)
    elif kind == "equal":
        x[:] = -3.5
    elif kind == "wide":                                    # max - min overflows
        x = (np.clip(x, -2.8, 2.8) * np.float32(1.2e38)).astype(np.float32)
    return x


@pytest.mark.parametrize("kind", ["normal", "outlier", "ties", "close", "masked", "nan", "tiny", "equal", "wide"])
@pytest.mark.parametrize("n", [1, 63, 65, 1024, 4096, 4097, 8193, 16384, 16385, 32767, 32769, 40960, 40961])
def test_topk_at_the_edges_of_the_one_launch_form(B, kind, n):
    """hca_topk with the row in one workgroup's registers (up to 40 Ki slots, five sizes of it) and over the chip."""
    rng = np.random.default_rng(n + len(kind))
    lens = [n, max(1, n - 31), 0]
    cap = n + 3
    sel = np.full((3, cap), 9e9, np.float32)                # past the row's end: larger than anything in it
    for b in range(3):
        sel[b, :lens[b]] = _scores(kind, lens[b], rng) if lens[b] else 0
    shape = B.make_shape(3, 1, 1, cap)
    dsel = torch.from_numpy(sel).cuda()
    for k in sorted({1, min(n, 5), max(1, n // 3), n}):
        ws = torch.empty(B.hca_workspace_bytes(shape, k, 1), dtype=torch.uint8, device="cuda")
        idx = torch.full((3, k), -7, dtype=torch.int32, device="cuda")
        count = torch.full((3,), -7, dtype=torch.int32, device="cuda")
        B.hca_topk(shape, dsel, lens, k, idx, count, ws)
        torch.cuda.synchronize()
        got, c = idx.cpu().numpy(), count.cpu().numpy()
        for b in range(3):
            want = min(k, lens[b])
            assert c[b] == want
            key = _order_key(sel[b, :lens[b]]).astype(np.int64)
            ref = np.sort(np.argsort(-key, kind="stable")[:want])
            assert np.array_equal(got[b, :want], ref), f"row {b}, k {k}"
            assert np.all(got[b, want:] == -7)


@pytest.mark.parametrize("kind", ["normal", "ramp", "ties", "steps", "seen", "missed", "lower", "nan", "nans", "seen nans", "masked"])
@pytest.mark.parametrize("n", [8191, 8192, 12288, 12289, 16384, 16385, 30011, 40960])
def test_topk_of_a_row_sifted_by_samples(B, kind, n):
    """Few of a row in one workgroup's registers: the list above the samples' bound, and rows whose samples mislead."""
    rng = np.random.default_rng(n + 7 * len(kind))
    t = np.arange(1024, dtype=np.int64)
    sampled = (t * n >> 10) + (((t * 40503 & 0xffff) * (n >> 10)) >> 16)
    x = rng.standard_normal(n).astype(np.float32)
    if kind == "ramp":
        x.sort()
    elif kind == "ties":                                    # more equal values than are ranked against each other
        x = np.round(x * 2) / 2
    elif kind == "seen":                                    # the sampled places hold the largest values: a list too short
        x[sampled] += 20
    elif kind == "missed":                                  # and the smallest: one too long, or with all its values in the top bin
        x[sampled] -= 20
    elif kind == "steps":                                   # ties whose bins hold as many as are ranked, and more
        x = np.round(x * 24) / 24
    elif kind == "lower":                                   # lists up to their room and past it
        x[sampled] -= 0.25 + 0.1 * rng.random()
    elif kind == "nan":
        x[n - 5] = np.nan
    elif kind in ("nans", "seen nans"):                     # of both signs, with all keys: the largest and the smallest
        if kind != "nans":
            x[sampled] += 20
        other = np.setdiff1d(np.arange(n), sampled)
        at = rng.choice(other, min(3000, n // 3), replace=False)
        x.view(np.uint32)[at] = rng.integers(0x7f800001, 0x80000000, at.size) | np.where(np.arange(at.size) % 9 == 0, 0, 1 << 31)
    elif kind == "masked":
        x[rng.random(n) < 0.5] = -np.inf
        x[rng.random(n) < 0.001] = np.inf
    shape = B.make_shape(1, 1, 1, n)
    dsel = torch.from_numpy(x).cuda()
    ref = np.argsort(-_order_key(x).astype(np.int64), kind="stable")
    for k in (1, 64, 777, 2048, 3000):
        ws = torch.empty(B.hca_workspace_bytes(shape, k, 1), dtype=torch.uint8, device="cuda")
        idx = torch.full((1, k), -7, dtype=torch.int32, device="cuda")
        count = torch.full((1,), -7, dtype=torch.int32, device="cuda")
        B.hca_topk(shape, dsel, [n], k, idx, count, ws)
        torch.cuda.synchronize()
        assert count.item() == k
        assert np.array_equal(idx.cpu().numpy()[0], np.sort(ref[:k])), f"k {k}"


def _sampled_slots(n, m=8192):
    """The slots whose scores topk_sample_rank looks at."""
    i = np.arange(min(n, m), dtype=np.uint64)
    low = np.uint64(0xffffffff)
    h = (i * np.uint64(0x9E3779B1)) & low
    h = ((h ^ h >> np.uint64(15)) * np.uint64(0x85EBCA77)) & low
    h = ((h ^ h >> np.uint64(13)) * np.uint64(0xC2B2AE3D)) & low
    h ^= h >> np.uint64(16)
    return (i if n <= m else (i * np.uint64(n) + (h * np.uint64(n) >> np.uint64(32))) // np.uint64(m)).astype(np.int64)


def _misread(n, rng):
    """Scores whose sampled slots hold all the large ones."""
    x = -np.abs(rng.standard_normal(n)).astype(np.float32)
    x[_sampled_slots(n)] *= -1
    return x


@pytest.mark.parametrize("kind", ["normal", "outlier", "ties", "close", "masked", "nan", "equal", "wide", "few", "misread",
                                  "lowest nan"])
@pytest.mark.parametrize("n", [40961, 65536, 300001])
def test_topk_of_long_rows_by_a_sampled_key(B, kind, n):
    """hca_topk over the chip: lists above the sampled key, equal slots taken in slot order where the lists fall short
    (few: more equal slots than others), a row its samples misrepresent, and a key that is all zeros; short rows beside."""
    rng = np.random.default_rng(n + len(kind))
    lens = [n, n - 4099, 5000, 1, 0]
    cap = n + 3
    sel = np.full((5, cap), 9e9, np.float32)                # past the row's end: larger than anything in it
    for b in range(5):
        if kind == "few":
            x = np.where(rng.random(lens[b]) < 0.99, np.finfo(np.float32).min, rng.standard_normal(lens[b]))
        elif kind == "misread":
            x = _misread(lens[b], rng)
        elif kind == "lowest nan":
            x = rng.standard_normal(lens[b]).astype(np.float32)
            x.view(np.uint32)[::3] = 0xffffffff
        else:
            x = _scores(kind, lens[b], rng) if lens[b] else 0
        sel[b, :lens[b]] = x
        if kind == "lowest nan" and lens[b]:
            sel[b, :lens[b]].view(np.uint32)[::3] = 0xffffffff        # (the bits, whatever a conversion did to them)
    shape = B.make_shape(5, 1, 1, cap)
    dsel = torch.from_numpy(sel).cuda()
    for k in (1, 5, 700, 3300, 8000):
        ws = torch.empty(B.hca_workspace_bytes(shape, k, 1), dtype=torch.uint8, device="cuda")
        idx = torch.full((5, k), -7, dtype=torch.int32, device="cuda")
        count = torch.full((5,), -7, dtype=torch.int32, device="cuda")
        for again in range(2):                              # the second time on the workspace as the first left it
            B.hca_topk(shape, dsel, lens, k, idx, count, ws)
        torch.cuda.synchronize()
        got, c = idx.cpu().numpy(), count.cpu().numpy()
        for b in range(5):
            want = min(k, lens[b])
            assert c[b] == want
            key = _order_key(sel[b, :lens[b]]).astype(np.int64)
            ref = np.sort(np.argsort(-key, kind="stable")[:want])
            assert np.array_equal(got[b, :want], ref), f"row {b}, k {k}"
            assert np.all(got[b, want:] == -7)


@pytest.mark.parametrize("kind", ["normal", "outlier", "ties", "close", "masked", "nan", "tiny", "equal", "wide", "few",
                                  "lowest nan"])
@pytest.mark.parametrize("n,k", [(40961, 14400), (90000, 20000), (300001, 15000)])
def test_topk_of_long_rows_beyond_the_sampled_key(B, kind, n, k):
    """hca_topk in its histogram form: a k whose lists the sampled form could not hold in registers; short rows beside."""
    rng = np.random.default_rng(n + len(kind))
    lens = [n, n - 4099, 16000, 1, 0]
    sel = np.full((5, n + 3), 9e9, np.float32)              # past the row's end: larger than anything in it
    for b in range(5):
        if kind == "few":
            x = np.where(rng.random(lens[b]) < 0.99, np.finfo(np.float32).min, rng.standard_normal(lens[b]))
        else:
            x = _scores(kind, lens[b], rng) if lens[b] else 0
        sel[b, :lens[b]] = x
        if kind == "lowest nan" and lens[b]:
            sel[b, :lens[b]].view(np.uint32)[::3] = 0xffffffff
    shape = B.make_shape(5, 1, 1, n + 3)
    dsel = torch.from_numpy(sel).cuda()
    ws = torch.empty(B.hca_workspace_bytes(shape, k, 1), dtype=torch.uint8, device="cuda")
    idx = torch.full((5, k), -7, dtype=torch.int32, device="cuda")
    count = torch.full((5,), -7, dtype=torch.int32, device="cuda")
    for again in range(2):                                  # the second time on the workspace as the first left it
        B.hca_topk(shape, dsel, lens, k, idx, count, ws)
    torch.cuda.synchronize()
    got, c = idx.cpu().numpy(), count.cpu().numpy()
    for b in range(5):
        want = min(k, lens[b])
        assert c[b] == want
        key = _order_key(sel[b, :lens[b]]).astype(np.int64)
        ref = np.sort(np.argsort(-key, kind="stable")[:want])
        assert np.array_equal(got[b, :want], ref), f"row {b}"
        assert np.all(got[b, want:] == -7)


@pytest.mark.parametrize("kind", ["runs of 16", "runs of 64", "period"])
@pytest.mark.parametrize("n,k", [(65536, 1024), (300000, 4096), (1048576, 4096)])
def test_scores_that_resemble_their_neighbours_do_not_slow_the_long_rows(B, kind, n, k):
    """hca_topk by a sampled key: a row whose best slots lie side by side, or at a period that a careless choice of places
    meets, is sampled as fairly as any other - else its samples are now and then all among its best, and the whole row is
    listed by one workgroup (0.2 to 1.7 ms).  Every one of 24 calls over 8 such rows may take twice the time of independent
    scores; independent samples overrun six deviations, or what the selection holds, in none of 10^5."""
    rows = 8
    gen = torch.Generator(device="cuda").manual_seed(n)
    shape = B.make_shape(1, rows, rows, n)
    idx = torch.zeros(rows, k, dtype=torch.int32, device="cuda")
    count = torch.zeros(rows, dtype=torch.int32, device="cuda")
    ws = torch.empty(B.hca_workspace_bytes(shape, k, 1), dtype=torch.uint8, device="cuda")
    took = []
    for turn in range(25):
        sel = torch.randn(rows, n, generator=gen, device="cuda")
        if turn and kind == "period":
            sel += 9.0 * ((torch.arange(n, device="cuda") + turn) % 212 < 3)
        elif turn:
            run = int(kind[8:])
            base = torch.randn(rows, n // run + 1, generator=gen, device="cuda")
            sel = (0.05 * sel + base.repeat_interleave(run, 1)[:, :n]).contiguous()
        took.append(_passes_us(lambda: B.hca_topk(shape, sel, [n], k, idx, count, ws), 4))
        picked = sel.gather(1, idx.long()).sort(dim=1).values
        assert torch.equal(picked, sel.topk(k, dim=1).values.sort(dim=1).values)
    assert max(took[1:]) < 2 * took[0], f"{took[0]:.1f} us for independent scores, {max(took[1:]):.1f} us"


def test_rows_scanned_again_share_the_whole_chip(B):
    """hca_score_topk over 64 rows, all of them misread by their samples and scanned again: the second scan takes about as
    long as the first (the call 1.8 times one without), every compute unit has a part in it and its loads are ahead of its
    scores.  Allowed: twice; with a quarter of the chip idle and each wave waiting for its loads it was 2.24 times."""
    from paper_2507_19823_amd.session import LayerState
    batch, hkv, n, k = 8, 8, 131072, 1024
    gen = torch.Generator(device="cuda").manual_seed(64)
    q = torch.randn(batch, hkv, 128, generator=gen, device="cuda").half()
    st = LayerState(batch, hkv, hkv, n, 4, 32, k_max=k, m_max=1)
    idx = torch.empty(batch, hkv, k, dtype=torch.int32, device="cuda")
    count = torch.empty(batch, hkv, dtype=torch.int32, device="cuda")
    sampled = torch.zeros(n // 16, dtype=torch.bool, device="cuda")
    sampled[torch.arange(512, device="cuda") * (n // 16) // 512] = True
    took, resc = [], torch.empty(64, dtype=torch.int32, device="cuda")
    for misread in (False, True):
        keys = torch.empty(batch, hkv, n, 128, dtype=torch.float16, device="cuda")
        for r in range(64):
            u = torch.rand(n, generator=gen, device="cuda")
            proj = torch.where(sampled.repeat_interleave(16), 1.0 + u, -1.0 - u) if misread else 4 * u - 2
            qf = q[r // hkv, r % hkv].float()
            keys[r // hkv, r % hkv] = (proj[:, None] * qf[None] / qf.norm() ** 2 * 40.0).half()
        st.n = [0] * batch
        st.quantize(keys)
        del keys
        took.append(_passes_us(lambda: B.hca_score_topk(st.shape, st.kcache, q, st.n, k, idx, count, st.ws)))
        B.hca_score_topk_report(st.shape, st.n, st.ws, torch.empty_like(resc), resc)
        assert resc.tolist() == [int(misread)] * 64
    assert took[1] < 2.0 * took[0], f"{took[0]:.1f} us without, {took[1]:.1f} us with a second scan of every row"


@pytest.mark.parametrize("n", [4096, 16384, 40960])
@pytest.mark.parametrize("kind", ["sink", "low", "sinks and lows", "masked", "tail masked", "-inf"])
def test_a_few_far_scores_do_not_slow_the_short_rows(B, kind, n):
    """hca_topk of rows in one workgroup: values far outside of the others, or masked slots, must not widen the bins until the
    rest of the row shares one of them (two to four times the call).  Allowed: 1.7 times the time of normal rows, and the
    result is the stable sort's."""
    rows, k = 8, 1024
    gen = torch.Generator(device="cuda").manual_seed(n)
    normal = torch.randn(rows, n, generator=gen, device="cuda") * 10
    far = normal.clone()
    if kind in ("sink", "sinks and lows"):
        far[:, 17] = 1e6
    if kind in ("low", "sinks and lows"):
        far[:, n // 2] = -1e6
    if kind == "sinks and lows":
        far[:, n - 5], far[:, 3] = 1e4, -1e9
    if kind == "masked":
        far[torch.rand(rows, n, generator=gen, device="cuda") < 0.5] = torch.finfo(torch.float32).min
    if kind == "tail masked":
        far[:, n // 2:] = torch.finfo(torch.float32).min
    if kind == "-inf":
        far[torch.rand(rows, n, generator=gen, device="cuda") < 0.3] = -torch.inf
    shape = B.make_shape(1, rows, rows, n)
    idx = torch.zeros(rows, k, dtype=torch.int32, device="cuda")
    count = torch.zeros(rows, dtype=torch.int32, device="cuda")
    ws = torch.empty(B.hca_workspace_bytes(shape, k, 1), dtype=torch.uint8, device="cuda")
    took = [_passes_us(lambda: B.hca_topk(shape, sel, [n], k, idx, count, ws)) for sel in (normal, far)]
    ref = torch.sort(far, dim=1, descending=True, stable=True).indices[:, :k].sort(dim=1).values.int()
    assert torch.equal(idx, ref)
    assert took[1] < 1.7 * took[0], f"{took[0]:.1f} us for normal rows, {took[1]:.1f} us"


@pytest.mark.parametrize("bits,gs", [(4, 32), (2, 64)])
@pytest.mark.parametrize("n", [40960, 40961])
def test_score_topk_on_both_sides_of_the_short_row_line(B, oracle, bits, gs, n):
    """hca_score_topk: rows of up to 40 Ki slots are scored whole and selected in one launch, longer ones go through the
    sampled threshold; the report and the running monitor describe both."""
    k = 777
    w = S.Workload("line", 82 + bits, 2, 8, 2, n, bits, gs, k)
    d = S.make_layer(w, want_values=False)
    st = _layer(w, k)
    st.quantize(d["keys"].cuda())
    st.n = [n, 1000]
    R = 4
    idx = torch.full((R, k), -7, dtype=torch.int32, device="cuda")
    count = torch.full((R,), -7, dtype=torch.int32, device="cuda")
    cand, resc = torch.full((R,), -1, dtype=torch.int32, device="cuda"), torch.full((R,), -1, dtype=torch.int32, device="cuda")
    mon = torch.zeros(R, 4, dtype=torch.int32, device="cuda")
    st.ws.fill_(255)
    B.hca_score_topk_monitor(st.shape, st.ws, None, True)
    B.hca_score_topk(st.shape, st.kcache, d["q"].cuda(), st.n, k, idx, count, st.ws)
    B.hca_score_topk_report(st.shape, st.n, st.ws, cand, resc)
    B.hca_score_topk_monitor(st.shape, st.ws, mon, False)
    torch.cuda.synchronize()
    oc = oracle.Cache(R, n, 128, bits, gs)
    oracle.quantize(oc, d["keys"].numpy().reshape(R, n, 128))
    oc.n[...] = np.repeat(st.n, 2)
    sel, _ = oracle.score(oc, d["q"].numpy().reshape(-1, 128), want_z=False)
    ridx, rcount = oracle.topk(sel, oc.n, k)
    for r in range(R):
        c = int(rcount[r])
        assert int(count[r]) == c and np.array_equal(idx[r, :c].cpu().numpy(), ridx[r, :c])
    cand, mon = cand.cpu().numpy(), mon.cpu().numpy()
    assert int(resc.sum()) == 0
    assert np.array_equal(mon[:, 0], [1] * R) and np.array_equal(mon[:, 1], cand) and np.array_equal(mon[:, 2], cand)
    if n <= 40960:
        assert np.array_equal(cand, np.repeat(st.n, 2))
    else:
        assert k <= cand[0] < n // 2


@pytest.mark.parametrize("g,c,G,T,rows", [
    (32, 33, 1, 16000, 8), (32, 64, 4, 11000, 6), (32, 65, 1, 8200, 8), (32, 128, 4, 4200, 8), (32, 129, 4, 2100, 16),
    (32, 255, 1, 2100, 8), (32, 256, 4, 2047, 8), (32, 256, 4, 2303, 8), (64, 256, 4, 1100, 8), (64, 200, 1, 1500, 8),
    (32, 257, 1, 9, 2), (32, 300, 4, 127, 2), (32, 511, 1, 1025, 1), (64, 513, 1, 300, 3), (32, 1023, 1, 8, 3),
    (32, 1024, 1, 5, 3), (32, 2048, 1, 700, 1), (64, 2049, 4, 260, 1), (32, 8192, 1, 150, 2), (64, 8191, 1, 33, 1),
    (32, 56, 1, 18800, 8), (32, 64, 1, 10300, 8), (32, 65, 1, 16200, 8), (32, 128, 4, 5200, 8), (32, 129, 4, 4100, 16),
    (32, 255, 1, 2600, 8), (32, 256, 4, 2571, 8), (64, 64, 1, 12400, 8), (64, 80, 1, 14000, 8), (64, 160, 1, 7000, 8),
    (64, 256, 4, 3100, 8), (64, 257, 1, 40, 32), (32, 300, 1, 65, 128), (64, 700, 1, 129, 64),
    (32, 33, 1, 12100, 8), (32, 48, 4, 8111, 8), (32, 160, 1, 3333, 8), (64, 33, 4, 8193, 8), (64, 129, 1, 3060, 8)])
def test_bulk_assignment_equals_the_exhaustive_chain(B, g, c, G, T, rows):
    """hca_vq_assign: the matrix-core forms (up to 256 centroids, more than 256) and the vector forms give the indices of
    single-token calls, whose kernel evaluates the exact chain for every centroid; awkward tokens and centroids included."""
    dbar = 128 // g
    gen = torch.Generator(device="cuda").manual_seed(g * c + T)
    m = torch.ones(128, device="cuda")
    m[[3, 40, 77, 100]] = 8.0
    cen = torch.randn(rows, g, c, dbar, generator=gen, device="cuda") * m.view(1, g, 1, dbar)
    cen[:, 1, c // 2:] = cen[:, 1, : c - c // 2].clone()                   # duplicates: the lower index wins
    cen[:, 2, 1::2] = cen[:, 2, 0:-1:2][:, : c // 2] * (1 + 2.0 ** -22)     # pairs a last bit or two apart
    cen[:, 3] *= 1e-4
    if c > 40:
        cen[0, 4, 17] = 300.0                                              # |c|^2 beyond the shortlist's range
    cen = cen.contiguous()
    k = (torch.randn(1, rows, T, 128, generator=gen, device="cuda") * m).half()
    k[0, 0, T // 2] = 0.0
    k[0, 0, T // 3] *= 40.0                                                 # out of range
    k[0, -1, T - 1] = 65504.0
    k[0, 0, T // 4, : 2 * dbar] = 6e-8                                      # denormal
    k[0, 0, T // 5, 8 * dbar] = float("inf")
    k[0, 0, T // 6, 9 * dbar] = float("nan")
    at = torch.randint(0, c, (T,), generator=gen, device="cuda")
    k[0, 0, :, 5 * dbar: 6 * dbar] = cen[0, 5, at].half()                   # tokens on top of a centroid
    shape = B.make_shape(1, rows * G, rows, T + 9)
    cb = B.make_codebook(g, c, cen)
    bulk = torch.zeros(B.hca_vq_pcache_bytes(shape, cb), dtype=torch.uint8, device="cuda")
    single = torch.zeros_like(bulk)
    acc = torch.full((1, rows, T + 9), 7.0, device="cuda")
    pos = torch.full((1, rows, T + 9), -7, dtype=torch.int32, device="cuda")
    B.hca_vq_assign(shape, cb, bulk, k, T, [4], acc, pos, [100])
    for t in range(0, T, 8):
        part = k[:, :, t:t + 8].contiguous()
        B.hca_vq_assign(shape, cb, single, part, part.shape[2], [4 + t])
    torch.cuda.synchronize()
    assert torch.equal(bulk, single)
    want = torch.arange(100, 100 + T, dtype=torch.int32, device="cuda").expand(rows, T)
    assert torch.equal(pos[0, :, 4:4 + T], want) and (pos[0, :, :4] == -7).all() and (pos[0, :, 4 + T:] == -7).all()
    assert (acc[0, :, 4:4 + T] == 0).all() and (acc[0, :, :4] == 7).all() and (acc[0, :, 4 + T:] == 7).all()


@pytest.mark.parametrize("g,c,G,T,rows", [
    (32, 96, 1, 9, 8), (32, 100, 4, 65, 2), (32, 128, 1, 1025, 8), (32, 129, 4, 2047, 8), (32, 255, 1, 257, 16),
    (32, 256, 1, 4000, 8), (64, 256, 4, 1023, 8), (64, 256, 1, 64, 8), (64, 96, 1, 300, 4), (64, 200, 4, 1024, 2),
    (64, 256, 1, 64, 32), (32, 128, 1, 64, 64), (64, 96, 1, 1500, 8), (64, 128, 4, 1100, 8), (32, 160, 1, 3500, 8),
    (64, 256, 1, 7500, 1), (64, 256, 1, 9000, 1), (32, 33, 1, 14000, 4), (64, 48, 1, 9000, 8)])
def test_blocks_of_few_tokens_against_96_to_256_centroids(B, g, c, G, T, rows):
    """The shortlist form with one-byte and with two-byte indices, and the vector form on the other side of the line."""
    test_bulk_assignment_equals_the_exhaustive_chain(B, g, c, G, T, rows)


def _passes_us(run, passes=20):
    """Time of one pass in microseconds, the best of five batches."""
    run()
    best = float("inf")
    for _ in range(5):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(passes):
            run()
        b.record()
        b.synchronize()
        best = min(best, a.elapsed_time(b) * 1000 / passes)
    return best


@pytest.mark.parametrize("g,c,T,full,rows", [(64, 8192, 257, 384, 8), (64, 4096, 257, 384, 8), (32, 8192, 130, 256, 8),
                                             (32, 256, 1800, 2048, 16)])
def test_a_ragged_end_does_not_slow_the_assignment(B, g, c, T, full, rows):
    """The matrix-core forms take tokens by the wave; the places past a block's last token hold copies of that token, which
    must not be looked up one by one when it is one of the few that need the chain of every centroid (in one of a hundred
    groups it is).  A ragged block may take a quarter longer than the full one."""
    gen = torch.Generator(device="cuda").manual_seed(c + T)
    cen = torch.randn(rows, g, c, 128 // g, generator=gen, device="cuda")
    cb = B.make_codebook(g, c, cen)
    k = torch.randn(1, rows, full, 128, generator=gen, device="cuda").half()
    shape = B.make_shape(1, rows, rows, full)
    pc = torch.zeros(B.hca_vq_pcache_bytes(shape, cb), dtype=torch.uint8, device="cuda")
    part = k[:, :, :T].contiguous()
    took = [_passes_us(lambda: B.hca_vq_assign(shape, cb, pc, x, x.shape[2], [0])) for x in (k, part)]
    assert took[1] < 1.25 * took[0], f"{full} tokens {took[0]:.1f} us, {T} tokens {took[1]:.1f} us"


@pytest.mark.parametrize("g,c,T", [(64, 1024, 8192), (64, 8192, 2048), (32, 4096, 4096)])
def test_a_far_centroid_does_not_slow_the_assignment(B, g, c, T):
    """One centroid per group far from all keys (one that no training round ever moved, say) can win no token, so it must
    not widen the shortlist: a token with too many candidates costs the exact chain of every centroid, several times the
    call.  The time may rise by half at most; the indices are those without it."""
    rows, dbar = 8, 128 // g
    gen = torch.Generator(device="cuda").manual_seed(c + T)
    cen = torch.randn(rows, g, c, dbar, generator=gen, device="cuda")
    far = cen.clone()
    far[:, :, c // 3] = 0.0
    far[:, :, c // 3, 0] = 100.0                           # |c|^2 = 10^4, within the shortlist's range
    near = cen.clone()
    near[:, :, c // 3] = near[:, :, 0]                     # never chosen either: the lower index wins
    k = torch.randn(1, rows, T, 128, generator=gen, device="cuda").half()
    shape = B.make_shape(1, rows, rows, T)
    took, out = [], []
    for book in (near, far):
        cb = B.make_codebook(g, c, book)
        pc = torch.zeros(B.hca_vq_pcache_bytes(shape, cb), dtype=torch.uint8, device="cuda")
        took.append(_passes_us(lambda: B.hca_vq_assign(shape, cb, pc, k, T, [0])))
        out.append(pc)
    assert torch.equal(out[0], out[1])
    assert took[1] < 1.5 * took[0], f"{took[0]:.0f} us without the far centroid, {took[1]:.0f} us with it"


@pytest.mark.parametrize("kind,most", [("line", 5.0), ("repeated", 14.0)])
def test_rivals_in_many_blocks_do_not_slow_the_assignment(B, kind, most):
    """Thousands of centroids of which many lie close together, next to each other on a line or 64 points 128 times each:
    tokens with more near blocks than are kept look into those, not into all of the codebook.  Allowed: 5 and 14 times an
    ordinary codebook's time (measured 2.8 and 10; with every centroid looked at 12 and 20)."""
    rows, g, c, T = 8, 32, 8192, 2000
    gen = torch.Generator(device="cuda").manual_seed(c)
    shape = B.make_shape(1, rows, rows, T)
    took = []
    for now in ("normal", kind):
        k = torch.randn(1, rows, T, g, 4, generator=gen, device="cuda")
        cen = 1.1 * torch.randn(rows, g, c, 4, generator=gen, device="cuda")
        if now == "line":
            k, cen = k[..., :1] + 0.01 * k, cen[..., :1] + 0.01 * cen
        if now == "repeated":
            cen = cen[:, :, torch.randint(0, 64, (c,), generator=gen, device="cuda")].contiguous()
        cb = B.make_codebook(g, c, cen)
        keys = k.reshape(1, rows, T, 128).half()
        pc = torch.zeros(B.hca_vq_pcache_bytes(shape, cb), dtype=torch.uint8, device="cuda")
        took.append(_passes_us(lambda: B.hca_vq_assign(shape, cb, pc, keys, T, [0]), 5))
    assert took[1] < most * took[0], f"{took[0]:.0f} us normal, {took[1]:.0f} us {kind}"


@pytest.mark.parametrize("g,c,G", [(32, 256, 4), (64, 256, 4), (64, 256, 1), (32, 96, 4), (32, 250, 1)])
def test_assignment_queue_fills_at_any_group(B, oracle, g, c, G):
    """Up to 256 centroids: a share of every group's centroids (none to all, another one in each group) exists twice, so
    that a workgroup of 256 tokens has from none to all of them queued for the exact chain of every centroid in a group.  Its
    queue passes the fill that makes room for the next group after one, two or several groups, and in both halves of
    the record, with the last workgroup of a row ragged."""
    dbar, rows = 128 // g, 8
    T = int((3.05 if g == 64 else 2.05 if c == 96 else 1.3) * (1 << 27)) // (rows * g * c) + 131
    rng = np.random.default_rng(g + c + G)
    cen = rng.standard_normal((rows, g, c, dbar)).astype(np.float32)
    for i in range(g):
        twice = int(c // 2 * ((5 * i) % 8) / 7)
        cen[:, i, c - twice:] = cen[:, i, :twice]
    k = rng.standard_normal((1, rows, T, 128)).astype(np.float16)
    shape = B.make_shape(1, rows * G, rows, T + 3)
    dcen = torch.from_numpy(cen).cuda()
    cb = B.make_codebook(g, c, dcen)
    pc = torch.zeros(B.hca_vq_pcache_bytes(shape, cb), dtype=torch.uint8, device="cuda")
    oc = oracle.VQCache(rows, T, cen)
    oracle.vq_assign(oc, k.reshape(rows, T, 128))
    dk = torch.from_numpy(k).cuda()
    wide = g * c * G > 32768
    for _ in range(3):
        pc.fill_(0xEE)
        B.hca_vq_assign(shape, cb, pc, dk, T, [2])
        out = torch.full((rows, T + 3, g * (2 if wide else 1)), 0xEE, dtype=torch.uint8, device="cuda")
        B.hca_vq_export_pcache(shape, cb, pc, [T + 2], out)
        got = out.cpu().numpy()
        got = got.view(np.uint16) if wide else got
        assert np.array_equal(got[:, 2:T + 2], oc.P[:, :T].astype(got.dtype))


@pytest.mark.parametrize("g,c,rows", [(64, 1024, 8), (32, 2048, 8), (32, 4096, 8), (64, 1500, 3)])
def test_append_forms_agree(B, g, c, rows):
    """Eight tokens per call (one wave per group where that fills the chip) and one (four waves share a group's codebook)."""
    gen = torch.Generator(device="cuda").manual_seed(c)
    cen = torch.randn(rows, g, c, 128 // g, generator=gen, device="cuda")
    cen[:, 1, c // 2:] = cen[:, 1, : c - c // 2].clone()
    k = torch.randn(1, rows, 8, 128, generator=gen, device="cuda").half()
    shape = B.make_shape(1, rows, rows, 16)
    cb = B.make_codebook(g, c, cen)
    both = [torch.zeros(B.hca_vq_pcache_bytes(shape, cb), dtype=torch.uint8, device="cuda") for _ in range(2)]
    B.hca_vq_assign(shape, cb, both[0], k, 8, [2])
    for t in range(8):
        B.hca_vq_assign(shape, cb, both[1], k[:, :, t:t + 1].contiguous(), 1, [2 + t])
    assert torch.equal(both[0], both[1])


@pytest.mark.parametrize("g,c,rows,T", [(32, 33, 8, 32000), (64, 1024, 32, 8), (64, 257, 128, 64)])
def test_assignment_time_has_no_step(B, g, c, rows, T):
    """One centroid more, with which a launch rule could change the form: the call takes what the exact chain of one more
    centroid takes, not 1.6 to 3.3 times as much.  Allowed: 1.3 times."""
    gen = torch.Generator(device="cuda").manual_seed(c)
    hkv = min(rows, 8)
    k = torch.randn(rows // hkv, hkv, T, 128, generator=gen, device="cuda").half()
    shape = B.make_shape(rows // hkv, hkv, hkv, T)
    took = []
    for cc in (c - 1, c):
        cen = torch.randn(hkv, g, cc, 128 // g, generator=gen, device="cuda")
        cb = B.make_codebook(g, cc, cen)
        pc = torch.zeros(B.hca_vq_pcache_bytes(shape, cb), dtype=torch.uint8, device="cuda")
        took.append(_passes_us(lambda: B.hca_vq_assign(shape, cb, pc, k, T, [0] * (rows // hkv))))
    assert took[1] < 1.3 * took[0], f"{took[0]:.1f} us with {c - 1} centroids, {took[1]:.1f} with {c}"


@pytest.mark.parametrize("bits,gs", [(4, 32), (2, 64)])
@pytest.mark.parametrize("n,M,protect,kind,spare", [
    (4096, 4095, 0, "zeros", False), (4097, 2049, 1, "dense", True), (9000, 1, 0, "dense", False),
    (9001, 4500, 4500, "dense", True), (20483, 20000, 64, "ties", False), (20483, 8191, 16, "ties", True),
    (8192, 63, 5, "mixed", True), (12289, 12288, 3, "mixed", False)])
def test_evict_at_chunk_edges(B, bits, gs, n, M, protect, kind, spare):
    """hca_evict: keep-list, moved scores, value rows and codes on both sides of the 4096-slot chunk and 64-slot wave edges,
    with the threshold at 0 (one counting pass), above it, below it and inside long ties (radix passes)."""
    w = S.Workload("ev", 83, 2, 4, 2, n, bits, gs, 8)
    d = S.make_layer(w, want_values=False)
    st = _layer(w, 8, m_max=M)
    st.quantize(d["keys"].cuda())
    codes0, scale0, zero0 = st.export()
    rng = np.random.default_rng(n + M)
    acc = np.zeros((4, n), np.float32)
    if kind == "zeros":
        acc[:, ::50] = rng.random((4, len(range(0, n, 50))))
    elif kind == "dense":
        acc[:] = rng.random((4, n)) + 0.5
    elif kind == "ties":
        acc[:] = rng.integers(1, 4, (4, n))
    else:                                                    # negative values and both zeros: the threshold lies below 0
        acc[:] = rng.standard_normal((4, n)) - 2
        acc[:, ::7], acc[:, 1::7] = 0.0, -0.0
    lens = [n, max(M, n - 100)]                              # the second sequence may have nothing to evict
    st.acc.copy_(torch.from_numpy(acc).view(2, 2, n))
    st.pos.copy_(torch.randint(0, 1 << 20, st.pos.shape, dtype=torch.int32, device="cuda"))
    pos0 = st.pos.cpu().numpy().reshape(4, n)
    st.n = list(lens)
    kept = torch.full((2, 2, M), -5, dtype=torch.int32, device="cuda")
    dst = (torch.zeros_like(st.kcache), torch.zeros_like(st.acc), torch.zeros_like(st.pos)) if spare else None
    st.evict(M, protect, kept, spare=dst)
    codes, scale, zero = st.export()
    torch.cuda.synchronize()
    kept = kept.cpu().numpy().reshape(4, M)
    flat = lambda x: x.cpu().numpy().reshape(4, n, -1)  # noqa: E731
    for r in range(4):
        ln = lens[r // 2]
        if ln <= M:
            assert np.all(kept[r] == -5)
            ref = np.arange(ln)
        else:
            ns = ln - protect
            key = _order_key(acc[r, :ns]).astype(np.int64)
            ref = np.concatenate([np.sort(np.argsort(-key, kind="stable")[:M - protect]), np.arange(ns, ln)])
            assert np.array_equal(kept[r], ref), f"row {r}"
        m = len(ref)
        assert np.array_equal(flat(st.acc)[r, :m, 0], acc[r, ref]) and np.array_equal(flat(st.pos)[r, :m, 0], pos0[r, ref])
        assert np.array_equal(flat(codes)[r, :m], flat(codes0)[r, ref])
        assert np.array_equal(flat(scale.view(torch.int16))[r, :m], flat(scale0.view(torch.int16))[r, ref])
        assert np.array_equal(flat(zero.view(torch.int16))[r, :m], flat(zero0.view(torch.int16))[r, ref])


@pytest.mark.parametrize("kind", ["far", "masked", "steps", "close"])
@pytest.mark.parametrize("n", [4096, 4097, 8193, 40961])
def test_topp_at_the_edges_of_its_bins(B, oracle, kind, n):
    """hca_topp bins by weight down to 2^-64 and by score within a window: rows whose slots nearly all weigh nothing, lie
    exactly on bin edges, are masked with -inf or the type's lowest value, or share one bin."""
    rng = np.random.default_rng(n)
    cap, R = n + 5, 3
    sel = np.full((R, cap), 1e30, np.float32)
    for r in range(R):
        if kind == "far":
            x = np.float32(-200) - rng.random(n).astype(np.float32) * 1e4
            x[rng.integers(0, n, 40)] = rng.standard_normal(40)
        elif kind == "masked":
            x = rng.standard_normal(n).astype(np.float32) * 3
            x[rng.random(n) < 0.5] = -np.inf if r else np.finfo(np.float32).min
        elif kind == "steps":                                # multiples of a power of two's 32nd part in logit
            x = (rng.integers(0, 2100, n) * (-np.log(2) / 32)).astype(np.float32)
        else:
            x = (5 + rng.random(n) * 1e-5).astype(np.float32)
        sel[r, :n] = x
    lens = [n, n - 1, max(1, n // 2)]
    shape = B.make_shape(3, 1, 1, cap)
    for tau, k_max in ((0.3, n), (0.999, n), (1.0, n), (0.9, 50)):
        idx = torch.full((R, k_max), -9, dtype=torch.int32, device="cuda")
        count = torch.full((R,), -9, dtype=torch.int32, device="cuda")
        mass = torch.full((R, 2), 7, dtype=torch.int64, device="cuda")
        ws = torch.full((B.hca_workspace_bytes(shape, k_max, 1),), 255, dtype=torch.uint8, device="cuda")
        B.hca_topp(shape, torch.from_numpy(sel).cuda(), lens, 1.0, tau, k_max, idx, count, mass, ws)
        torch.cuda.synchronize()
        oidx, ocount, _, omass = oracle.topp(sel, lens, 1.0, tau, k_max)
        assert np.array_equal(mass.cpu().numpy().view(np.uint64), omass) and np.array_equal(count.cpu().numpy(), ocount)
        for r in range(R):
            assert np.array_equal(idx[r, :ocount[r]].cpu().numpy(), oidx[r, :ocount[r]]), (r, tau)


def _spread_scores(kind, rows, n, gen):
    """Rows whose slots crowd in a narrow band, or do not, with and without what lies far outside of it."""
    x = torch.randn(rows, n, generator=gen, device="cuda")
    at = torch.arange(n, device="cuda")
    if kind == "flat":
        x = x * 0.1
    elif kind == "flat, sink and low":
        x = x * 1e-3
        x[:, 5], x[:, 7] = 120.0, -300.0
    elif kind == "flat, half masked":
        x = torch.where(torch.rand(rows, n, generator=gen, device="cuda") < 0.5, torch.finfo(torch.float32).min, x * 0.1)
    elif kind == "flat, tail masked":
        x = torch.where(at >= n // 2, -torch.inf, x * 1e-3)
    elif kind == "far from zero":
        x = 50 + x * 0.01
    elif kind == "drift":
        x = x * 5 + at * (60.0 / n)
    elif kind == "two bands":
        x = torch.where(at < n // 100, x * 3 + 60, x)
    else:
        x = x * 11
    return x


@pytest.mark.parametrize("kind", ["flat", "flat, sink and low", "flat, half masked", "flat, tail masked", "far from zero",
                                  "drift", "two bands", "normal"])
@pytest.mark.parametrize("n", [65, 300, 9000, 140001])
def test_topp_whatever_the_spread(B, oracle, kind, n):
    """The window of the fine bins, found from two or from sixteen waves of a row; bins resolved by direct comparison (up to 128
    keys), from LDS and from the lists; lists shared by the waves (up to eight chunks) and not."""
    R, cap = 3, n + 2
    sel = torch.full((R, cap), 1e30, device="cuda")
    sel[:, :n] = _spread_scores(kind, R, n, torch.Generator(device="cuda").manual_seed(n))
    lens = [n, n - 1, max(1, n // 2)]
    shape = B.make_shape(3, 1, 1, cap)
    host = sel.cpu().numpy()
    for tau, k_max in ((0.5, n), (0.9, n), (1.0, n), (0.9, max(1, n // 30))):
        idx = torch.full((R, k_max), -9, dtype=torch.int32, device="cuda")
        count = torch.full((R,), -9, dtype=torch.int32, device="cuda")
        mass = torch.full((R, 2), 7, dtype=torch.int64, device="cuda")
        ws = torch.full((B.hca_workspace_bytes(shape, k_max, 1),), 255, dtype=torch.uint8, device="cuda")
        B.hca_topp(shape, sel, lens, 0.0884, tau, k_max, idx, count, mass, ws)
        oidx, ocount, _, omass = oracle.topp(host, lens, 0.0884, tau, k_max)
        assert np.array_equal(mass.cpu().numpy().view(np.uint64), omass) and np.array_equal(count.cpu().numpy(), ocount)
        for r in range(R):
            assert np.array_equal(idx[r, :ocount[r]].cpu().numpy(), oidx[r, :ocount[r]]), (r, tau)


@pytest.mark.parametrize("kind", ["flat", "flat, sink and low", "flat, half masked", "flat, tail masked"])
def test_topp_time_does_not_hang_on_the_spread(B, kind):
    """A row of nearly equal weights has to be resolved as finely as any other: its bin of interest must not hold most of the
    row, which one workgroup would then go through alone (five times the call).  Allowed: twice the time of normal rows."""
    rows, n, k = 8, 131072, 4096
    shape = B.make_shape(1, rows, rows, n)
    idx = torch.zeros(rows, k, dtype=torch.int32, device="cuda")
    count = torch.zeros(rows, dtype=torch.int32, device="cuda")
    ws = torch.empty(B.hca_workspace_bytes(shape, k, 1), dtype=torch.uint8, device="cuda")
    took = []
    for which in ("normal", kind):
        sel = _spread_scores(which, rows, n, torch.Generator(device="cuda").manual_seed(3))
        took.append(_passes_us(lambda: B.hca_topp(shape, sel, [n], 0.0884, 0.9, k, idx, count, None, ws)))
    assert took[1] < 2 * took[0], f"{took[0]:.0f} us for normal rows, {took[1]:.0f} us"


@pytest.mark.parametrize("gqa,groups,c", [(4, 32, 64), (2, 64, 256), (1, 32, 256), (4, 32, 1024)])
def test_codebook_attend_of_many_rows_equals_that_of_few(B, gqa, groups, c):
    """hca_vq_attend_gathered asks for the values before the table reads in launches of at most 256 workgroups and in the wide
    form, else behind them; 17 sequences of 8 KV heads in one call (more than 256 workgroups) and one at a time."""
    batch, hkv, n, k = 17, 8, 1500, 700
    gen = torch.Generator(device="cuda").manual_seed(c + gqa)
    cen = torch.randn(hkv, groups, c, 128 // groups, generator=gen, device="cuda")
    cb = B.make_codebook(groups, c, cen)
    keys = torch.randn(batch, hkv, n, 128, generator=gen, device="cuda").half()
    q = torch.randn(batch, hkv * gqa, 128, generator=gen, device="cuda").half()
    v = torch.randn(batch, hkv, n, 128, generator=gen, device="cuda").half()
    idx = torch.stack([torch.randperm(n, generator=gen, device="cuda")[:k].sort().values for _ in range(batch * hkv)])
    idx = idx.int().view(batch, hkv, k).contiguous()
    count = torch.full((batch, hkv), k, dtype=torch.int32, device="cuda")
    count[3], count[5, 2] = 513, 0

    def run(b):
        part = slice(b, b + 1) if b is not None else slice(0, batch)
        nb = 1 if b is not None else batch
        shape = B.make_shape(nb, hkv * gqa, hkv, n)
        pc = torch.zeros(B.hca_vq_pcache_bytes(shape, cb), dtype=torch.uint8, device="cuda")
        B.hca_vq_assign(shape, cb, pc, keys[part].contiguous(), n, [0] * nb)
        lut = torch.zeros(B.hca_vq_lut_bytes(shape, cb) // 4, device="cuda")
        sel = torch.zeros(nb, hkv, n, device="cuda")
        qq = q[part].contiguous()
        B.hca_vq_score(shape, cb, pc, qq, [n] * nb, lut, sel)
        ws = torch.zeros(B.hca_vq_workspace_bytes(shape, cb, k), dtype=torch.uint8, device="cuda")
        pos = torch.arange(n, dtype=torch.int32, device="cuda").repeat(nb * hkv).view(nb, hkv, n).contiguous()
        ii, cc, y = idx[part].contiguous(), count[part].contiguous(), torch.full((nb, hkv * gqa, 128), 9.0, device="cuda")
        acc = torch.zeros(nb, hkv, n, device="cuda")
        B.hca_gather_values(shape, ii, cc, k, pos, None, 0, 0, v[part].contiguous(), n, ws)
        B.hca_vq_attend_gathered(shape, cb, pc, lut, ii, cc, k, 0.0884, y, acc, ws)
        torch.cuda.synchronize()
        return y, acc
    y, acc = run(None)
    one = [run(b) for b in range(batch)]
    assert torch.equal(torch.nan_to_num(y, 7.0), torch.nan_to_num(torch.cat([o[0] for o in one]), 7.0))
    assert torch.equal(acc, torch.cat([o[1] for o in one])) and (acc > 0).any()
    keep = torch.ones(batch, hkv, dtype=torch.bool)
    keep[5, 2] = False
    assert torch.isfinite(y.view(batch, hkv, gqa, 128)[keep.cuda()]).all()


@pytest.mark.parametrize("gqa,groups,c,n", [(4, 32, 8192, 12288), (4, 32, 300, 12289), (4, 64, 513, 16384), (4, 32, 1024, 16385),
                                            (2, 32, 8192, 12289), (1, 64, 8192, 257), (1, 32, 511, 4097)])
def test_wide_codebook_scan_shares(B, gqa, groups, c, n):
    # 256 rows: one share per row up to 12 Ki slots, 16 Ki above, two above that; every 37th row has fewer tokens.
    # The scores are integer sums on a power-of-two grid, so they have to be equal
    rows, batch = 8, 32
    sh = B.make_shape(batch, rows * gqa, rows, n + 3)
    gen = torch.Generator(device="cuda").manual_seed(n + c)
    cen = torch.randn(rows, groups, c, 128 // groups, device="cuda", generator=gen)
    cb = B.make_codebook(groups, c, cen)
    size = B.hca_vq_pcache_bytes(sh, cb) // 2
    pc = torch.randint(0, c, (size,), device="cuda", dtype=torch.int16, generator=gen)
    q = torch.randn(batch, rows * gqa, 128, device="cuda", generator=gen).half()
    lut = torch.zeros(B.hca_vq_lut_bytes(sh, cb) // 4, device="cuda")
    sel = torch.full((batch, rows, n + 3), -7.0, device="cuda")
    z = torch.full((batch, rows * gqa, n + 3), -7.0, device="cuda")
    lens = [n if b % 5 else max(1, n - 300 * (b + 1)) for b in range(batch)]
    B.hca_vq_score(sh, cb, pc.view(torch.uint8), q, lens, lut, sel, z)
    torch.cuda.synchronize()
    tile = 16384
    tiles = (n + 3 + tile - 1) // tile
    codes = pc.view(batch * rows, tiles, groups, tile)
    table = lut[: batch * rows * groups * c * gqa].view(batch * rows, groups, c, gqa)
    for row in (0, 7, 8, 121, 255):
        m = lens[row // rows]
        expo = (24 - torch.frexp(table[row].abs().amax((0, 1))).exponent).tolist()
        scale = torch.tensor([2.0 ** e for e in expo], dtype=torch.float64, device="cuda")       # exact powers of two
        fix = torch.round(table[row].double() * scale).long()
        total = torch.zeros(tiles * tile, gqa, dtype=torch.long, device="cuda")
        for i in range(groups):
            total += fix[i][codes[row, :, i].reshape(-1).long()]
        want = (total.float().double() / scale).float()[:m]
        got = z.view(batch * rows, gqa, n + 3)[row]
        assert torch.equal(got[:, :m].T, want), (row, m)
        assert torch.equal(sel.view(batch * rows, n + 3)[row, :m], want.amax(1))
        assert bool((got[:, m:] == -7.0).all()) and bool((sel.view(batch * rows, n + 3)[row, m:] == -7.0).all())
