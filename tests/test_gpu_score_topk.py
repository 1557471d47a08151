"""GPU parity of hca_score_topk (scan and top-k in one call, Sec. 3.2) against the oracle's score + top-k."""
import numpy as np
import pytest
import torch

import synth_inputs as S

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def H():
    import paper_2507_19823_amd as H
    assert torch.cuda.is_available(), "GPU tests need the MI355X"
    H.lib()
    return H


@pytest.fixture(autouse=True, params=[0, 256], ids=["default", "wg256"])
def select_wg(request, H):
    """Every case runs with two forms of the selection over the candidate lists: the default one (1024 threads for a
    call, 512 in a step driver) and the one of 256 threads.  (Rows of up to 96 Ki in small batches are selected from their
    scores, whatever the form.)"""
    H.hca_tune("select_wg", request.param)
    yield request.param
    H.hca_tune("select_wg", 0)


def _rows(t):
    a = t.detach().cpu().numpy()
    return a.reshape(a.shape[0] * a.shape[1], *a.shape[2:])


def _run(H, oracle, w, keys, q, lens, k):
    """Quantises `keys` on both sides, cuts the sequences to `lens`, selects k per row; compares index sets."""
    from paper_2507_19823_amd import binding as B
    from paper_2507_19823_amd.session import LayerState
    st = LayerState(w.batch, w.n_q_heads, w.n_kv_heads, w.n, w.bits, w.group, k_max=k, want_z=False)
    oc = oracle.Cache(w.batch * w.n_kv_heads, w.n, 128, w.bits, w.group)
    st.quantize(keys.cuda())
    oracle.quantize(oc, _rows(keys))
    st.n = list(lens)
    oc.n[...] = np.repeat(lens, w.n_kv_heads)
    R = w.batch * w.n_kv_heads
    idx = torch.full((R, k), -9, dtype=torch.int32, device="cuda")
    count = torch.full((R,), -9, dtype=torch.int32, device="cuda")
    B.hca_score_topk(st.shape, st.kcache, q.cuda(), st.n, k, idx, count, st.ws)
    torch.cuda.synchronize()
    sel, _ = oracle.score(oc, q.numpy().reshape(-1, 128), want_z=False)
    ridx, rcount = oracle.topk(sel, oc.n, k)
    gi, gc = idx.cpu().numpy(), count.cpu().numpy()
    for r in range(R):
        c = min(k, lens[r // w.n_kv_heads])
        assert gc[r] == c == rcount[r], f"row {r}: count {gc[r]} / {rcount[r]} / {c}"
        assert np.array_equal(gi[r, :c], ridx[r, :c]), f"row {r}: index sets differ"
        assert np.all(gi[r, c:] == -9)
    cand = torch.full((R,), -1, dtype=torch.int32, device="cuda")
    resc = torch.full((R,), -1, dtype=torch.int32, device="cuda")
    B.hca_score_topk_report(st.shape, st.n, st.ws, cand, resc)
    torch.cuda.synchronize()
    return cand.cpu().numpy(), resc.cpu().numpy()


@pytest.mark.parametrize("bits,gs", [(4, 32), (2, 64)])
@pytest.mark.parametrize("n,k,lens", [
    (300, 64, [300, 17]), (5000, 256, [5000, 0]), (5000, 5000, [4999, 5000]), (70001, 2048, [70001, 33000]),
    (300000, 1024, [300000, 150001]),
])
def test_score_topk_matches_the_oracle(H, oracle, bits, gs, n, k, lens):
    w = S.Workload("st", 90 + bits, 2, 8, 2, n, bits, gs, k)
    d = S.make_layer(w, want_values=False)
    cand, resc = _run(H, oracle, w, d["keys"], d["q"], lens, k)
    for r in range(w.batch * w.n_kv_heads):
        nr_ = lens[r // w.n_kv_heads]
        if nr_ > 0:
            assert min(k, nr_) <= cand[r] <= nr_
            assert resc[r] == 0, "seeded random keys: the sampled threshold must hold"
    if n >= 70001:      # long rows: the threshold discards almost everything
        assert cand[0] < n // 8


@pytest.mark.parametrize("bits,gs", [(4, 32), (2, 64)])
def test_the_largest_k(H, oracle, bits, gs):
    """k = 16384, the most the step driver accepts: more candidates than are held in registers, one row barely
    longer than k."""
    n, k = 120000, 16384
    lens = [n, k + 5]
    w = S.Workload("stmax", 95 + bits, 2, 8, 2, n, bits, gs, k)
    d = S.make_layer(w, want_values=False)
    cand, resc = _run(H, oracle, w, d["keys"], d["q"], lens, k)
    assert int(cand.min()) >= k


@pytest.mark.parametrize("hq,hkv", [(4, 2), (2, 2), (6, 3)])
def test_fewer_query_heads_per_kv_head(H, oracle, hq, hkv):
    """Groups of two query heads and of one: the selection score is the maximum over the heads that exist."""
    w = S.Workload("gqa", 97 + hq, 2, hq, hkv, 40000, 4, 32, 512)
    d = S.make_layer(w, want_values=False)
    _run(H, oracle, w, d["keys"], d["q"], [40000, 12345], 512)


def test_ties_in_a_row_of_medium_length(H, oracle):
    """Every key the same, 50 000 slots: none scores above the sampled key, the k lowest slots of those equal to it win."""
    w = S.Workload("tie", 95, 1, 4, 1, 50000, 4, 32, 777)
    d = S.make_layer(w, want_values=False)
    keys = d["keys"][:, :, :1].expand(-1, -1, w.n, -1).contiguous()
    cand, resc = _run(H, oracle, w, keys, d["q"], [w.n], w.k)
    assert cand[0] == w.n and resc[0] == 0        # one key value: none below the sampled key


def _tied_layer(w, tied):
    """Keys of which `tied` per row, here and there, are the same and score highest; the others random."""
    d = S.make_layer(w, want_values=False)
    q = d["q"].clone()
    q[:, 1:] = q[:, :1]                                       # four equal query heads
    keys = d["keys"].clone()
    g = torch.Generator().manual_seed(tied)
    for b in range(w.batch):
        at = torch.randperm(w.n, generator=g)[:tied]
        keys[b, 0, at] = (q[b, 0].float() * 100 / q[b, 0].float().norm()).half()
    return dict(d, q=q, keys=keys)


@pytest.mark.parametrize("bits,gs", [(4, 32), (2, 64)])
@pytest.mark.parametrize("n,tied,k,second", [
    (150000, 150000, 777, 150000), (150000, 20000, 4000, 60000), (150000, 60000, 1, 33333), (200000, 66000, 16000, 200000),
    (150000, 17000, 16999, 20000), (120000, 30000, 31000, 100000)])
def test_ties_in_lists_too_long_for_the_registers(H, oracle, bits, gs, n, tied, k, second):
    """The selecting scan's lists with more than 16 384 pairs at one key, some or all of them to be taken: up to 65 536
    pairs found by position, more walked chunk by chunk; the lowest slots win."""
    w = S.Workload("tied", 93 + bits, 2, 4, 1, n, bits, gs, k)
    d = _tied_layer(w, tied)
    cand, resc = _run(H, oracle, w, d["keys"], d["q"], [n, second], k)
    assert cand[0] >= max(k, tied) and resc[0] == 0


@pytest.mark.parametrize("bits,gs,tpb", [(4, 32, 16), (2, 64, 32)])
def test_a_sample_that_misleads_still_gives_the_exact_set(H, oracle, bits, gs, tpb):
    """The sample reads block floor(s * nblocks / S), s < S = 8192 / (slots per block).  Those blocks get keys along
    the query (large scores), all others keys against it: the sampled threshold then admits far fewer than k
    slots and the row has to go through the second, unthresholded scan."""
    n, k = 200000, 1024
    w = S.Workload("mis", 96 + bits, 1, 4, 1, n, bits, gs, k)
    d = S.make_layer(w, want_values=False)
    q = d["q"].clone()
    q[0, 1:] = q[0, :1]                                       # four equal query heads
    g = torch.Generator().manual_seed(5)
    noise = 0.05 * torch.randn(n, 128, generator=g)
    nblocks = (n + tpb - 1) // tpb
    Sn = min(nblocks, 8192 // tpb)
    sampled = torch.zeros(nblocks, dtype=torch.bool)
    sampled[(torch.arange(Sn, dtype=torch.int64) * nblocks) // Sn] = True
    sign = torch.where(sampled.repeat_interleave(tpb)[:n], 1.0, -1.0)[:, None]
    keys = (sign * q[0, 0].float()[None, :] * (0.5 + torch.rand(n, 1, generator=g)) + noise).to(torch.float16)
    cand, resc = _run(H, oracle, w, keys[None, None], q, [n], k)
    assert resc[0] == 1 and k <= cand[0] <= n      # the row went through the second scan


@pytest.mark.parametrize("bits,gs,tpb", [(4, 32, 16), (2, 64, 32)])
@pytest.mark.parametrize("lens", [(230001, 100003, 1), (150000, 230001, 0)])
def test_several_rows_of_a_call_need_the_second_scan(H, oracle, bits, gs, tpb, lens):
    """Three sequences of two KV heads: the first head's rows are misread as above and scanned again, some with the second
    threshold and some whole, the other head's are not, and rows shorter than k, of one slot or of none are among them; twice
    on one workspace, as the second scan's counts live where the next call's samples go."""
    n, k, batch, hkv = 230001, 3000, 3, 2
    w = S.Workload("mis3", 97 + bits, batch, 2 * hkv, hkv, n, bits, gs, k)
    d = S.make_layer(w, want_values=False)
    q = d["q"].clone()
    q[:, 1] = q[:, 0]                                          # head 0's two query heads are equal
    g = torch.Generator().manual_seed(6)
    keys = d["keys"].clone()
    for b in range(batch):
        nblocks = max(1, (lens[b] + tpb - 1) // tpb)
        Sn = min(nblocks, 8192 // tpb)
        sampled = torch.zeros((n + tpb - 1) // tpb, dtype=torch.bool)
        sampled[(torch.arange(Sn, dtype=torch.int64) * nblocks) // Sn] = True
        inside = sampled.repeat_interleave(tpb)[:n]
        u = torch.rand(n, generator=g)
        mid = torch.rand(n, generator=g) < (0.05 if b != 1 else 0.0)
        proj = torch.where(inside, 1.0 + u, torch.where(mid, 1.85 + 0.1 * u, -1.0 - u))
        keys[b, 0] = (proj[:, None] * q[b, 0].float()[None, :] / q[b, 0].float().norm() ** 2 * 40.0
                      + 0.02 * torch.randn(n, 128, generator=g)).to(torch.float16)
    for _ in range(2):
        cand, resc = _run(H, oracle, w, keys, q, lens, k)
        for b in range(batch):
            if lens[b] > 8192:
                assert resc[2 * b] == 1 and resc[2 * b + 1] == 0
                assert k <= cand[2 * b] <= lens[b] and cand[2 * b + 1] >= k


@pytest.mark.parametrize("bits,gs,tpb", [(4, 32, 16), (2, 64, 32)])
@pytest.mark.parametrize("batch,hkv", [(8, 8), (13, 5)], ids=["64rows", "65rows"])
@pytest.mark.parametrize("k", [1000, 6000])
@pytest.mark.parametrize("bad", ["all", "odd", "allbutone"])
def test_most_rows_of_a_large_call_need_the_second_scan(H, kernels_of, select_wg, bits, gs, tpb, batch, hkv, k, bad):
    """64 rows, the most that one launch finishes, and 65, of ragged lengths: every row, every other one or all but one
    misread by their samples and scanned again, by the second threshold (k = 1000) or whole (6000), so that each workgroup
    of the launch has a share of a row and some rows' own take part.  Against the selection from written scores, twice
    on one workspace."""
    from paper_2507_19823_amd import binding as B
    from paper_2507_19823_amd.session import LayerState
    n, rows = 45000, batch * hkv
    lens = [n - 1301 * (b % 5) for b in range(batch)]
    g = torch.Generator(device="cuda").manual_seed(rows + k + bits)
    q = torch.randn(batch, hkv, 128, generator=g, device="cuda").half()
    misread = [{"all": True, "odd": r % 2 == 1, "allbutone": r != rows // 2}[bad] for r in range(rows)]
    st = LayerState(batch, hkv, hkv, n, bits, gs, k_max=k)
    keys = torch.empty(batch, hkv, n, 128, dtype=torch.float16, device="cuda")
    for r in range(rows):
        b, h = r // hkv, r % hkv
        nblocks = (lens[b] + tpb - 1) // tpb
        Sn = min(nblocks, 8192 // tpb)
        sampled = torch.zeros((n + tpb - 1) // tpb, dtype=torch.bool, device="cuda")
        sampled[(torch.arange(Sn, device="cuda") * nblocks) // Sn] = True
        u = torch.rand(n, generator=g, device="cuda")
        proj = torch.where(sampled.repeat_interleave(tpb)[:n], 1.0 + u, -1.0 - u) if misread[r] else 4 * u - 2
        qf = q[b, h].float()
        noise = 0.02 * torch.randn(n, 128, generator=g, device="cuda")
        keys[b, h] = (proj[:, None] * qf[None] / qf.norm() ** 2 * 40.0 + noise).half()
    st.quantize(keys)
    st.n = list(lens)
    st.score(q)
    st.topk(k)
    ref, ref_count = st.idx.clone(), st.count.clone()
    form = kernels_of(lambda: B.hca_score_topk(st.shape, st.kcache, q, st.n, k, st.idx, st.count, st.ws))
    assert any("tk_finish" in x for x in form) == (rows <= 64 and select_wg == 0), form
    for _ in range(2):
        idx = torch.full((batch, hkv, k), -9, dtype=torch.int32, device="cuda")
        count = torch.full((batch, hkv), -9, dtype=torch.int32, device="cuda")
        cand, resc = (torch.full((rows,), -1, dtype=torch.int32, device="cuda") for _ in range(2))
        B.hca_score_topk(st.shape, st.kcache, q, st.n, k, idx, count, st.ws)
        B.hca_score_topk_report(st.shape, st.n, st.ws, cand, resc)
        torch.cuda.synchronize()
        assert torch.equal(count, ref_count) and torch.equal(idx, ref)
        assert resc.tolist() == [int(x) for x in misread] and int(cand.min()) >= k


def test_second_scan_with_the_deeper_threshold(H, oracle):
    """As above, but the slots outside the sampled blocks score only a little lower than those inside: the first
    threshold (inside the sampled blocks' range) lets too few through, the second one - the 8r-th largest sample,
    counted against during the first scan - lets enough through, and the second scan keeps far fewer than n."""
    n, k, tpb = 300000, 2048, 16
    w = S.Workload("mis2", 99, 1, 4, 1, n, 4, 32, k)
    d = S.make_layer(w, want_values=False)
    q = d["q"].clone()
    q[0, 1:] = q[0, :1]
    g = torch.Generator().manual_seed(7)
    nblocks = (n + tpb - 1) // tpb
    Sn = min(nblocks, 8192 // tpb)
    sampled = torch.zeros(nblocks, dtype=torch.bool)
    sampled[(torch.arange(Sn, dtype=torch.int64) * nblocks) // Sn] = True
    inside = sampled.repeat_interleave(tpb)[:n]
    # projection on the query (x 40 = score): inside the sampled blocks uniform in [1.0, 2.0], so the first
    # threshold (123rd largest sample) sits near 1.985 and the second (984th, rounded down to its 12-bit bin:
    # scores 72..80) at 1.8; outside, 3 % of the slots uniform in [1.85, 1.95] - below the first, above the
    # second, some 8700 of them -, the rest negative
    u = torch.rand(n, generator=g)
    mid = torch.rand(n, generator=g) < 0.03
    proj = torch.where(inside, 1.0 + u, torch.where(mid, 1.85 + 0.1 * u, -1.0 - u))
    keys = (proj[:, None] * q[0, 0].float()[None, :] / q[0, 0].float().norm() ** 2 * 40.0
            + 0.02 * torch.randn(n, 128, generator=g)).to(torch.float16)
    cand, resc = _run(H, oracle, w, keys[None, None], q, [n], k)
    assert resc[0] == 1 and k <= cand[0] < n // 4


@pytest.mark.parametrize("kind", ["crowded", "misread", "equal"])
@pytest.mark.parametrize("n", [41000, 70000, 98304])
def test_rows_of_medium_length(H, oracle, n, kind):
    """Rows whose scores are written and selected from: the best slots crowded into a few thousand neighbours (more than a
    chunk's room for pairs), a row its samples misrepresent (their places as topk_sample_rank takes them), equal scores."""
    from test_gpu_dispatch import _sampled_slots
    k = 3000
    w = S.Workload("mid", 91, 2, 4, 1, n, 4, 32, k)
    d = S.make_layer(w, want_values=False)
    q = d["q"].clone()
    q[:, 1:] = q[:, :1]                                       # four equal query heads
    g = torch.Generator().manual_seed(n)
    large = torch.zeros(n, dtype=torch.bool)
    if kind == "crowded":
        large[20000:24500] = True
    elif kind == "misread":
        large[torch.from_numpy(_sampled_slots(n))] = True
    size = torch.where(large, 1.0, -1.0)[:, None] * (0.5 + torch.rand(n, 1, generator=g))
    keys = (size * q[:, 0].float()[:, None, :] + 0.02 * torch.randn(2, n, 128, generator=g)).to(torch.float16)[:, None]
    if kind == "equal":
        keys = keys[:, :, :1].expand(-1, -1, n, -1).contiguous()
    lens = [n, n - 7 if kind == "crowded" else 5000]
    cand, resc = _run(H, oracle, w, keys, q, lens, k)
    # misread: only sampled slots score high, so those above the r-th largest sample are r - 1 <= 766 (n = 41 000) < k; the
    # second key, the 4r-th, lets 3064 or more through there and too few (4r = 1460, at 98 304) in the longest rows
    assert cand[0] >= k and resc[0] == (kind == "misread")
    if kind == "misread" and n != 70000:
        assert (cand[0] == n) == (n == 98304)


@pytest.mark.parametrize("run", [16, 64])
def test_rows_of_medium_length_whose_neighbours_resemble_each_other(H, run):
    """No row of 320 in runs of equal direction misleads its samples (16 neighbouring slots per sample do so in one of 75)."""
    from paper_2507_19823_amd import binding as B
    from paper_2507_19823_amd.session import LayerState
    b, hkv, n, k = 2, 8, 65536, 1024
    g = torch.Generator(device="cuda").manual_seed(run)
    st = LayerState(b, hkv, hkv, n, 4, 32, k_max=k, want_z=False)
    idx = torch.zeros(b, hkv, k, dtype=torch.int32, device="cuda")
    cand, resc, count = (torch.zeros(b, hkv, dtype=torch.int32, device="cuda") for _ in range(3))
    for turn in range(20):
        base = torch.randn(b, hkv, n // run, 128, generator=g, device="cuda").repeat_interleave(run, 2)
        st.n = [0] * b
        st.quantize((base + 0.05 * torch.randn(base.shape, generator=g, device="cuda")).half())
        q = torch.randn(b, hkv, 128, generator=g, device="cuda").half()
        B.hca_score_topk(st.shape, st.kcache, q, st.n, k, idx, count, st.ws)
        B.hca_score_topk_report(st.shape, st.n, st.ws, cand, resc)
        st.score(q)
        assert (count == k).all() and (resc == 0).all() and (cand >= k).all(), f"turn {turn}: {resc.tolist()}"
        assert torch.equal(st.sel.gather(2, idx.long()).sort(dim=2).values, st.sel.topk(k, dim=2).values.sort(dim=2).values)


def test_running_monitor_over_several_calls(H):
    """hca_score_topk_monitor: calls counted, fewest / most pairs of a first scan and second scans per row, over
    three selections at different lengths (compared with the per-call report after each)."""
    from paper_2507_19823_amd import binding as B
    from paper_2507_19823_amd.session import LayerState
    w = S.Workload("mon", 93, 2, 8, 2, 60000, 4, 32, 512)
    d = S.make_layer(w, want_values=False)
    st = LayerState(w.batch, w.n_q_heads, w.n_kv_heads, w.n, w.bits, w.group, k_max=w.k, want_z=False)
    st.quantize(d["keys"].cuda())
    R = w.batch * w.n_kv_heads
    idx = torch.zeros(R, w.k, dtype=torch.int32, device="cuda")
    count = torch.zeros(R, dtype=torch.int32, device="cuda")
    cand = torch.zeros(R, dtype=torch.int32, device="cuda")
    resc = torch.zeros(R, dtype=torch.int32, device="cuda")
    mon = torch.full((R, 4), -7, dtype=torch.int32, device="cuda")
    B.hca_score_topk_monitor(st.shape, st.ws, None, True)
    seen = []
    for lens in ([60000, 700], [31000, 31000], [45000, 60000]):
        st.n = list(lens)
        B.hca_score_topk(st.shape, st.kcache, d["q"].cuda(), st.n, w.k, idx, count, st.ws)
        B.hca_score_topk_report(st.shape, st.n, st.ws, cand, resc)
        torch.cuda.synchronize()
        assert int(resc.sum()) == 0
        seen.append(cand.cpu().numpy().copy())
    B.hca_score_topk_monitor(st.shape, st.ws, mon, True)
    torch.cuda.synchronize()
    m, seen = mon.cpu().numpy(), np.stack(seen)
    assert np.all(m[:, 0] == 3) and np.all(m[:, 3] == 0)
    assert np.array_equal(m[:, 1], seen.min(0)) and np.array_equal(m[:, 2], seen.max(0))
    B.hca_score_topk_monitor(st.shape, st.ws, mon, False)       # after the reset above
    torch.cuda.synchronize()
    m = mon.cpu().numpy()
    assert np.all(m[:, 0] == 0) and np.all(m[:, 1] == 2**31 - 1) and np.all(m[:, 2] == 0) and np.all(m[:, 3] == 0)


@pytest.mark.parametrize("own_idx", [False, True])
def test_step_driver_pair_with_a_row_that_needs_the_second_scan(H, oracle, own_idx):
    """Two layers through hca_pipeline_step with paired scan launches: layer 0's keys mislead the sample (as in
    test_a_sample_that_misleads_still_gives_the_exact_set), layer 1's do not.  The paired fall-back launches
    (second scan of the failed row, second selection) must leave the oracle's index sets for both layers; the
    running monitor counts one second scan on layer 0's workspace and none on layer 1's."""
    import ctypes as C
    from paper_2507_19823_amd import binding as B
    n, k, tpb = 200000, 1024, 16
    w = S.Workload("mispair", 98, 1, 4, 1, n, 4, 32, k)
    R, cap, Lr = 1, n + 8, 2
    d = S.make_layer(w, want_values=False)
    q = d["q"].clone()
    q[0, 1:] = q[0, :1]
    g = torch.Generator().manual_seed(5)
    nblocks = (n + tpb - 1) // tpb
    Sn = min(nblocks, 8192 // tpb)
    sampled = torch.zeros(nblocks, dtype=torch.bool)
    sampled[(torch.arange(Sn, dtype=torch.int64) * nblocks) // Sn] = True
    sign = torch.where(sampled.repeat_interleave(tpb)[:n], 1.0, -1.0)[:, None]
    k0 = (sign * q[0, 0].float()[None, :] * (0.5 + torch.rand(n, 1, generator=g))
          + 0.05 * torch.randn(n, 128, generator=g)).to(torch.float16)[None, None]
    keys = [k0, d["keys"]]
    shape = B.make_shape(1, 4, 1, cap)
    dev = "cuda"
    kc = [torch.zeros(B.hca_kcache_bytes(shape), dtype=torch.uint8, device=dev) for _ in range(Lr)]
    acc = [torch.zeros(1, 1, cap, dtype=torch.float32, device=dev) for _ in range(Lr)]
    pos = [torch.arange(cap, dtype=torch.int32, device=dev).view(1, 1, cap).contiguous() for _ in range(Lr)]
    vals = torch.zeros(1, 1, 64, 128, dtype=torch.float16).pin_memory()          # every value row reads row < 64
    vd = torch.zeros(1, 1, 8, 128, dtype=torch.float16, device=dev)
    y = torch.zeros(Lr, 1, 4, 128, dtype=torch.float32, device=dev)
    ocs = []
    for l in range(Lr):
        B.hca_quantize_keys(shape, kc[l], keys[l].cuda(), n, [0])
        pos[l].zero_()                                                         # all slots share value row 0
        oc = oracle.Cache(R, cap, 128, 4, 32)
        oracle.quantize(oc, keys[l].numpy().reshape(R, n, 128))
        ocs.append(oc)
    streams = [torch.cuda.current_stream(), torch.cuda.Stream(), torch.cuda.Stream(), torch.cuda.Stream()]
    dsc = B.hca_pipeline_desc()
    dsc.stream_scan, dsc.stream_topk, dsc.stream_gather, dsc.stream_attend = (s_.cuda_stream for s_ in streams)
    wsb = B.hca_workspace_bytes(shape, k, 1)
    keep = []
    wsel = [torch.zeros(wsb, dtype=torch.uint8, device=dev) for _ in range(3)]
    for i in range(3):
        dsc.ws_select[i] = wsel[i].data_ptr()
    dsc.n_sel, dsc.fused_select, dsc.n_pipe, dsc.dual_scan = 3, 1, 4, 2
    sets = []
    for i in range(4):
        a = torch.full((1, 1, k), -3, dtype=torch.int32, device=dev)
        b_ = torch.zeros(1, 1, dtype=torch.int32, device=dev)
        c_ = torch.zeros(wsb, dtype=torch.uint8, device=dev)
        sets.append((a, b_, c_))
        dsc.idx[i], dsc.count[i], dsc.ws_attend[i] = a.data_ptr(), b_.data_ptr(), c_.data_ptr()
    wt = torch.zeros(wsb, dtype=torch.uint8, device=dev)
    dsc.ws_topk = wt.data_ptr()
    lidx = torch.full((Lr, k), -3, dtype=torch.int32, device=dev)
    lcnt = torch.zeros(Lr, 1, dtype=torch.int32, device=dev)
    if own_idx:
        dsc.layer_idx, dsc.layer_count, dsc.layer_idx_stride = lidx.data_ptr(), lcnt.data_ptr(), k
    pl = B.hca_pipeline_create(shape, Lr, dsc, 0)
    for i in range(2):
        B.hca_score_topk_monitor(shape, wsel[i], None, True)
    layers = (B.hca_layer * Lr)()
    k_new = torch.zeros(1, 1, 1, 128, dtype=torch.float16, device=dev)         # the appended token: a zero key
    qd = q.cuda()
    for l in range(Lr):
        layers[l].kcache, layers[l].acc, layers[l].pos = kc[l].data_ptr(), acc[l].data_ptr(), pos[l].data_ptr()
        layers[l].v_host, layers[l].v_hbm, layers[l].y = vals.data_ptr(), vd.data_ptr(), y[l].data_ptr()
        layers[l].k_new, layers[l].q = k_new.data_ptr(), qd.data_ptr()
    nres = (C.c_int64 * Lr)(n, n)
    torch.cuda.synchronize()
    B.hca_pipeline_step(pl, layers, nres, 0, k, 64, 64, 8, 0.0884, None, 0, -1)
    torch.cuda.synchronize()
    mon = torch.zeros(2, R, 4, dtype=torch.int32, device=dev)
    for i in range(2):
        B.hca_score_topk_monitor(shape, wsel[i], mon[i], False)
    torch.cuda.synchronize()
    for l in range(Lr):
        oracle.quantize(ocs[l], np.zeros((R, 1, 128), np.float16))
        sel, _ = oracle.score(ocs[l], q.numpy().reshape(-1, 128), want_z=False)
        oidx, ocount = oracle.topk(sel, ocs[l].n, k)
        gi = (lidx[l] if own_idx else sets[l][0].view(-1)).cpu().numpy()
        assert np.array_equal(gi, oidx[0]), f"layer {l}: index sets differ"
    m = mon.cpu().numpy()
    assert m[0, 0, 0] == 1 and m[0, 0, 3] == 1, "layer 0 should have needed the second scan"
    assert m[1, 0, 0] == 1 and m[1, 0, 3] == 0
    B.hca_pipeline_destroy(pl)


@pytest.mark.parametrize("dual", [0, 2])
@pytest.mark.parametrize("k", [60, 8000, 16384])
def test_step_driver_selects_at_the_edges_of_what_is_held_in_registers(
        H, oracle, k, dual, lens=(50000, 16384, 16383, 8192, 8191, 4096, 64, 63, 0)):
    """The step driver's own form of the selection (512 threads; 256 in the fixture's second form), on rows whose lists
    end at and beside the edges: one pair, a wave's worth, a step of registers, all 16384 and one more, and a long row."""
    import ctypes as C
    from paper_2507_19823_amd import binding as B
    lens = list(lens)
    n, nb, Lr = max(lens), len(lens), 2
    cap = n + 8
    w = S.Workload("held", 92, nb, 4, 1, n, 4, 32, k)
    dev = "cuda"
    d = S.make_layer(w, want_values=False)
    shape = B.make_shape(nb, 4, 1, cap)
    kc = [torch.zeros(B.hca_kcache_bytes(shape), dtype=torch.uint8, device=dev) for _ in range(Lr)]
    acc = [torch.zeros(nb, 1, cap, device=dev) for _ in range(Lr)]
    pos = [torch.zeros(nb, 1, cap, dtype=torch.int32, device=dev) for _ in range(Lr)]
    keys = [d["keys"], d["keys"].flip(2).contiguous()]
    ocs = []
    for l in range(Lr):
        B.hca_quantize_keys(shape, kc[l], keys[l].cuda(), n, [0] * nb)
        oc = oracle.Cache(nb, cap, 128, 4, 32)
        oracle.quantize(oc, keys[l].numpy().reshape(nb, n, 128))
        oc.n[...] = lens
        oracle.quantize(oc, np.zeros((nb, 1, 128), np.float16))                # the token that the step appends
        ocs.append(oc)
    streams = [torch.cuda.current_stream(), torch.cuda.Stream(), torch.cuda.Stream(), torch.cuda.Stream()]
    dsc = B.hca_pipeline_desc()
    dsc.stream_scan, dsc.stream_topk, dsc.stream_gather, dsc.stream_attend = (s_.cuda_stream for s_ in streams)
    wsb = B.hca_workspace_bytes(shape, k, 1)
    ws = [torch.zeros(wsb, dtype=torch.uint8, device=dev) for _ in range(8)]
    bufs = [(torch.zeros(nb, k, dtype=torch.int32, device=dev), torch.zeros(nb, dtype=torch.int32, device=dev))
            for _ in range(4)]
    dsc.n_sel, dsc.fused_select, dsc.n_pipe, dsc.dual_scan = 3, 1, 4, dual
    for i in range(3):
        dsc.ws_select[i] = ws[i].data_ptr()
    for i in range(4):
        dsc.idx[i], dsc.count[i], dsc.ws_attend[i] = bufs[i][0].data_ptr(), bufs[i][1].data_ptr(), ws[3 + i].data_ptr()
    dsc.ws_topk = ws[7].data_ptr()
    lidx = torch.full((Lr, nb, k), -3, dtype=torch.int32, device=dev)
    lcnt = torch.zeros(Lr, nb, dtype=torch.int32, device=dev)
    dsc.layer_idx, dsc.layer_count, dsc.layer_idx_stride = lidx.data_ptr(), lcnt.data_ptr(), nb * k
    pl = B.hca_pipeline_create(shape, Lr, dsc, 0)
    vd = torch.zeros(nb, 1, 8, 128, dtype=torch.float16, device=dev)           # every slot's value is row 0
    y = torch.zeros(Lr, nb, 4, 128, device=dev)
    k_new = torch.zeros(nb, 1, 1, 128, dtype=torch.float16, device=dev)
    qd = d["q"].cuda()
    layers = (B.hca_layer * Lr)()
    for l in range(Lr):
        layers[l].kcache, layers[l].acc, layers[l].pos = kc[l].data_ptr(), acc[l].data_ptr(), pos[l].data_ptr()
        layers[l].v_hbm, layers[l].y = vd.data_ptr(), y[l].data_ptr()
        layers[l].k_new, layers[l].q = k_new.data_ptr(), qd.data_ptr()
    nres = (C.c_int64 * (Lr * nb))(*(lens * Lr))
    torch.cuda.synchronize()
    B.hca_pipeline_step(pl, layers, nres, 0, k, 0, 0, 8, 0.0884, None, 0, -1)
    torch.cuda.synchronize()
    for l in range(Lr):
        sel, _ = oracle.score(ocs[l], d["q"].numpy().reshape(-1, 128), want_z=False)
        oidx, ocount = oracle.topk(sel, ocs[l].n, k)
        for r in range(nb):
            c = min(k, lens[r] + 1)
            assert lcnt[l, r].item() == c == ocount[r]
            assert np.array_equal(lidx[l, r, :c].cpu().numpy(), oidx[r, :c]), f"layer {l} row {r}: index sets differ"
    B.hca_pipeline_destroy(pl)


def _runs(n, kind):
    """Slots with large scores: the two ends of the row, three runs far apart, the last chunk's neighbourhood, or forty
    short runs - thousands of pairs in a few lists, with hundreds of empty ones before, between and after them."""
    large = torch.zeros(n, dtype=torch.bool)
    if kind == "ends":
        large[:n // 25] = large[-(n // 25):] = True
    elif kind == "three":
        for a in (n // 7, n // 2, n - n // 9):
            large[a:a + n // 33] = True
    elif kind == "last":
        large[-(n // 12):] = True
    else:
        for i in range(40):
            a = (i * n) // 40 + 37 * (i % 5)
            large[a:a + n // 500] = True
    return large


def _runs_layer(w, kind):
    d = S.make_layer(w, want_values=False)
    g = torch.Generator().manual_seed(w.n)
    q = d["q"].clone()
    q[:, 1:] = q[:, :1]                                       # four equal query heads
    size = torch.where(_runs(w.n, kind), 1.0, -1.0)[:, None] * (0.5 + torch.rand(w.n, 1, generator=g))
    keys = size * q[:, 0].float()[:, None, :] + 0.02 * torch.randn(w.batch, w.n, 128, generator=g)
    return dict(d, q=q, keys=keys.to(torch.float16)[:, None])


@pytest.mark.parametrize("kind", ["ends", "three", "last", "short"])
@pytest.mark.parametrize("n", [150000, 300000])
def test_pairs_in_a_few_lists_far_apart(H, oracle, n, kind):
    w = S.Workload("runs", 94, 2, 4, 1, n, 4, 32, 4000)
    d = _runs_layer(w, kind)
    _run(H, oracle, w, d["keys"], d["q"], [n, n - n // 3], w.k)


@pytest.mark.parametrize("kind", ["ends", "three", "short"])
@pytest.mark.parametrize("dual", [0, 2])
def test_step_driver_with_pairs_in_a_few_lists_far_apart(H, oracle, monkeypatch, dual, kind):
    """The step driver's forms on such rows (its 512-thread form holds 128 groups of positions per wave)."""
    make = S.make_layer

    def clustered(w, want_values=True):
        monkeypatch.setattr(S, "make_layer", make)
        return _runs_layer(w, kind)

    monkeypatch.setattr(S, "make_layer", clustered)
    test_step_driver_selects_at_the_edges_of_what_is_held_in_registers(H, oracle, 3000, dual)


@pytest.mark.parametrize("dual", [0, 2])
@pytest.mark.parametrize("tied,k", [(70000, 777), (20000, 3000), (17000, 16384)])
def test_step_driver_with_ties_in_lists_too_long_for_the_registers(H, oracle, monkeypatch, dual, tied, k):
    make = S.make_layer

    def ties(w, want_values=True):
        monkeypatch.setattr(S, "make_layer", make)
        return _tied_layer(w, tied)

    monkeypatch.setattr(S, "make_layer", ties)
    test_step_driver_selects_at_the_edges_of_what_is_held_in_registers(H, oracle, k, dual, (90000, 71000, 16385, 0))


@pytest.mark.parametrize("dual", [0, 2])
def test_step_driver_with_the_1024_thread_form(H, oracle, dual):
    """select_wg = 1024 in a step driver, which takes 512 threads by itself: single layers and pairs of them."""
    H.hca_tune("select_wg", 1024)
    test_step_driver_selects_at_the_edges_of_what_is_held_in_registers(H, oracle, 8000, dual)
