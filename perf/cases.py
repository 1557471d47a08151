"""Workloads whose speed is measured: what a program that decodes with this library asks of it.

A case is one call sequence of the public interface at one size.  The kinds:

  step      one decode step of one layer through LayerState: append the new key, score all resident keys and
            select the top k in one call, softmax and weighted sum over the selected values
  select    the selection of one layer alone (hca_score_topk), for the long contexts
  paper     the paper's own selection and weights: scan with the softmax denominator, the cumulative-weight
            rule, weighted sum with the un-renormalised weights
  stack     one decode step over several layers through the step driver, in the form the benchmark times: two
            layers per scan, values in pinned host memory, most of them summed by host threads
  quantize  key compression of one block at the end of a prefill block
  evict     accumulated-score eviction of one layer
  vqstep    one decode step of one layer with the codebook key format
  vqassign  nearest-centroid assignment of one prefill block

Shapes are the synthetic workloads' (1 head at 4 Ki tokens; 32 query heads over 8 KV heads at 32 Ki, 4 x 128 Ki,
1 Mi, 2-bit codes at 2 Mi resident) and sizes between and around them; keys carry 4 outlier channels per KV head,
every query has planted tokens that share its direction.
"""
import ctypes
import math
import weakref

import torch

import paper_2507_19823_amd as H
from paper_2507_19823_amd import binding as B
from paper_2507_19823_amd.session import LayerState

D = 128
SM = 1.0 / math.sqrt(D)
PLANTED = 16            # tokens per query head that share its direction
NEW_ROWS = 64           # rows of the HBM slice that holds the values of appended tokens


def listed():
    return [
        # one head, 4 Ki tokens, values in host memory: nothing but launches and latency
        dict(name="step-4k-one-head", kind="step", batch=1, hq=1, hkv=1, n=4096, bits=4, k=256, values="host"),
        # short context of a Llama-3-8B layer, half the values in HBM
        dict(name="step-32k", kind="step", batch=1, hq=32, hkv=8, n=32768, bits=4, k=1024, values="half"),
        # four sequences of different lengths served together, values kept in HBM
        dict(name="step-128k-b4", kind="step", batch=4, hq=32, hkv=8, n=131072, bits=4, k=2048, values="hbm"),
        # the longest resident set of one layer: half of a 4 Mi context, 2-bit codes
        dict(name="select-2m-2bit", kind="select", batch=1, hq=32, hkv=8, n=2097152, bits=2, k=8192),
        # the paper's Eq. 4 and Eq. 5 at a length that is no multiple of anything
        dict(name="paper-500k", kind="paper", batch=1, hq=32, hkv=8, n=500003, bits=4, k=8192, tau=0.9),
        # the benchmark's form of a decode step, four layers of its thirty-two
        dict(name="stack-4x1m", kind="stack", batch=1, hq=32, hkv=8, n=1048576, bits=4, k=4096, layers=4),
        # one prefill block of 64 Ki tokens appended behind an uneven number of resident ones
        dict(name="quantize-64k", kind="quantize", batch=1, hkv=8, n0=4099, T=65536, bits=4),
        # a cache brought down to half its length
        dict(name="evict-512k-half", kind="evict", batch=1, hkv=8, n=524288, M=262144, protect=16, bits=4, hit=0.1,
             place="spare"),
        # codebook keys, one byte per group: decode step, values in HBM
        dict(name="vqstep-1m-c256", kind="vqstep", batch=1, hq=32, hkv=8, n=1048576, g=32, c=256, k=4096, tau=0.0),
        # the paper's codebook size, two bytes per group, its cumulative-weight selection
        dict(name="vqstep-300k-c8192", kind="vqstep", batch=1, hq=32, hkv=8, n=300001, g=32, c=8192, k=4096, tau=0.9),
        # prefill block into the small and into the paper's codebook
        dict(name="vqassign-64k-c256", kind="vqassign", batch=1, hkv=8, n0=1003, T=65536, g=32, c=256),
        dict(name="vqassign-16k-c8192", kind="vqassign", batch=1, hkv=8, n0=1003, T=16384, g=32, c=8192),
    ]


def _log(rng, lo, hi):
    """A size whose logarithm is uniform between those of lo and hi; mostly no round number."""
    v = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    return v if rng.random() < 0.7 else max(lo, v // 64 * 64)


def draw(rng):
    kind = rng.choice(["step", "step", "step", "select", "select", "paper", "stack", "quantize", "evict", "vqstep",
                       "vqstep", "vqassign", "vqassign"])
    batch = rng.choice([1, 1, 2, 3, 4, 7])
    hq, hkv = rng.choice([(32, 8), (32, 8), (16, 8), (8, 8), (4, 1), (1, 1), (14, 7)])
    rows = batch * hkv
    if kind == "step":
        n = min(_log(rng, 1000, 300000), 4194304 // rows)
        return dict(kind=kind, batch=batch, hq=hq, hkv=hkv, n=n, bits=rng.choice([4, 4, 2]), k=min(n, _log(rng, 64, 2048)),
                    values=rng.choice(["host", "half", "hbm"]))
    if kind == "select":
        n = min(_log(rng, 60000, 2097152), 8388608 // rows)
        return dict(kind=kind, batch=batch, hq=hq, hkv=hkv, n=n, bits=rng.choice([4, 2]), k=min(n, _log(rng, 256, 8192)))
    if kind == "paper":
        n = min(_log(rng, 2000, 600000), 4194304 // rows)
        return dict(kind=kind, batch=batch, hq=hq, hkv=hkv, n=n, bits=rng.choice([4, 2]), k=min(n, _log(rng, 256, 8192)),
                    tau=rng.choice([0.5, 0.7, 0.9, 0.95]))
    if kind == "stack":
        return dict(kind=kind, batch=1, hq=32, hkv=8, n=_log(rng, 131072, 1048576), bits=rng.choice([4, 4, 2]),
                    k=256 * rng.randint(8, 16), layers=rng.randint(2, 4))
    if kind == "quantize":
        return dict(kind=kind, batch=batch, hkv=hkv, n0=rng.randint(0, 9000), T=min(_log(rng, 1, 100000), 800000 // rows + 1),
                    bits=rng.choice([4, 2]))
    if kind == "evict":
        n = min(_log(rng, 4000, 524288), 4194304 // rows)
        M = max(1, int(n * rng.choice([0.5, 0.75, 0.99])))
        return dict(kind=kind, batch=batch, hkv=hkv, n=n, M=M, protect=min(M, rng.choice([0, 16, 64])),
                    bits=rng.choice([4, 2]), hit=rng.choice([0.02, 0.1, 0.6]), place=rng.choice(["spare", "same"]))
    g = rng.choice([32, 32, 64])
    c = rng.choice([64, 128, 256, 256, 1024, 4096, 8192])
    if kind == "vqstep":
        n = min(_log(rng, 4000, 1048576), (4194304 if c <= 256 else 2097152) // rows)
        return dict(kind=kind, batch=batch, hq=hq, hkv=hkv, n=n, g=g, c=c, k=min(n, _log(rng, 256, 4096)),
                    tau=rng.choice([0.0, 0.0, 0.9]))
    T = min(_log(rng, 1000, 65536), (1 << 30) * 2 // (rows * g * c) + 1, 500000 // rows)
    return dict(kind=kind, batch=batch, hkv=hkv, n0=rng.randint(0, 9000), T=T, g=g, c=c)


# ---- inputs -------------------------------------------------------------------------------------

def _gen(seed, tag):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 64 + tag)
    return g


def _lens(c):
    """Resident tokens per sequence before the step: the first sequence is the longest."""
    return [max(1, c["n"] - b * (c["n"] // 7) // max(1, c["batch"] - 1) - 13 * b) for b in range(c["batch"])]


def _outliers(c, seed):
    """fp32 [batch, hkv, D]: 8 on four channels of every KV head, else 1."""
    u = torch.rand(c["batch"], c["hkv"], D, generator=_gen(seed, 0), device="cuda")
    m = torch.ones_like(u)
    return m.scatter_(2, u.topk(4, dim=2).indices, 8.0)


def _randn16(shape, gen):
    out = torch.empty(shape, dtype=torch.float16, device="cuda")
    flat = out.view(-1, D)
    for r in range(0, flat.shape[0], 1 << 20):
        part = flat[r:r + (1 << 20)]
        part.copy_(torch.randn(part.shape, generator=gen, device="cuda"))
    return out


def _keys(c, T, seed, tag=1):
    """fp16 [batch, hkv, T, D]."""
    k = _randn16((c["batch"], c["hkv"], T, D), _gen(seed, tag))
    m = _outliers(c, seed).to(torch.float16)
    for b in range(c["batch"]):
        for h in range(c["hkv"]):
            k[b, h] *= m[b, h]
    return k


def _keys_queries(c, seed, layer=0):
    """Resident keys with planted tokens, the step's new key and the queries: fp16 [B,Hkv,n,D], [B,Hkv,1,D], [B,Hq,D]."""
    seed = seed * 16 + layer
    G = c["hq"] // c["hkv"]
    keys = _keys(c, c["n"], seed)
    new = _keys(c, 1, seed, 2)
    g = _gen(seed, 3)
    m = _outliers(c, seed).repeat_interleave(G, dim=1)
    u = (torch.randn(c["batch"], c["hq"], D, generator=g, device="cuda") * m).to(torch.float16)
    q = u.float() + 0.3 * torch.randn(u.shape, generator=g, device="cuda")
    if c["kind"] == "paper":
        # flatter weights, so that the cumulative rule keeps thousands of tokens; the planted ones stay in the set
        q = 0.3 * torch.randn(u.shape, generator=g, device="cuda") * m
    q = q.to(torch.float16)
    each = max(1, min(PLANTED, c["n"] // (2 * G)))
    lens = _lens(c)
    for b in range(c["batch"]):
        for h in range(c["hkv"]):
            if lens[b] < each * G or c["kind"] == "paper":
                continue
            at = torch.randperm(lens[b], generator=g, device="cuda")[:each * G]
            keys[b, h, at] = u[b, h * G:(h + 1) * G].repeat_interleave(each, dim=0)
    return keys, new, q


def _values(c, seed, rows):
    return _randn16((c["batch"], c["hkv"], rows, D), _gen(seed, 4))


def _pinned(v):
    out = torch.empty(v.shape, dtype=v.dtype, pin_memory=True)
    out.copy_(v)
    return out


def _codebook(c, seed):
    """fp32 [hkv, g, c, D/g]: centroids spread like the sub-vectors they stand for."""
    dbar = D // c["g"]
    m = _outliers(c, seed)[0].view(c["hkv"], c["g"], 1, dbar)
    return (torch.randn(c["hkv"], c["g"], c["c"], dbar, generator=_gen(seed, 5), device="cuda") * m).contiguous()


class _State:
    """Names what a program holds between calls."""


def _prepare_step(c, seed):
    s = _State()
    keys, s.new, s.q = _keys_queries(c, seed)
    s.lens = _lens(c)
    s.layer = LayerState(c["batch"], c["hq"], c["hkv"], c["n"] + NEW_ROWS, c["bits"], 32 if c["bits"] == 4 else 64,
                         k_max=c["k"], m_max=1)
    s.layer.kcache.zero_()
    s.layer.quantize(keys, [0] * c["batch"])
    del keys
    s.layer.n = list(s.lens)
    if c["kind"] == "step":
        n = c["n"]
        s.n_host = {"host": n, "half": n // 2, "hbm": 0}[c["values"]]
        v = _values(c, seed, n + NEW_ROWS)
        s.v_host = _pinned(v[:, :, :s.n_host]) if s.n_host else None
        s.v_hbm = v[:, :, s.n_host:].contiguous()
    return s


def _run_step(c, s):
    L = s.layer
    L.n = list(s.lens)
    L.quantize(s.new, s.lens)
    L.score_topk(s.q, c["k"])
    L.attend(s.q, s.v_host, s.n_host, s.v_hbm)
    return {"y": L.y, "acc": L.acc, "idx": L.idx, "count": L.count}


def _run_select(c, s):
    s.layer.score_topk(s.q, c["k"])
    return {"idx": s.layer.idx, "count": s.layer.count}


def _prepare_paper(c, seed):
    s = _prepare_step(c, seed)
    s.v = _values(c, seed, c["n"])
    s.layer.sel.zero_()
    s.lse = torch.zeros(c["batch"], c["hq"], device="cuda")
    s.mass = torch.zeros(c["batch"], c["hkv"], 2, dtype=torch.int64, device="cuda")
    return s


def _run_paper(c, s):
    L = s.layer
    B.hca_score_qkeys_lse(L.shape, L.kcache, s.q, s.lens, SM, L.sel, s.lse, L.ws)
    B.hca_topp(L.shape, L.sel, s.lens, SM, c["tau"], c["k"], L.idx, L.count, s.mass, L.ws)
    B.hca_gather_values(L.shape, L.idx, L.count, c["k"], L.pos, None, 0, 0, s.v, c["n"], L.ws)
    B.hca_attend_gathered_global(L.shape, L.kcache, s.q, L.idx, L.count, c["k"], SM, s.lse, L.y, L.acc, L.ws)
    return {"sel": L.sel, "lse": s.lse, "mass": s.mass, "idx": L.idx, "count": L.count, "y": L.y, "acc": L.acc}


_streams = []
_drivers = weakref.WeakValueDictionary()       # a program has one step driver (and its host threads) for all sequences


class _Driver:
    def __init__(self, c):
        if not _streams:               # scan on the current stream, the other three stages on one stream each
            _streams.extend(torch.cuda.Stream() for _ in range(3))
        n, k, hkv, nl = c["n"], c["k"], c["hkv"], c["layers"]
        self.shape = B.make_shape(1, c["hq"], hkv, n + NEW_ROWS, c["bits"], 32 if c["bits"] == 4 else 64)
        self.keep = []
        self.idx = self.buffer((nl, hkv, k), torch.int32)
        self.count = self.buffer((nl, hkv), torch.int32)
        d = B.hca_pipeline_desc()
        d.stream_scan, d.stream_topk, d.stream_gather, d.stream_attend = [
            x.cuda_stream for x in [torch.cuda.current_stream()] + _streams]
        wsb = B.hca_workspace_bytes(self.shape, k, 1)
        d.fused_select, d.n_sel = 1, max(nl, 6)
        for i in range(d.n_sel):
            d.ws_select[i] = self.buffer(wsb).data_ptr()
        d.n_pipe = 8
        for i in range(d.n_pipe):
            d.idx[i] = self.buffer((hkv, k), torch.int32).data_ptr()
            d.count[i] = self.buffer((hkv,), torch.int32).data_ptr()
            d.ws_attend[i] = self.buffer(wsb).data_ptr()
        d.ws_topk = self.buffer(wsb).data_ptr()
        d.dual_scan = 2
        d.host_chunks, d.host_threads, d.gather_wgs = 14 * (k // 256) // 16, 14, 4
        d.layer_idx, d.layer_count, d.layer_idx_stride = self.idx.data_ptr(), self.count.data_ptr(), hkv * k
        torch.cuda.synchronize()
        self.handle = B.hca_pipeline_create(self.shape, nl, d, 0)

    def buffer(self, shape, dtype=torch.uint8):
        self.keep.append(torch.zeros(shape, dtype=dtype, device="cuda"))
        return self.keep[-1]

    def __del__(self):
        if getattr(self, "handle", None):
            torch.cuda.synchronize()
            B.hca_pipeline_destroy(self.handle)


def _prepare_stack(c, seed):
    s = _State()
    n, k, hkv, nl = c["n"], c["k"], c["hkv"], c["layers"]
    key = (n, k, hkv, c["hq"], c["bits"], nl)
    s.driver = _drivers.get(key) or _Driver(c)
    _drivers[key] = s.driver
    s.shape, s.keep = s.driver.shape, []
    s.v_host = torch.empty(1, hkv, n, D, dtype=torch.float16, pin_memory=True)     # one store serves every layer
    s.v_host.copy_(_values(c, seed, n))
    B.hca_host_prefault(s.v_host, 16)
    s.y = torch.zeros(nl, c["hq"], D, device="cuda")
    s.acc = []
    s.layers = (B.hca_layer * nl)()
    for l in range(nl):
        keys, new, q = _keys_queries(c, seed, l)
        kc = torch.zeros(B.hca_kcache_bytes(s.shape), dtype=torch.uint8, device="cuda")
        acc, pos = _slot_arrays(c, n + NEW_ROWS)
        B.hca_quantize_keys(s.shape, kc, keys, n, [0], acc, pos, [0])
        del keys
        hbm = _randn16((1, hkv, NEW_ROWS, D), _gen(seed * 16 + l, 6))
        s.keep += [kc, pos, new, q, hbm]
        s.acc.append(acc)
        ly = s.layers[l]
        ly.kcache, ly.acc, ly.pos = kc.data_ptr(), acc.data_ptr(), pos.data_ptr()
        ly.k_new, ly.q, ly.y = new.data_ptr(), q.data_ptr(), s.y[l].data_ptr()
        ly.v_host, ly.v_hbm = s.v_host.data_ptr(), hbm.data_ptr()
    s.nres = (ctypes.c_int64 * nl)()
    return s


def _run_stack(c, s):
    for l in range(c["layers"]):
        s.nres[l] = c["n"]
    B.hca_pipeline_step(s.driver.handle, s.layers, s.nres, c["n"], c["k"], c["n"], c["n"], NEW_ROWS, SM)
    return {"y": s.y, "idx": s.driver.idx, "count": s.driver.count, "acc": s.acc}


def _slot_arrays(c, cap):
    return (torch.zeros(c["batch"], c["hkv"], cap, device="cuda"),
            torch.zeros(c["batch"], c["hkv"], cap, dtype=torch.int32, device="cuda"))


def _prepare_quantize(c, seed):
    s = _State()
    s.shape = B.make_shape(c["batch"], c["hkv"], c["hkv"], c["n0"] + c["T"] + 5, c["bits"], 32 if c["bits"] == 4 else 64)
    s.kcache = torch.zeros(B.hca_kcache_bytes(s.shape), dtype=torch.uint8, device="cuda")
    s.acc, s.pos = _slot_arrays(c, c["n0"] + c["T"] + 5)
    s.at = [max(0, c["n0"] - 37 * b) for b in range(c["batch"])]
    if c["n0"]:
        B.hca_quantize_keys(s.shape, s.kcache, _keys(c, c["n0"], seed, 7), c["n0"], [0] * c["batch"], s.acc, s.pos,
                            [0] * c["batch"])
    s.keys = _keys(c, c["T"], seed)
    return s


def _run_quantize(c, s):
    B.hca_quantize_keys(s.shape, s.kcache, s.keys, c["T"], s.at, s.acc, s.pos, s.at)
    return {"kcache": s.kcache, "acc": s.acc, "pos": s.pos}


def _prepare_evict(c, seed):
    s = _State()
    s.layer = LayerState(c["batch"], c["hkv"], c["hkv"], c["n"], c["bits"], 32 if c["bits"] == 4 else 64, k_max=1,
                         m_max=c["M"])
    L = s.layer
    L.kcache.zero_()
    L.quantize(_keys(c, c["n"], seed), [0] * c["batch"])
    s.lens = _lens(c)
    g = _gen(seed, 8)
    w = torch.rand(L.acc.shape, generator=g, device="cuda")
    u = torch.rand(L.acc.shape, generator=g, device="cuda")
    L.acc.copy_(torch.where(u < c["hit"], w.pow(8), torch.zeros_like(w)))    # few tokens carry most of the weight
    s.kept = torch.full((c["batch"], c["hkv"], c["M"]), -1, dtype=torch.int32, device="cuda")
    if c["place"] == "spare":
        s.dst = (torch.zeros_like(L.kcache), torch.zeros_like(L.acc), torch.zeros_like(L.pos))
    else:
        s.dst = (None, None, None)
    return s


def _run_evict(c, s):
    L = s.layer
    B.hca_evict(L.shape, L.kcache, L.acc, L.pos, s.lens, c["M"], c["protect"], s.kept, L.ws, *s.dst)
    if c["place"] == "spare":
        return {"kcache": s.dst[0], "acc": s.dst[1], "pos": s.dst[2], "kept": s.kept}
    return {"kcache": L.kcache, "acc": L.acc, "pos": L.pos, "kept": s.kept}


def _prepare_vqstep(c, seed):
    s = _State()
    keys, s.new, s.q = _keys_queries(c, seed)
    cap = c["n"] + NEW_ROWS
    s.shape = B.make_shape(c["batch"], c["hq"], c["hkv"], cap)
    s.cen = _codebook(c, seed * 16)
    s.cb = B.make_codebook(c["g"], c["c"], s.cen)
    s.pcache = torch.zeros(B.hca_vq_pcache_bytes(s.shape, s.cb), dtype=torch.uint8, device="cuda")
    s.acc, s.pos = _slot_arrays(c, cap)
    B.hca_vq_assign(s.shape, s.cb, s.pcache, keys, c["n"], [0] * c["batch"], s.acc, s.pos, [0] * c["batch"])
    del keys
    s.lens = _lens(c)
    s.now = [x + 1 for x in s.lens]
    s.lut = torch.zeros(B.hca_vq_lut_bytes(s.shape, s.cb) // 4, device="cuda")
    s.sel = torch.zeros(c["batch"], c["hkv"], cap, device="cuda")
    s.idx = torch.full((c["batch"], c["hkv"], c["k"]), -1, dtype=torch.int32, device="cuda")
    s.count = torch.zeros(c["batch"], c["hkv"], dtype=torch.int32, device="cuda")
    s.y = torch.zeros(c["batch"], c["hq"], D, device="cuda")
    s.v = _values(c, seed, cap)
    s.ws = torch.empty(B.hca_vq_workspace_bytes(s.shape, s.cb, c["k"]), dtype=torch.uint8, device="cuda")
    return s


def _run_vqstep(c, s):
    k = c["k"]
    B.hca_vq_assign(s.shape, s.cb, s.pcache, s.new, 1, s.lens, s.acc, s.pos, s.lens)
    B.hca_vq_score(s.shape, s.cb, s.pcache, s.q, s.now, s.lut, s.sel)
    if c["tau"]:
        B.hca_topp(s.shape, s.sel, s.now, SM, c["tau"], k, s.idx, s.count, None, s.ws)
    else:
        B.hca_topk(s.shape, s.sel, s.now, k, s.idx, s.count, s.ws)
    B.hca_gather_values(s.shape, s.idx, s.count, k, s.pos, None, 0, 0, s.v, s.v.shape[2], s.ws)
    B.hca_vq_attend_gathered(s.shape, s.cb, s.pcache, s.lut, s.idx, s.count, k, SM, s.y, s.acc, s.ws)
    return {"sel": s.sel, "idx": s.idx, "count": s.count, "y": s.y, "acc": s.acc}


def _prepare_vqassign(c, seed):
    s = _State()
    cap = c["n0"] + c["T"] + 5
    s.shape = B.make_shape(c["batch"], c["hkv"], c["hkv"], cap)
    s.cen = _codebook(c, seed)
    s.cb = B.make_codebook(c["g"], c["c"], s.cen)
    s.pcache = torch.zeros(B.hca_vq_pcache_bytes(s.shape, s.cb), dtype=torch.uint8, device="cuda")
    s.acc, s.pos = _slot_arrays(c, cap)
    s.at = [max(0, c["n0"] - 37 * b) for b in range(c["batch"])]
    s.keys = _keys(c, c["T"], seed)
    return s


def _run_vqassign(c, s):
    B.hca_vq_assign(s.shape, s.cb, s.pcache, s.keys, c["T"], s.at, s.acc, s.pos, s.at)
    return {"pcache": s.pcache, "acc": s.acc, "pos": s.pos}


_PREPARE = {"step": _prepare_step, "select": _prepare_step, "paper": _prepare_paper, "stack": _prepare_stack,
            "quantize": _prepare_quantize, "evict": _prepare_evict, "vqstep": _prepare_vqstep,
            "vqassign": _prepare_vqassign}
_RUN = {"step": _run_step, "select": _run_select, "paper": _run_paper, "stack": _run_stack, "quantize": _run_quantize,
        "evict": _run_evict, "vqstep": _run_vqstep, "vqassign": _run_vqassign}


def prepare(case, seed):
    H.lib()
    s = _PREPARE[case["kind"]](case, seed)
    s.case = case
    torch.cuda.synchronize()
    return s


def run(state):
    return _RUN[state.case["kind"]](state.case, state)


# ---- what a pass cannot do without, and how exact its results are ------------------------------------------

def work(case):
    c, kind = case, case["kind"]
    hkv, batch = c["hkv"], c["batch"]
    if kind in ("quantize", "vqassign"):
        keys = batch * hkv * c["T"]
        if kind == "quantize":
            return {"bytes": keys * (256 + D * c["bits"] // 8 + 4 * D // (32 if c["bits"] == 4 else 64) + 8),
                    "flops": keys * D * 4}
        wide = c["c"] > 256
        return {"bytes": keys * (256 + c["g"] * (2 if wide else 1) + 8) + hkv * D * c["c"] * 4,
                "flops": keys * D * c["c"] * 2}
    if kind == "evict":
        rows = sum(hkv * x for x in _lens(c))
        slot = D * c["bits"] // 8 + 4 * D // (32 if c["bits"] == 4 else 64) + 8
        moved = sum(hkv * min(x, c["M"]) for x in _lens(c))
        return {"bytes": rows * 4 + moved * (2 * slot + 4), "flops": rows}
    G = c["hq"] // hkv
    layers = c.get("layers", 1)
    tokens = layers * sum(hkv * x for x in _lens(c))
    picked = layers * sum(hkv * min(c["k"], x) for x in _lens(c))
    if kind == "vqstep":
        per = c["g"] * (2 if c["c"] * c["g"] * G > 32768 or c["c"] > 256 else 1) + 4
        return {"bytes": tokens * per + hkv * D * c["c"] * 4 + picked * 260, "flops": tokens * c["g"] * G}
    per = D * c["bits"] // 8 + 4 * D // (32 if c["bits"] == 4 else 64) + (4 if kind == "paper" else 0)
    values = 0 if kind == "select" else picked * 260
    return {"bytes": tokens * per + values + picked * 4, "flops": tokens * D * 2 * G}


def tolerance(case):
    if case["kind"] in ("quantize", "evict", "vqassign", "select"):
        return "exact"
    # sums in fp32, whole numbers are the same whatever the order of the additions
    return {"rel": 1e-5, "max": 1e-3}


# ---- the same in 64 bits -----------------------------------------------------------------------------------

def _dequantised(x, bits):
    """fp64 [n, D]: the keys after compression, from their definition."""
    group, top = (32, 15) if bits == 4 else (64, 3)
    x = x.float().view(-1, D // group, group)
    lo, hi = x.amin(2, keepdim=True), x.amax(2, keepdim=True)
    scale = ((hi - lo).double() / top).float().to(torch.float16).float()     # in 64 bits: the correctly rounded quotient
    scale = torch.where(scale == 0, torch.ones_like(scale), scale)
    code = ((x - lo) * (1.0 / scale.double()).float()).round().clamp(0, top)
    return (scale.double() * code.double() + lo.double()).view(-1, D)


def _fixed(q):
    """fp64 [heads, D]: the queries on their 15-bit grids."""
    q = q.cpu().double()                             # powers of two are exact there, and half-way cases stay half-way
    s = 13 - torch.floor(torch.log2(q.abs().amax(1, keepdim=True)))
    return (torch.round(q * 2.0 ** s) * 2.0 ** -s).cuda()


def _scores(keys, q, bits):
    """fp64 [n, heads]."""
    out = torch.empty(keys.shape[0], q.shape[0], dtype=torch.float64, device="cuda")
    qt = _fixed(q).t().contiguous()
    for r in range(0, keys.shape[0], 1 << 17):
        out[r:r + (1 << 17)] = _dequantised(keys[r:r + (1 << 17)], bits) @ qt
    return out


def _vq_scores(keys, q, cen):
    """fp64 [n, heads]: Eq. 3 for one KV head."""
    n, g = keys.shape[0], cen.shape[0]
    out = torch.zeros(n, q.shape[0], dtype=torch.float64, device="cuda")
    dbar = D // g
    number = torch.arange(cen.shape[1], device="cuda")
    for i in range(g):
        x, cc = keys[:, i * dbar:(i + 1) * dbar].float(), cen[i]
        table = cc.double() @ q[:, i * dbar:(i + 1) * dbar].double().t().contiguous()
        for r in range(0, n, 1 << 17):
            d = torch.zeros(min(1 << 17, n - r), cen.shape[1], device="cuda")
            for ch in range(dbar):                   # the distance's own roundings decide which index a token has
                e = (x[r:r + (1 << 17), ch, None] - cc[:, ch]).double()
                d = (e * e + d).float()
            near = ((d.view(torch.int32).long() << 13) | number).amin(1) & 8191     # ties to the lowest index
            out[r:r + (1 << 17)] += table[near]
    return out


def _weighted(z, at, V, all_tokens):
    """(y [heads, D], weights [picked, heads]) over the slots `at`."""
    l = z * SM
    a = torch.softmax(l, 0)[at] if all_tokens else torch.softmax(l[at], 0)
    return a.t().contiguous() @ V[at].double(), a


def _prefix(sel, tau, k):
    """The slots that the cumulative rule keeps."""
    w, order = torch.sort(torch.softmax(sel * SM, 0), descending=True, stable=True)
    need = int((torch.cumsum(w, 0) < tau).sum()) + 1
    return order[:min(need, k, sel.numel())].sort().values


def _exact_layer(c, seed, layer, V):
    B_, G, lens = c["batch"], c["hq"] // c["hkv"], _lens(c)
    cap = c["n"] + NEW_ROWS
    keys, new, q = _keys_queries(c, seed, layer)
    y = torch.zeros(B_, c["hq"], D, dtype=torch.float64, device="cuda")
    acc = torch.zeros(B_, c["hkv"], cap, dtype=torch.float64, device="cuda")
    sel = torch.zeros(B_, c["hkv"], cap, dtype=torch.float64, device="cuda")
    lse = torch.zeros(B_, c["hq"], dtype=torch.float64, device="cuda")
    cen = _codebook(c, seed * 16) if c["kind"] == "vqstep" else None
    for b in range(B_):
        for h in range(c["hkv"]):
            x = keys[b, h, :lens[b]]
            if c["kind"] != "paper":
                x = torch.cat([x, new[b, h]])
            heads = q[b, h * G:(h + 1) * G]
            z = _scores(x, heads, c["bits"]) if cen is None else _vq_scores(x, heads, cen[h])
            top = z.amax(1)
            sel[b, h, :top.numel()] = top
            lse[b, h * G:(h + 1) * G] = torch.logsumexp(z * SM, 0)
            if c.get("tau"):
                at = _prefix(top, c["tau"], c["k"])
            else:
                at = torch.sort(top, descending=True, stable=True).indices[:c["k"]].sort().values
            yy, a = _weighted(z, at, V(b, h), c["kind"] == "paper")
            y[b, h * G:(h + 1) * G] = yy
            acc[b, h, at] = a.clamp_min(1e-30).sum(1)
    return {"y": y, "acc": acc, "sel": sel, "lse": lse}


def exact(case, seed):
    c, kind = case, case["kind"]
    if kind in ("quantize", "evict", "vqassign", "select"):
        return None                                  # bytes and whole numbers only
    if kind == "vqstep" and sum(_lens(c)) * c["hkv"] * c["g"] * c["c"] > 2e11:
        return None
    if kind == "stack":
        V = _values(c, seed, c["n"])[0]
        out = []
        for l in range(c["layers"]):
            new = _randn16((1, c["hkv"], NEW_ROWS, D), _gen(seed * 16 + l, 6))[0]
            out.append(_exact_layer(c, seed, l, lambda b, h: torch.cat([V[h], new[h]])))
        return {"y": torch.cat([o["y"] for o in out]), "idx": None, "count": None, "acc": [o["acc"] for o in out]}
    rows = c["n"] + (0 if kind == "paper" else NEW_ROWS)
    V = _values(c, seed, rows)
    e = _exact_layer(c, seed, 0, lambda b, h: V[b, h])
    if kind == "step":
        return {"y": e["y"], "acc": e["acc"], "idx": None, "count": None}
    if kind == "vqstep":
        return {"sel": e["sel"], "idx": None, "count": None, "y": e["y"], "acc": e["acc"]}
    return {"sel": e["sel"], "lse": e["lse"], "mass": None, "idx": None, "count": None, "y": e["y"], "acc": e["acc"]}
