"""The sizes, placements and shapes where a launch rule changes from one form of a kernel to another: the forms must
agree bit for bit with each other or with the oracle on both sides of the line."""
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
    out = []
    for n_host in (1200, 0, 600, 1150, 1):                # 1150: the HBM slice is short, 1: nearly nothing on the host
        vh = values[:, :, :n_host].contiguous().pin_memory() if n_host else None
        vd = values[:, :, n_host:].contiguous().cuda() if n_host < 1200 else None
        st.y.fill_(-1.0)
        st.attend(q, vh, n_host, vd, use_acc=False)
        torch.cuda.synchronize()
        out.append(st.y.clone())
    assert torch.isfinite(out[0]).all()
    for n_host, y in zip((0, 600, 1150, 1), out[1:]):
        assert torch.equal(y, out[0]), f"n_host_rows = {n_host}"
