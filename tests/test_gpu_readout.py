"""GPU: the readout kernels at the edges of their tiles and row blocks, against
the oracle's float64 attention.  Each test prints its case before any GPU step.
"""
import numpy as np
import pytest

from paper_2606_26762_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_26762_amd import protokv as pk
    pk.lib()
    yield


def H():
    from tests import gpu_harness
    return gpu_harness


def _stream(h, wl, **pkw):
    pair = h.Pair(wl, **pkw)
    for _ in range(wl.frames):
        pair.step()
    return pair


# rows per kv head 1, 31, 33 and 224 (32 per wave, the last wave nearly empty in
# the third); contexts of 70 keys (no bank yet) and of 105 + 37 S (32 per tile:
# last tiles of 6, 13, 24 and 14 keys, the near / pseudo boundary inside a tile)
@pytest.mark.parametrize("grp,tq,S,frames", [(1, 31, 8, 2), (1, 1, 8, 12), (3, 11, 3, 12), (7, 32, 1, 12)])
def test_float32_readout(grp, tq, S, frames):
    """float32 KV on float32 MFMAs.  Bound: the logits (|q| <= 60, |k| <= 2.5,
    |q.k| / sqrt(D) <= 14) carry at most 24 roundings' worth of error, 2e-5; a
    weight twice that; an output of values up to 5 below 2e-4, an lse below
    3e-5.  An infinite value in the last key reaches its own dim and no other."""
    import torch
    h = H()
    wl = W.WORKLOADS["tiny"].with_(num_layers=2, num_kv_heads=2, num_q_heads=2 * grp, grid_h=5, grid_w=7,
                                   frames=frames, window_frames=3, capacity=37, query_tokens=tq)
    h.log(f"case: float32 readout rows {grp * tq} S={S} frames {frames}")
    pair = _stream(h, wl, S=S)
    q = pair.query(np.random.default_rng(grp * 100 + tq))
    pseudo = pair.oracle[0].synthesize()
    oo, ol = pair.oracle[0].attend(q, wl.num_kv_heads, pseudo)
    pair.gpu.synthesize(0)
    qd = torch.from_numpy(q).to("cuda").contiguous()
    o, lse = pair.gpu.attend(0, qd)
    torch.cuda.synchronize()
    err, el = np.abs(o.cpu().numpy() - oo).max(), np.abs(lse.cpu().numpy() - ol).max()
    h.log(f"readout err {err:.2e}, lse err {el:.2e}")
    assert err <= 2e-4 and el <= 3e-5
    if frames == 2:
        k, v = (torch.randn(1, 2, 2, 35, 128, device="cuda") * 0.1 for _ in range(2))
        v[0, 0, 0, 34, 7] = float("inf")
        pair.gpu.append_frame([0], k, v)
        pair.gpu.synthesize(0)
        o, _ = pair.gpu.attend(0, qd * 0.01)
        torch.cuda.synchronize()
        inf = torch.isinf(o)
        assert bool(inf[0, :, 0, 7].all()) and int(inf.sum()) == tq and not bool(torch.isnan(o).any())
