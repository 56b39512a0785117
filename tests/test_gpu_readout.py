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


def _histograms(kind, C, rng):
    """[8][C] counts, every subspace with the same total."""
    if kind == "equal":
        return np.full((8, C), 3, dtype=np.int64)
    top = {"collide": 6, "join below 8": 57, "join above 8": 58, "join below 16": 48, "join above 16": 49,
           "half below": 607, "half above": 608, "wide": 400}.get(kind)
    if top is not None:   # one count vector, permuted per subspace: products collide
        base = np.array([top, top - 1, top - 1] + [top * (C - i) // C for i in range(3, C)], dtype=np.int64)[:C]
        return np.stack([base[rng.permutation(C)] for _ in range(8)])
    top = {"count below": 4094, "count above": 4095}[kind]   # one subspace peaked, the others even
    out = np.full((8, C), top // C, dtype=np.int64)
    out[:, :top % C] += 1
    out[3] = 0
    out[3, C // 2] = top
    return out


# S = 8 and 16 are the lists' own lengths; C = 2 has fewer codewords than
# ranks; of 256 units x 260 slots, 16 to a wave, waves straddle units
@pytest.mark.parametrize("S,C,units,cap", [(8, 16, 2, 40), (5, 12, 2, 40), (1, 2, 2, 40), (16, 16, 2, 40),
                                           (9, 2, 2, 40), (8, 16, 256, 260)])
def test_decode_at_the_edges_of_its_products(S, C, units, cap):
    """Exact top-S tuples with every slot of a launch on one side of a limit:
    half products below and above 2^37, joined products below and above the
    mantissa's room beside the tag, counts of 4094 and 4095, all products
    equal, products colliding across tuples.  Rows bitwise against the oracle's."""
    from oracle import protokv_oracle as O
    h = H()
    kvh = min(units, 8)
    wl = W.WORKLOADS["7b"].with_(num_layers=units // kvh, num_kv_heads=kvh, num_q_heads=kvh, grid_h=7, grid_w=7,
                                 frames=0, window_frames=2, capacity=cap, query_tokens=1)
    p = h.oracle_params(wl, S=S, C=C, B=max(32, S))
    cb = W.make_codebooks_device(wl, samples=256, iters=3, C=C)[0]
    gpu = h.pk.ProtoKV(h.gpu_config(wl, p), cb)
    gen = W.DeviceStream(wl)
    while gpu.stream_info(0).active_slots < cap or gpu.stream_info(0).evicted_tokens < 20000:
        gpu.append_frame([0], *gen.next_frame())
        gpu.fold()
    state = gpu.get_state(0)
    rng = np.random.default_rng(S * 100 + C)
    sample = [0, units - 1]
    kinds = ["equal", "collide", "join below 8", "join above 8", "join below 16", "join above 16", "half below",
             "half above", "wide", "count below", "count above"]
    for kind in kinds if units == 2 else ["collide", "wide", "half above"]:
        h.log(f"case: decode limits {kind} S={S} C={C} units={units} K={cap}")
        bank = state.bank()
        hist = np.stack([_histograms(kind, C, rng) for _ in range(2 * cap)]).reshape(2, cap, 8, C)
        for u in range(units):
            for name, x in (("hist_k", hist[0]), ("hist_v", hist[1])):
                bank[name][u, :, :, :C] = np.roll(x, u, axis=0)
            bank["n_res"][u] = hist[0, 0, 0].sum()
            bank["n"][u] = hist[0, 0, 0].sum() + 1
        rows = h.pk.encode_bank(bank, units, cap).reshape(units, -1)
        for u in range(units):
            state.set_bank_rows(u, rows[u])
        gpu.set_state(0, state)
        gpu.synthesize(0)
        gk, gv, _ = gpu.read_pseudo()
        for u in sample:
            ps = O.synthesize(h.bank_from_rows(bank, u, p), cb[u], p)
            n = len(ps.keys)
            assert np.array_equal(gk[u][:n], ps.keys) and np.array_equal(gv[u][:n], ps.values), f"{kind} unit {u}"


def _large_histograms(kind, C, slot, rng):
    """[8][C] counts of one slot, every subspace with the same total <= 65534."""
    if kind == "mixed":   # one slot of a wave's 16 beyond 4094
        kind = "descending to 7000" if slot % 16 == 5 else "descending to 40"
    if kind.startswith("flat"):   # "flat n": products equal; "flat n -": nearly, and colliding
        top = int(kind.split()[1])
        base = np.full(C, top, dtype=np.int64)
        if kind.endswith("-"):
            base[rng.permutation(C)[:C // 2]] -= 1
    elif kind.startswith("descending"):
        top = int(kind.split()[-1])
        base = np.array([top * (C - i) // C for i in range(C)], dtype=np.int64)
    else:   # "peaks n": n codewords share 65534
        n = int(kind.split()[1])
        base = np.zeros(C, dtype=np.int64)
        base[:n] = 65534 // n
    return np.stack([base[rng.permutation(C)] for _ in range(8)])


@pytest.mark.parametrize("S,C", [(8, 16), (16, 16), (3, 12), (9, 2), (16, 11)])
def test_decode_of_large_counts(S, C):
    """Exact top-S tuples of slots with thousands of residuals a codeword: half
    products up to 4095^4 and joined ones up to 4095^8, 40 bits below and just
    below what their formats hold, and beyond 4094 up to 65534 residuals in one
    codeword, alone in a wave or throughout.  Rows bitwise against the oracle's."""
    import ctypes
    from oracle import protokv_oracle as O
    h = H()
    cap = 37
    wl = W.WORKLOADS["7b"].with_(num_layers=2, num_kv_heads=1, num_q_heads=1, grid_h=7, grid_w=7, frames=0,
                                 window_frames=2, capacity=cap, query_tokens=1)
    p = h.oracle_params(wl, S=S, C=C, B=max(32, S))
    cb = W.make_codebooks_device(wl, samples=256, iters=3, C=C)[0]
    gpu = h.pk.ProtoKV(h.gpu_config(wl, p), cb)
    gen = W.DeviceStream(wl)
    for _ in range(4):
        gpu.append_frame([0], *gen.next_frame())
        gpu.fold()
    state = gpu.get_state(0)
    # a stream position that allows 65534 residuals a slot
    hd, T = state.header, wl.tokens_per_frame
    hd.folds = -(-65534 // T)
    hd.frames, hd.evicted_tokens = hd.folds + wl.window_frames, hd.folds * T
    state.blob[:ctypes.sizeof(hd)] = np.frombuffer(bytes(hd), dtype=np.uint8)
    rng = np.random.default_rng(S * 100 + C)
    for kind in ("flat 4094", "flat 4094 -", "descending to 4094", "flat 4095", "flat 4095 -", "descending to 7000",
                 "mixed", "peaks 2", "peaks 1"):
        h.log(f"case: decode of large counts {kind} S={S} C={C}")
        bank = state.bank()
        for u in range(wl.units):
            for k in range(cap):
                hist = [_large_histograms(kind, C, k, rng) for _ in range(2)]
                bank["hist_k"][u, k, :, :C], bank["hist_v"][u, k, :, :C] = hist
                n = int(hist[0][0].sum())
                assert n <= 65534 and all(int(x.sum(axis=1).max()) == int(x.sum(axis=1).min()) == n for x in hist)
                bank["n_res"][u, k], bank["n"][u, k] = n, n + 1
        rows = h.pk.encode_bank(bank, wl.units, cap).reshape(wl.units, -1)
        for u in range(wl.units):
            state.set_bank_rows(u, rows[u])
        gpu.set_state(0, state)
        gpu.synthesize(0)
        gk, gv, _ = gpu.read_pseudo()
        for u in range(wl.units):
            ps = O.synthesize(h.bank_from_rows(bank, u, p), cb[u], p)
            n = len(ps.keys)
            assert np.array_equal(gk[u][:n], ps.keys) and np.array_equal(gv[u][:n], ps.values), f"{kind} unit {u}"


# rows per kv head 1, 32 and 9; formed tiles of 5 slots x 5, 6 and of 3 x 9 (the
# rest of the 32 rows masked), last tiles of 2, 1 and 1 slots; loaded contexts of
# 105 (last tile of 9 keys) and, without a bank, 70
@pytest.mark.parametrize("grp,tq,S,cap,frames,theta", [(1, 1, 5, 37, 12, 0.0), (8, 4, 6, 36, 12, 1e4),
                                                       (3, 3, 9, 31, 12, 0.0), (1, 9, 8, 37, 2, 0.0)])
def test_few_row_readout(grp, tq, S, cap, frames, theta):
    """bf16 readout of at most 32 query rows per kv head, pseudo-token rows formed
    in the wave and then written, against the oracle; without a bank an infinite
    value in the last key reaches its own dim and no other."""
    import torch
    h = H()
    wl = W.WORKLOADS["7b"].with_(num_layers=3, num_kv_heads=1, num_q_heads=grp, grid_h=5, grid_w=7, frames=frames,
                                 window_frames=3, capacity=cap, query_tokens=tq)
    h.log(f"case: few rows {grp * tq} S={S} K={cap} frames {frames} theta {theta}")
    pair = _stream(h, wl, S=S, B=max(32, S), rope_theta=theta)
    q = pair.query(np.random.default_rng(S))
    pseudo = pair.oracle[0].synthesize()
    oo, ol = pair.oracle[0].attend(q, wl.num_kv_heads, pseudo)
    qd = torch.from_numpy(q).to("cuda", torch.bfloat16).contiguous()
    pair.gpu.synthesize(0)
    for form in ("formed", "written"):
        o, lse = pair.gpu.attend(0, qd)
        torch.cuda.synchronize()
        err, el = np.abs(o.float().cpu().numpy() - oo).max(), np.abs(lse.cpu().numpy() - ol).max()
        h.log(f"{form} rows: err {err:.2e}, lse {el:.2e}")
        assert err <= h.READOUT_ATOL and el <= h.LSE_ATOL
        pair.gpu.read_pseudo()   # writes the rows
    if frames == 2:
        k, v = (torch.randn(1, 3, 1, 35, 128, device="cuda").bfloat16() for _ in range(2))
        v[0, 0, 0, 34, 7] = float("inf")
        pair.gpu.append_frame([0], k, v)
        pair.gpu.synthesize(0)
        o, _ = pair.gpu.attend(0, qd * 0.01)
        torch.cuda.synchronize()
        inf = torch.isinf(o)
        assert bool(inf[0, :, 0, 7].all()) and int(inf.sum()) == tq and not bool(torch.isnan(o).any())


# 40 .. 48 rows (key halves shared by wave pairs) and 136 (a wave per 32 rows); 12,
# 9, 4 and 4 whole slots per 64-row tile (60, 63, 52 and 64 rows), last tiles short
@pytest.mark.parametrize("grp,tq,S,cap,theta", [(4, 10, 5, 37, 0.0), (8, 17, 7, 40, 1e4), (4, 12, 13, 30, 0.0),
                                                (8, 5, 16, 33, 1e4)])
def test_formed_tiles_of_whole_slots(grp, tq, S, cap, theta):
    """bf16 readout of more than 32 query rows per kv head, pseudo-token tiles of
    whole slots formed in LDS and then rows written, against the oracle."""
    import torch
    h = H()
    wl = W.WORKLOADS["7b"].with_(num_layers=2, num_kv_heads=1, num_q_heads=grp, grid_h=7, grid_w=7, frames=12,
                                 window_frames=3, capacity=cap, query_tokens=tq)
    h.log(f"case: formed tiles rows {grp * tq} S={S} K={cap} theta {theta}")
    pair = _stream(h, wl, S=S, B=max(32, S), rope_theta=theta)
    q = pair.query(np.random.default_rng(S))
    oo, ol = pair.oracle[0].attend(q, wl.num_kv_heads, pair.oracle[0].synthesize())
    qd = torch.from_numpy(q).to("cuda", torch.bfloat16).contiguous()
    pair.gpu.synthesize(0)
    for form in ("formed", "written"):
        o, lse = pair.gpu.attend(0, qd)
        torch.cuda.synchronize()
        err, el = np.abs(o.float().cpu().numpy() - oo).max(), np.abs(lse.cpu().numpy() - ol).max()
        h.log(f"{form} rows: err {err:.2e}, lse {el:.2e}")
        assert err <= h.READOUT_ATOL and el <= h.LSE_ATOL
        pair.gpu.read_pseudo()   # writes the rows


def _seeking_query(pair, pseudo, seed):
    """A query of which every second row of the sampled units looks for one key,
    the keys spread over the context from first to last: its logit, 25, is far
    above those before it, so a row's running maximum grows late."""
    q = pair.query(np.random.default_rng(seed))
    wl, ora = pair.wl, pair.oracle[0]
    grp = wl.num_q_heads // wl.num_kv_heads
    rows = wl.query_tokens * grp
    for i, u in enumerate(pair.sample):
        l, h = divmod(u, wl.num_kv_heads)
        k = ora.context(i, pseudo[i])[0]
        for r in range(0, rows, 2):
            key = k[r * (len(k) - 1) // max(rows - 1, 1)]
            q[l, r // grp, h * grp + r % grp] = key * (25.0 * np.sqrt(128.0) / float(key @ key))
    return W.quantize(q, wl.kv_dtype)


def _check_readout(h, pair, q, form):
    """The device's readout of the sampled units against the oracle's.  Weights are
    rounded to bf16 and their sum is taken over the rounded ones, so where a few
    equal rows hold all the mass the lse errs by up to bf16's unit roundoff, 2^-8
    (float32's own errors stay below 1e-4)."""
    import torch
    wl, grp = pair.wl, pair.wl.num_q_heads // pair.wl.num_kv_heads
    o, lse = pair.gpu.attend(0, torch.from_numpy(q).to("cuda", torch.bfloat16).contiguous())
    torch.cuda.synchronize()
    go, gl = o.float().cpu().numpy(), lse.cpu().numpy()
    oo, ol = pair.oracle[0].attend(q, wl.num_kv_heads, pair.oracle[0].synthesize())
    worst, worst_lse = 0.0, 0.0
    for u in pair.sample:
        l, kvh = divmod(u, wl.num_kv_heads)
        heads = slice(kvh * grp, (kvh + 1) * grp)
        worst = max(worst, float(np.abs(go[l][:, heads] - oo[l][:, heads]).max()))
        worst_lse = max(worst_lse, float(np.abs(gl[l][:, heads] - ol[l][:, heads]).max()))
    h.log(f"{form} rows: err {worst:.2e}, lse {worst_lse:.2e}")
    assert worst <= h.READOUT_ATOL and worst_lse <= 2.0 ** -8 + 1e-4


# One workgroup (two in the first case) for a kv head's whole context, so that it
# goes through at least four formed tiles: of 8 slots, 40 and 27 a split; of 5, 9,
# 4 and 8 slots with 5, 5, 2 and 5 in the last; 105 near keys, or 105 + 37 x 8
# .. 53 x 5 written rows, are two, five and more loaded tiles.  Rows 40 (two waves
# per 32 rows, a key half each) and 136 (a wave per 32)
@pytest.mark.parametrize("units,grp,tq,S,cap,theta,opt", [
    (128, 8, 5, 8, 67, 0.0, {}), (192, 8, 5, 5, 53, 1e4, {}), (192, 8, 17, 7, 41, 1e4, {"ema": True}),
    (192, 8, 17, 16, 18, 1e4, {}), (192, 8, 5, 16, 18, 0.0, {"ema": True}), (192, 8, 5, 8, 37, 0.0, {"use_pq": False}),
    (192, 8, 17, 5, 53, 0.0, {"ema": True})])
def test_formed_tiles_in_turn(units, grp, tq, S, cap, theta, opt):
    """bf16 readout of more than 32 query rows per kv head, several tiles of each
    kind to a workgroup: staging, centres, rotation tables and tiles three, two and
    one ahead, the running maximum growing late.  Formed rows and then written
    ones, against the oracle on three units."""
    h = H()
    wl = W.WORKLOADS["7b"].with_(num_layers=units // 8, num_kv_heads=8, num_q_heads=8 * grp, grid_h=5, grid_w=7,
                                 frames=8, window_frames=3, capacity=cap, query_tokens=tq)
    h.log(f"case: formed tiles in turn units {units} rows {grp * tq} S={S} K={cap} theta {theta} {opt}")
    pair = _stream(h, wl, sample=[0, units // 2 + 3, units - 1], cb_samples=64, cb_iters=2, S=S, B=max(32, S),
                   rope_theta=theta, **opt)
    q = pair.query(np.random.default_rng(S)) if theta else _seeking_query(pair, pair.oracle[0].synthesize(), S)
    pair.synthesize()
    _check_readout(h, pair, q, "formed")
    pair.check_rows()   # writes the rows
    _check_readout(h, pair, q, "written")


# One workgroup of eight waves a kv head: 588 near keys (and 3 x 52 written rows) in
# tiles of 32 give every wave two or three loaded tiles, 52 slots at 5, 4 and 2 to a
# tile one to four formed ones; half the waves take the formed ones first.  Rows 7,
# 32, 7 and 21
@pytest.mark.parametrize("grp,tq,S,theta,opt", [(7, 1, 5, 0.0, {"ema": True}), (8, 4, 8, 0.0, {}), (7, 1, 16, 1e4, {}),
                                                (7, 3, 3, 0.0, {}), (7, 1, 8, 0.0, {"use_pq": False})])
def test_few_rows_many_tiles(grp, tq, S, theta, opt):
    """bf16 readout of at most 32 query rows, several tiles of each kind to a wave:
    the next tile's loads under this one's products, the wave's LDS used again,
    the running maximum growing late.  Formed rows and then written ones, against
    the oracle on three units."""
    h = H()
    units, cap = 192, 52
    wl = W.WORKLOADS["7b"].with_(num_layers=units // 8, num_kv_heads=8, num_q_heads=8 * grp, grid_h=14, grid_w=14,
                                 frames=5, window_frames=3, capacity=cap, query_tokens=tq)
    h.log(f"case: few rows, many tiles rows {grp * tq} S={S} theta {theta} {opt}")
    pair = _stream(h, wl, sample=[0, units // 2 + 3, units - 1], cb_samples=64, cb_iters=2, S=S, B=max(32, S),
                   rope_theta=theta, **opt)
    q = pair.query(np.random.default_rng(S)) if theta else _seeking_query(pair, pair.oracle[0].synthesize(), S)
    pair.synthesize()
    _check_readout(h, pair, q, "formed")
    pair.check_rows()   # writes the rows
    _check_readout(h, pair, q, "written")


# 588 near keys + 60 x 16 or 60 x 3 rows: 49 and 24 tiles of 32 over at most 16
# splits, three or four and two to a wave, the last of 12 keys; rows 33 and 7
@pytest.mark.parametrize("grp,tq,S", [(3, 11, 16), (7, 1, 3)])
def test_float32_readout_many_tiles(grp, tq, S):
    """float32 KV, several tiles to a wave, the running maximum growing late.  A dot
    product goes through at most 24 roundings, so a logit errs by less than e = 24
    2^-24 |q| |k| / sqrt(D); its weight by twice that.  A sum over a wave's keys and
    the splits' is a chain of at most 4 x 32 + 16 roundings, 192 with those of the
    exponentials and the rescaling."""
    import torch
    h = H()
    wl = W.WORKLOADS["tiny"].with_(num_layers=2, num_kv_heads=2, num_q_heads=2 * grp, grid_h=14, grid_w=14, frames=5,
                                   window_frames=3, capacity=60, query_tokens=tq)
    h.log(f"case: float32 readout, many tiles rows {grp * tq} S={S}")
    pair = _stream(h, wl, S=S)
    pseudo = pair.oracle[0].synthesize()
    q = _seeking_query(pair, pseudo, S)
    oo, ol = pair.oracle[0].attend(q, wl.num_kv_heads, pseudo)
    pair.gpu.synthesize(0)
    o, lse = pair.gpu.attend(0, torch.from_numpy(q).to("cuda").contiguous())
    torch.cuda.synchronize()
    ctx = [pair.oracle[0].context(i, ps) for i, ps in enumerate(pseudo)]
    kmax = max(float(np.linalg.norm(c[0], axis=1).max()) for c in ctx)
    vmax = max(float(np.abs(c[1]).max()) for c in ctx)
    e = 24 * 2.0 ** -24 * float(np.linalg.norm(q, axis=-1).max()) * kmax / np.sqrt(128.0)
    err, el = np.abs(o.cpu().numpy() - oo).max(), np.abs(lse.cpu().numpy() - ol).max()
    h.log(f"readout err {err:.2e} (bound {(2 * e + 192 * 2.0 ** -24) * vmax:.1e}), lse err {el:.2e} ({e + 192 * 2.0 ** -24:.1e})")
    assert err <= (2 * e + 192 * 2.0 ** -24) * vmax and el <= e + 192 * 2.0 ** -24
