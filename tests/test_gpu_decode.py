"""GPU parity of viscache_append_kv / viscache_decode_attn against the oracle's
decode attention (Sec. 2, decoding), through the C ABI, including decode over
a cache that viscache_prune has just compressed."""
import numpy as np
import pytest

from tests.parity import fused_error

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
TOL = 1e-4


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2608_24063_amd as vc
    vc.lib()
    return torch.device("cuda:0")


def _bits(sg, seed, stream, shape):
    return sg.normal_bf16(seed, stream, shape)


def _check_out(orc, q, K, V, out, scale, what):
    ref = orc.attend(q, K, V, scale)
    err = fused_error(ref[None, :], out[None, :])
    assert err <= TOL, f"{what}: decode error {err}"


@pytest.mark.parametrize("d,Hq,Hkv", [(128, 8, 2), (64, 28, 4), (128, 64, 8)])
def test_decode_random_caches(dev, orc, sg, d, Hq, Hkv):
    from paper_2608_24063_amd.tensors import DecodeCache
    from synthgen.device import bf16_tensor, to_host_bf16
    L, B = 2, 2
    units = L * B * Hkv
    # Empty, sub-tile and tile edges, and units long enough to be cut over
    # several workgroups.
    lens = [0, 1, 31, 33, 3100, 511, 1023, 1024, 1100, 5, 64, 2049, 2, 1025, 47, 4097][:units]
    lens += [17] * (units - len(lens))
    caps = [x + 3 for x in lens]
    c = DecodeCache(L, B, Hq, Hkv, d, caps, dev)
    Kp = _bits(sg, 7, 1, (c.total_rows, d))
    Vp = _bits(sg, 7, 2, (c.total_rows, d))
    c.k_pool.copy_(bf16_tensor(Kp, dev))
    c.v_pool.copy_(bf16_tensor(Vp, dev))
    c.len.copy_(torch.tensor(lens, dtype=torch.int32))
    q = _bits(sg, 7, 3, (L, B, Hq, d))
    out = torch.full((L, B, Hq, d), float("nan"), dtype=torch.float32, device=dev)
    scale = d ** -0.5
    c.attend(bf16_tensor(q, dev), out, scale)
    torch.cuda.synchronize()
    o = out.cpu().numpy()
    G = Hq // Hkv
    for l in range(L):
        for b in range(B):
            for g in range(Hkv):
                u = (l * B + b) * Hkv + g
                r0, n = c.offs_host[u], lens[u]
                for hh in range(G):
                    h = g * G + hh
                    if n == 0:
                        assert np.all(o[l, b, h] == 0)
                        continue
                    _check_out(orc, q[l, b, h], Kp[r0:r0 + n], Vp[r0:r0 + n], o[l, b, h], scale,
                               f"l={l} b={b} h={h} n={n}")


def test_append_respects_capacity(dev, sg):
    from paper_2608_24063_amd.tensors import DecodeCache
    from synthgen.device import bf16_tensor, to_host_bf16
    L, B, Hq, Hkv, d = 2, 1, 4, 2, 64
    caps = [3, 2, 5, 1]
    c = DecodeCache(L, B, Hq, Hkv, d, caps, dev)
    c.len.copy_(torch.tensor([0, 2, 4, 0], dtype=torch.int32))
    kn = _bits(sg, 9, 1, (L, B, Hkv, d))
    vn = _bits(sg, 9, 2, (L, B, Hkv, d))
    c.append(bf16_tensor(kn, dev), bf16_tensor(vn, dev))
    torch.cuda.synchronize()
    assert c.len.cpu().tolist() == [1, 2, 5, 1]
    K = to_host_bf16(c.k_pool)
    V = to_host_bf16(c.v_pool)
    kn2, vn2 = kn.reshape(-1, d), vn.reshape(-1, d)
    for u, pos in [(0, 0), (2, 4), (3, 0)]:
        np.testing.assert_array_equal(K[c.offs_host[u] + pos], kn2[u])
        np.testing.assert_array_equal(V[c.offs_host[u] + pos], vn2[u])
    assert np.all(K[c.offs_host[1]:c.offs_host[1] + 2] == 0)  # full unit untouched


def test_decode_over_pruned_cache(dev, orc, sg):
    """prune -> cache of (kept visual | text window | generated) rows ->
    append + attend for a few steps, each step checked against the oracle."""
    import paper_2608_24063_amd as vc
    from paper_2608_24063_amd.tensors import DecodeCache, PruneCall
    from synthgen.device import bf16_tensor, to_host_bf16, upload_layers
    w = sg.TINY
    n = [int(x) for x in w.n_vis()]
    params = vc.make_params(w.retention)
    dv, host = upload_layers(w, range(w.L), dev, keep_host=True)
    pc = PruneCall(w.B, w.L, w.Hq, w.Hkv, w.d, w.W, n, params, [dv["K"][l] for l in range(w.L)],
                   [dv["V"][l] for l in range(w.L)], [dv["Q"][l] for l in range(w.L)])
    pc.run()
    steps = 6
    caps, kept_rows = [], []
    for l in range(w.L):
        for b in range(w.B):
            for g in range(w.Hkv):
                k = pc.k[b * w.L + l]
                kept_rows.append(k)
                caps.append(k + w.W + steps)
    c = DecodeCache(w.L, w.B, w.Hq, w.Hkv, w.d, caps, dev)
    text_k = _bits(sg, w.seed, 11, (len(caps), w.W, w.d))
    text_v = _bits(sg, w.seed, 12, (len(caps), w.W, w.d))
    lens = []
    for l in range(w.L):
        for b in range(w.B):
            for g in range(w.Hkv):
                u = (l * w.B + b) * w.Hkv + g
                r0 = c.offs_host[u]
                k = kept_rows[u]
                if k:
                    a0, a1 = pc.unit_rows(l, b, g)
                    c.k_pool[r0:r0 + k] = pc.k_out[l][a0:a1]
                    c.v_pool[r0:r0 + k] = pc.v_out[l][a0:a1]
                c.k_pool[r0 + k:r0 + k + w.W] = bf16_tensor(text_k[u], dev)
                c.v_pool[r0 + k:r0 + k + w.W] = bf16_tensor(text_v[u], dev)
                lens.append(k + w.W)
    c.len.copy_(torch.tensor(lens, dtype=torch.int32))
    scale = w.d ** -0.5
    out = torch.empty((w.L, w.B, w.Hq, w.d), dtype=torch.float32, device=dev)
    for t in range(steps):
        kn = _bits(sg, w.seed, 100 + 3 * t, (w.L, w.B, w.Hkv, w.d))
        vn = _bits(sg, w.seed, 101 + 3 * t, (w.L, w.B, w.Hkv, w.d))
        q = _bits(sg, w.seed, 102 + 3 * t, (w.L, w.B, w.Hq, w.d))
        c.append(bf16_tensor(kn, dev), bf16_tensor(vn, dev))
        c.attend(bf16_tensor(q, dev), out, scale)
        torch.cuda.synchronize()
        K, V, o = to_host_bf16(c.k_pool), to_host_bf16(c.v_pool), out.cpu().numpy()
        ln = c.len.cpu().numpy()
        for l in range(w.L):
            for b in range(w.B):
                for g in range(w.Hkv):
                    u = (l * w.B + b) * w.Hkv + g
                    assert ln[u] == lens[u] + t + 1
                    r0 = c.offs_host[u]
                    for hh in (0, w.G - 1):
                        h = g * w.G + hh
                        _check_out(orc, q[l, b, h], K[r0:r0 + ln[u]], V[r0:r0 + ln[u]], o[l, b, h], scale,
                                   f"step {t} l={l} h={h}")


@pytest.mark.parametrize("d,Hq,Hkv", [(128, 28, 4), (64, 8, 2)])
def test_decode_step_matches_append_then_attend(dev, orc, sg, d, Hq, Hkv):
    """viscache_decode_step (one launch) against viscache_append_kv followed by
    viscache_decode_attn on a copy of the same cache, over several steps:
    identical outputs (bit for bit), lengths and pools; the oracle checks the
    attention.  Lengths cross tile edges, units are cut over several
    workgroups, and one reaches capacity."""
    from paper_2608_24063_amd.tensors import DecodeCache
    from synthgen.device import bf16_tensor, to_host_bf16
    L, B = 2, 1
    units = L * B * Hkv
    lens = [0, 1022, 1023, 31, 2047, 5, 64, 3000][:units]
    caps = [x + 4 for x in lens]
    caps[1] = lens[1] + 2  # reaches capacity after two appends
    a = DecodeCache(L, B, Hq, Hkv, d, caps, dev)
    c = DecodeCache(L, B, Hq, Hkv, d, caps, dev)
    Kp = _bits(sg, 21, 1, (a.total_rows, d))
    Vp = _bits(sg, 21, 2, (a.total_rows, d))
    for cc in (a, c):
        cc.k_pool.copy_(bf16_tensor(Kp, dev))
        cc.v_pool.copy_(bf16_tensor(Vp, dev))
        cc.len.copy_(torch.tensor(lens, dtype=torch.int32))
    scale = d ** -0.5
    cur = list(lens)
    for t in range(4):
        kn = _bits(sg, 22 + t, 1, (L, B, Hkv, d))
        vn = _bits(sg, 22 + t, 2, (L, B, Hkv, d))
        q = _bits(sg, 22 + t, 3, (L, B, Hq, d))
        kt, vt, qt = bf16_tensor(kn, dev), bf16_tensor(vn, dev), bf16_tensor(q, dev)
        out_a = torch.full((L, B, Hq, d), float("nan"), dtype=torch.float32, device=dev)
        out_c = torch.full((L, B, Hq, d), float("nan"), dtype=torch.float32, device=dev)
        a.append(kt, vt)
        a.attend(qt, out_a, scale)
        c.step(kt, vt, qt, out_c, scale)
        torch.cuda.synchronize()
        assert torch.equal(out_a, out_c), f"step {t}: fused step differs from append + attend"
        assert a.len.cpu().tolist() == c.len.cpu().tolist()
        cur = [min(x + 1, cap) for x, cap in zip(cur, caps)]
        assert c.len.cpu().tolist() == cur
        assert torch.equal(a.k_pool, c.k_pool) and torch.equal(a.v_pool, c.v_pool)
    # The oracle on the final step.
    K = to_host_bf16(c.k_pool)
    V = to_host_bf16(c.v_pool)
    o = out_c.cpu().numpy()
    G = Hq // Hkv
    for l in range(L):
        for b in range(B):
            for g in range(Hkv):
                u = (l * B + b) * Hkv + g
                r0, n = c.offs_host[u], cur[u]
                for hh in range(0, G, 3):
                    h = g * G + hh
                    _check_out(orc, q[l, b, h], K[r0:r0 + n], V[r0:r0 + n], o[l, b, h], scale,
                               f"step l={l} g={g} h={h} n={n}")
    _counters_zero(c, units)


def _counters_zero(c, units):
    """The fused step's arrival counters (at the front of its workspace) are
    back at zero, and the words past the decode workspace are untouched."""
    import paper_2608_24063_amd as vc
    base = vc.viscache_decode_workspace_bytes(c.shape, c.max_cap)
    assert int(c.step_ws[base:base + 4 * units].view(torch.int32).abs().sum()) == 0
    assert int(c.step_ws[:4 * units].view(torch.int32).abs().sum()) == 0


def test_decode_many_units_and_long_unit(dev, orc, sg):
    """More units than one pass of the block prefix sum covers (1280), most
    of them short or empty, and one 40000-row unit cut into more than a
    hundred pieces (a grid beyond the resident slots, merges of many
    partials): the fused step equals append + attend bit for bit, and the
    oracle checks every unit."""
    from paper_2608_24063_amd.tensors import DecodeCache
    from synthgen.device import bf16_tensor, to_host_bf16
    L, B, Hq, Hkv, d = 2, 80, 16, 8, 64
    units = L * B * Hkv
    rng = np.random.default_rng(5)
    lens = [int(x) for x in rng.integers(0, 70, size=units)]
    lens[3], lens[700], lens[1279] = 40000, 5000, 0
    caps = [x + 2 for x in lens]
    caps[1279] = 0  # no room at all
    a = DecodeCache(L, B, Hq, Hkv, d, caps, dev)
    c = DecodeCache(L, B, Hq, Hkv, d, caps, dev)
    Kp = _bits(sg, 31, 1, (a.total_rows, d))
    Vp = _bits(sg, 31, 2, (a.total_rows, d))
    for cc in (a, c):
        cc.k_pool.copy_(bf16_tensor(Kp, dev))
        cc.v_pool.copy_(bf16_tensor(Vp, dev))
        cc.len.copy_(torch.tensor(lens, dtype=torch.int32))
    scale = d ** -0.5
    kn = _bits(sg, 32, 1, (L, B, Hkv, d))
    vn = _bits(sg, 32, 2, (L, B, Hkv, d))
    q = _bits(sg, 32, 3, (L, B, Hq, d))
    kt, vt, qt = bf16_tensor(kn, dev), bf16_tensor(vn, dev), bf16_tensor(q, dev)
    out_a = torch.full((L, B, Hq, d), float("nan"), dtype=torch.float32, device=dev)
    out_c = torch.full((L, B, Hq, d), float("nan"), dtype=torch.float32, device=dev)
    a.append(kt, vt)
    a.attend(qt, out_a, scale)
    c.step(kt, vt, qt, out_c, scale)
    torch.cuda.synchronize()
    assert torch.equal(out_a, out_c), "fused step differs from append + attend"
    cur = [min(x + 1, cap) for x, cap in zip(lens, caps)]
    assert c.len.cpu().tolist() == cur and a.len.cpu().tolist() == cur
    assert torch.equal(a.k_pool, c.k_pool) and torch.equal(a.v_pool, c.v_pool)
    _counters_zero(c, units)
    K = to_host_bf16(c.k_pool)
    V = to_host_bf16(c.v_pool)
    o = out_c.cpu().numpy()
    G = Hq // Hkv
    for l in range(L):
        for b in range(B):
            for g in range(Hkv):
                u = (l * B + b) * Hkv + g
                r0, n = c.offs_host[u], cur[u]
                h = g * G + (u % G)
                if n == 0:
                    assert np.all(o[l, b, g * G:(g + 1) * G] == 0)
                    continue
                _check_out(orc, q[l, b, h], K[r0:r0 + n], V[r0:r0 + n], o[l, b, h], scale, f"u={u} n={n}")


@pytest.mark.parametrize("d,Hkv", [(64, 1), (128, 2), (128, 65)])
def test_step_layers_with_unlike_capacities(dev, sg, d, Hkv):
    """One launch per layer over layers whose capacities differ widely (the
    pruned cache of a layer-wise budget), sharing one workspace: the results
    and lengths of one launch for all layers, over several steps.  Calls of a
    few units and of more than 64, units in one piece and in many, and more
    pieces than the launch has workgroups for at the smallest bound.  The
    piece bounds of the two launches differ, so results agree to fp32 rounding
    (weights as bf16 pairs, within 2^-17)."""
    from paper_2608_24063_amd.tensors import DecodeCache
    L, B, G, steps = 4, 1, 2, 3
    caps = []
    for l, top in enumerate((5000, 40, 900, 2100)):
        caps += [max(steps + 1, top // (1 + u % 7)) for u in range(B * Hkv)]
    gen = torch.Generator(device=dev).manual_seed(d + Hkv)
    rnd = lambda *s: torch.randn(s, generator=gen, device=dev).to(torch.bfloat16)
    a, b = (DecodeCache(L, B, Hkv * G, Hkv, d, caps, dev) for _ in range(2))
    a.k_pool.copy_(rnd(*a.k_pool.shape))
    a.v_pool.copy_(rnd(*a.v_pool.shape))
    b.k_pool.copy_(a.k_pool)
    b.v_pool.copy_(a.v_pool)
    lens = torch.tensor([c - steps for c in caps], dtype=torch.int32)
    a.len.copy_(lens)
    b.len.copy_(lens)
    oa, ob = (torch.empty((L, B, Hkv * G, d), dtype=torch.float32, device=dev) for _ in range(2))
    for t in range(steps):
        k, v, q = rnd(L, B, Hkv, d), rnd(L, B, Hkv, d), rnd(L, B, Hkv * G, d)
        a.step_layers(k, v, q, oa, d ** -0.5)
        b.step(k, v, q, ob, d ** -0.5)
        torch.cuda.synchronize()
        assert float((oa - ob).abs().max()) <= 2.0 ** -16 * float(a.v_pool.float().abs().max())
        assert torch.equal(a.len, b.len) and a.len.cpu().tolist() == (lens + t + 1).tolist()
    assert torch.equal(a.k_pool, b.k_pool) and torch.equal(a.v_pool, b.v_pool)


@pytest.mark.parametrize("units,lo,hi", [(130, 100, 900), (130, 770, 780), (300, 100, 900), (300, 513, 514),
                                         (300, 300, 600), (300, 1025, 1030), (700, 100, 300), (700, 100, 900),
                                         (700, 40, 2500)])
def test_cut_of_many_units(dev, units, lo, hi):
    """The device's cut with one chunk of units and with several: the smallest
    piece bound fits, a larger one does (found after the first or with it), or
    none of the four.  Against the planned step, whose pieces are cut on the
    host: equal to fp32 rounding (weights as bf16 pairs, within 2^-17)."""
    import random
    from paper_2608_24063_amd.tensors import DecodeCache
    rng, d = random.Random(units), 64
    caps = [rng.randint(lo, hi) for _ in range(units)]
    a, b = (DecodeCache(1, 1, units, units, d, caps, dev) for _ in range(2))
    gen = torch.Generator(device=dev).manual_seed(units)
    rnd = lambda *s: torch.randn(s, generator=gen, device=dev).to(torch.bfloat16)
    lens = torch.tensor([c - rng.randint(1, 30) for c in caps], dtype=torch.int32)
    a.k_pool.copy_(rnd(*a.k_pool.shape))
    a.v_pool.copy_(rnd(*a.v_pool.shape))
    b.k_pool.copy_(a.k_pool)
    b.v_pool.copy_(a.v_pool)
    for x in (a, b):
        x.len.copy_(lens)
    b.plan()
    k, v, q = rnd(1, 1, units, d), rnd(1, 1, units, d), rnd(1, 1, units, d)
    oa, ob = (torch.full((1, 1, units, d), float("nan"), device=dev) for _ in range(2))
    a.step(k, v, q, oa, d ** -0.5)
    b.step_planned(k, v, q, ob, d ** -0.5)
    torch.cuda.synchronize()
    assert a.len.cpu().tolist() == b.len.cpu().tolist() == [int(n) + 1 for n in lens]
    assert float((oa - ob).abs().max()) <= 2.0 ** -16 * float(a.v_pool.float().abs().max())
