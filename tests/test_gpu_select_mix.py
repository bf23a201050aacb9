"""The top-n_keep select, the gate compaction and the multi-scale mix at the
sizes where their splits can go wrong, against plain definitions: one wave's
groups and ragged ones, the LDS caches' limits and the uncached forms (through
lookme_select, which may run beside other kernels, and lookme_inject), all keys
equal (more than the direct ranking holds), keys that share their leading
digits, as many of them as the ranking holds and one more, and rows of one, two
and more chunks a thread."""

import numpy as np
import pytest
import torch

from synth import Workload, make_inputs, make_multiscale

pytestmark = pytest.mark.gpu

DEV = "cuda"


def _table():
    from paper_2607_16305_amd import lookme as lk
    wl = Workload("sel", "f32", 16, 1, 64, 64, 2, 8, 16, 16, 2, 50)
    inp = make_inputs(wl, seed=2, device=DEV)
    return lk.Table(inp["scene_keys"], inp["prim_keys"], inp["values"], 2)


def _injected(tab, crit, keep):
    """The kept set that lookme_inject writes (its own form of the select)."""
    layers, n = crit.shape[:2]
    kept = torch.full((layers, keep), -7, dtype=torch.int32, device=DEV)
    scene = torch.zeros((layers, n), dtype=torch.int32, device=DEV)
    prim = torch.zeros((layers, n, 2), dtype=torch.int32, device=DEV)
    w = torch.zeros((layers, n, 2), device=DEV)
    hidden = torch.zeros((layers, n, 16), device=DEV)
    tab.inject(crit, scene, prim, w, hidden, keep, kept, layers=layers)
    return kept


def _check_kept(crit, squares, keeps):
    """kept of both forms = the n_keep largest, lowest token on ties.
    squares [layers, n]: the exact sums of squares."""
    tab = _table()
    for keep in keeps:
        kept = torch.full((crit.shape[0], keep), -7, dtype=torch.int32, device=DEV)
        tab.select(crit, kept, keep, layers=crit.shape[0])
        other = _injected(tab, crit, keep)
        torch.cuda.synchronize()
        for l, sq in enumerate(squares):
            want = np.sort(np.argsort(-sq, kind="stable")[:keep])
            assert np.array_equal(kept[l].cpu().numpy(), want), (keep, l)
            assert np.array_equal(other[l].cpu().numpy(), want), ("inject", keep, l)


@pytest.mark.parametrize("values", ["spread", "equal", "near", "few"])
@pytest.mark.parametrize("n", [1, 63, 64, 65, 1000, 1025, 4096, 4097, 8192, 8193, 32767, 32768,
                               32769, 70001])
def test_select_is_the_stable_top(n, values):
    """One nonzero element a row, a small integer or power of two, so that
    every square is exact."""
    print(f"[select-mix] select n {n} {values}", flush=True)
    rng = np.random.default_rng(n)
    x = {"spread": np.exp2(rng.integers(-20, 20, n)) * rng.integers(1, 100, n),
         "equal": np.full(n, 3.0), "near": 2048.0 + rng.integers(0, 300, n),
         "few": rng.integers(0, 3, n)}[values].astype(np.float64)
    crit = torch.zeros((2, n, 4), device=DEV)
    crit[0, :, 1] = torch.tensor(x, device=DEV, dtype=torch.float32)
    crit[1, :, 2] = torch.tensor(x[::-1].copy(), device=DEV, dtype=torch.float32)
    _check_kept(crit, [(v.astype(np.float32) ** 2).astype(np.float32) for v in (x, x[::-1])],
                sorted({1, max(1, n // 3), n}))


@pytest.mark.parametrize("n,layers,width", [(5000, 2, 64), (9000, 2, 64), (40000, 2, 64),
                                            (9000, 4, 1024)])
@pytest.mark.parametrize("listed", [1, 255, 256, 257, 700])
def test_select_among_keys_that_share_their_digits(n, layers, width, listed):
    """`listed` keys 1 + m^2 2^-22 with m < 180 share their 16 leading bits;
    the boundary falls among them, the others are well below and above.  Many
    layers of wide keys (a projection of several rounds) run lookme_select in
    lookme_inject's form."""
    print(f"[select-mix] listed {listed} of {n}, {layers} layers", flush=True)
    rng = np.random.default_rng(n + listed)
    m = rng.integers(0, 180, (layers, n))
    at = np.argsort(rng.random((layers, n)), axis=1)
    big = n // 4
    one, two = np.ones((layers, n)), m * 2.0 ** -11
    for l in range(layers):
        one[l, at[l, listed:listed + big]], two[l, at[l, listed:listed + big]] = 2.0, 0.0
        one[l, at[l, listed + big:]], two[l, at[l, listed + big:]] = 0.5, 0.0
    crit = torch.zeros((layers, n, 4), device=DEV)
    crit[:, :, 0] = torch.tensor(one, device=DEV)
    crit[:, :, 3] = torch.tensor(two, device=DEV)
    squares = [(a * a + b * b).astype(np.float32) for a, b in zip(one, two)]
    keeps = sorted({big + 1, big + listed // 2 + 1, big + listed})
    if width == 64:
        return _check_kept(crit, squares, keeps)
    from paper_2607_16305_amd import lookme as lk
    zeros = lambda *s: torch.zeros(s, dtype=torch.bfloat16, device=DEV)
    tab = lk.Table(zeros(2, width), zeros(2, 4, width), zeros(8, 16), 2)
    wide = crit.to(torch.bfloat16)   # m 2^-11 and the others are bf16 values
    wide = torch.cat([wide, torch.zeros_like(wide)], 2)
    for keep in keeps:
        kept = torch.full((layers, keep), -7, dtype=torch.int32, device=DEV)
        tab.select(wide, kept, keep, layers=layers)
        torch.cuda.synchronize()
        for l, sq in enumerate(squares):
            want = np.sort(np.argsort(-sq, kind="stable")[:keep])
            assert np.array_equal(kept[l].cpu().numpy(), want), (keep, l)


@pytest.mark.parametrize("n", [1, 64, 1023, 4096, 65536, 65601, 140000])
def test_gate_lists_the_open_rows(n):
    print(f"[select-mix] gate n {n}", flush=True)
    delta = torch.randn((2, n, 4), device=DEV, generator=torch.Generator(DEV).manual_seed(n))
    delta[:, ::5] = 0.0
    w = torch.zeros((2, 4), device=DEV)
    w[0, 0], w[1, 3] = 1.0, -1.0
    kept = torch.full((2, n), -7, dtype=torch.int32, device=DEV)
    count = torch.full((2,), -7, dtype=torch.int32, device=DEV)
    _table().gate(delta, w, kept, count, layers=2)
    torch.cuda.synchronize()
    for l, z in enumerate((delta[0, :, 0], -delta[1, :, 3])):
        want = torch.nonzero(z > 0)[:, 0].to(torch.int32)
        assert int(count[l]) == want.numel()
        assert torch.equal(kept[l, :want.numel()], want)
        assert torch.all(kept[l, want.numel():] == -1)


@pytest.mark.parametrize("dtype,d_v,scales,k", [("bf16", 64, 1, 4), ("bf16", 2112, 3, 7),
                                                ("bf16", 4160, 2, 12), ("f32", 1056, 5, 17),
                                                ("f32", 2080, 8, 3), ("bf16", 3584, 8, 8),
                                                ("bf16", 576, 7, 8), ("f32", 1920, 8, 5),
                                                ("bf16", 512, 8, 16), ("bf16", 1344, 3, 24),
                                                ("bf16", 2048, 2, 20), ("bf16", 2112, 2, 24)])
def test_multiscale_mix_against_float64(dtype, d_v, scales, k):
    """H + sum_m alpha_m R^m from the library's own picks.  bf16: the stored
    value's rounding (2^-9 of it), an R^m that rounds the other way (2^-8 of
    it) and what such a q or R^m moves the weights by (of the same size
    again) stay below 2^-7 of the largest |H| + |R|; float32: 1e-5 of it.  A
    scale with an index out of range contributes zero and is counted."""
    from paper_2607_16305_amd import lookme as lk
    from tests.harness import MultiScaleRun
    print(f"[select-mix] mix {dtype} {d_v} {scales} {k}", flush=True)
    wl = Workload("mix", dtype, 150, 1, 64, 64, 4 * scales, 24, d_v, d_v + 64, k, 40,
                  value_std=1.0)
    inp = make_inputs(wl, seed=5, device=DEV)
    r = MultiScaleRun(inp, make_multiscale(wl, 5, scales, device=DEV)).run()
    kept = torch.arange(0, 150, 3, dtype=torch.int32, device=DEV)
    prim = r.prim.clone()
    prim[0, 6, 0] = 24                       # token 6, scale 0: out of range
    lk.lookme_index_errors()
    h = r.h_in.clone()
    r.table.inject_multiscale(kept, r.scene, prim, r.w, h, kept.numel())
    torch.cuda.synchronize()
    assert lk.lookme_index_errors() == 1
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    P, Sm = r.P, r.S // r.M
    H, V = r.h_in.double(), inp["values"].double()
    t = kept.long()
    R = []
    for m in range(scales):
        rows = (r.scene[m, t].long() + m * Sm)[:, None] * P + prim[m, t].long().clamp(max=P - 1)
        Rm = (r.w[m, t].double()[:, :, None] * V[rows]).sum(1).to(dt).double()
        if m == 0:
            Rm[2] = 0                        # token 6 is the third kept row
        R.append(Rm)
    R = torch.stack(R)
    q = (H[t] @ r.ms["w_he_t"].double().T).to(dt).double()
    a = torch.softmax((q[None] * R).sum(2) / d_v ** 0.5, 0)
    want = H.clone()
    want[t, :d_v] += (a[:, :, None] * R).sum(0)
    mag = H.abs().max() + R.abs().max()
    tol = (2.0 ** -7 if dtype == "bf16" else 1e-5) * mag
    assert float((h.double() - want).abs().max()) <= float(tol)
    other = torch.ones(150, dtype=torch.bool, device=DEV)
    other[t] = False
    assert torch.equal(h[other], r.h_in[other])
