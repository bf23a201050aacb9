"""The top-n_keep select, the gate compaction and the multi-scale mix at the
sizes where their splits can go wrong, against plain definitions: one wave's
groups and ragged ones, the LDS caches' limits and the uncached form, all keys
equal (more than the direct ranking holds), keys that share their leading
digits, and rows of one, two and more chunks a thread."""

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


@pytest.mark.parametrize("values", ["spread", "equal", "near", "few"])
@pytest.mark.parametrize("n", [1, 63, 64, 65, 1000, 1025, 4096, 4097, 32768, 32769, 70001])
def test_select_is_the_stable_top(n, values):
    """One nonzero element a row, a small integer or power of two, so that
    every square is exact: kept = the n_keep largest, lowest token on ties."""
    print(f"[select-mix] select n {n} {values}", flush=True)
    rng = np.random.default_rng(n)
    x = {"spread": np.exp2(rng.integers(-20, 20, n)) * rng.integers(1, 100, n),
         "equal": np.full(n, 3.0), "near": 2048.0 + rng.integers(0, 300, n),
         "few": rng.integers(0, 3, n)}[values].astype(np.float64)
    crit = torch.zeros((2, n, 4), device=DEV)
    crit[0, :, 1] = torch.tensor(x, device=DEV, dtype=torch.float32)
    crit[1, :, 2] = torch.tensor(x[::-1].copy(), device=DEV, dtype=torch.float32)
    tab = _table()
    for keep in sorted({1, max(1, n // 3), n}):
        kept = torch.full((2, keep), -7, dtype=torch.int32, device=DEV)
        tab.select(crit, kept, keep, layers=2)
        torch.cuda.synchronize()
        for l, v in enumerate((x, x[::-1])):
            sq = (v.astype(np.float32) ** 2).astype(np.float32)
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
                                                ("bf16", 576, 7, 8), ("f32", 1920, 8, 5)])
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
