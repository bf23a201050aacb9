"""Products large enough for the phased matrix-core kernel (256 x 256 tiles),
at the sizes where its tiling can go wrong: one K stage and an odd number of
them, ragged row and column edges, batches whose tiles all lie in the cut last
round and ones with whole tiles before it, float32, every epilogue, and
counted kept lists (tiles numbered from the device's counts), down to the few
live tiles that run on 64 x 64 ones.  Against the oracle with the bounds of
its checks, or against float64 with a bound from the roundings on the way.
Each case says which of its products the phased kernel takes, and that is
asserted: a moved rule does not empty the test."""

import ctypes

import numpy as np
import pytest
import torch

from synth import (Workload, make_fusion, make_gate, make_inputs, make_propagation,
                   make_relevance)

pytestmark = pytest.mark.gpu

DEV = "cuda"
ES = {"bf16": 2, "f32": 4}


def _phased(dtype, rows, cols, k, batches=1, tile_cols=256):
    """Whether the library runs this product on 256-row tiles."""
    from paper_2607_16305_amd import lookme as lk
    f = lk.load()._ZN6lookme14product_phasedEillill
    f.argtypes = [ctypes.c_int, ctypes.c_int64, ctypes.c_int64, ctypes.c_int, ctypes.c_int64,
                  ctypes.c_int64]
    f.restype = ctypes.c_bool
    return f(1 if dtype == "bf16" else 0, rows, cols, tile_cols, batches, k * ES[dtype])


CASES = {
    # name: (workload, d_ff, counted, (gate/up, down) on the phased kernel).
    # Gate/up tiles are 256 x 128 outputs, down tiles 256 x 256.
    # 4.1 row blocks, d_h 4.03 column tiles; gate/up's 90 tiles have 3 K stages
    # and run on 64 x 64 ones, down's 50 are all cut in quarters
    "bf16_ragged_cut": (Workload("lp_a", "bf16", 2100, 2, 64, 64, 20, 60, 192, 1032, 8, 50,
                                 usage="uniform", value_std=1.0), 1088, False, (False, True)),
    # the same edges with 9 K stages: 90 tiles of d_ff 8.5 column tiles, all cut
    "bf16_ragged_cut_k9": (Workload("lp_e", "bf16", 2100, 2, 64, 64, 20, 60, 576, 1032, 8, 50,
                                    usage="uniform", value_std=1.0), 1088, False, (True, True)),
    # one K stage; 264 tiles in both products: 256 whole, 8 cut
    "bf16_whole_and_cut": (Workload("lp_b", "bf16", 8200, 1, 64, 64, 20, 60, 64, 2048, 4, 100,
                                    usage="uniform", value_std=1.0), 1024, False, (True, True)),
    # 72 and 32 tiles: 64 x 64 ones
    "f32_ragged": (Workload("lp_c", "f32", 1500, 2, 64, 64, 12, 40, 96, 840, 3, 60,
                            usage="uniform", value_std=1.0), 1056, False, (False, False)),
    # 252 and 224 whole tiles, ragged both ways, 3 and 33 K stages
    "f32_whole": (Workload("lp_f", "f32", 7000, 2, 64, 64, 12, 40, 96, 2000, 3, 50,
                           usage="uniform", value_std=1.0), 1056, False, (True, True)),
    # 300 tiles in both: 256 whole, 44 cut
    "f32_whole_and_cut": (Workload("lp_g", "f32", 7500, 2, 64, 64, 12, 40, 64, 2400, 3, 50,
                                   usage="uniform", value_std=1.0), 1248, False, (True, True)),
    # counts near half of the rows, another for each layer
    "bf16_counted_l3": (Workload("lp_d", "bf16", 2300, 3, 64, 64, 20, 60, 128, 776, 8, 50,
                                 usage="uniform", value_std=1.0), 832, True, (True, True)),
    "f32_counted_l2": (Workload("lp_h", "f32", 4000, 2, 64, 64, 20, 60, 96, 1800, 8, 50,
                                usage="uniform", value_std=1.0), 1056, True, (True, True)),
}


@pytest.mark.parametrize("name", list(CASES))
def test_fused_injection_on_large_tiles(name):
    from tests.harness import FusedRun, GatedRun, check_fused_run, check_gated_run
    wl, d_ff, counted, phased = CASES[name]
    print(f"[large-products] {name}: {wl} d_ff {d_ff}", flush=True)
    cap = wl.n_tokens if counted else wl.n_keep
    assert (_phased(wl.dtype, cap, d_ff, wl.d_v, wl.layers, 128),
            _phased(wl.dtype, cap, wl.d_h, d_ff, wl.layers)) == phased
    inp = make_inputs(wl, seed=21, device=DEV)
    fus = make_fusion(wl, 21, d_ff, device=DEV)
    if counted:
        r = GatedRun(inp, make_gate(wl, 21, device=DEV), "fused", fus, None).run()
        last = int(r.count[0]) - 1
    else:
        r = FusedRun(inp, fus).run()
        last = r.kept.shape[1] - 1
    # the first and last kept rows (the edges of the row blocks) and a sample
    kept0 = r.kept[0].cpu().numpy()
    toks = np.unique(np.concatenate([
        np.random.default_rng(21).choice(wl.n_tokens, 40, replace=False), kept0[:10],
        kept0[max(0, last - 9):last + 1], kept0[250:262]]))
    rep = (check_gated_run if counted else check_fused_run)(r, tokens=toks)
    assert rep.ok, str(rep)


def test_propagation_on_large_tiles():
    """The propagation product with its residual: 1500 rows of 2048 columns
    and a ragged last tile, 48 tiles."""
    from tests.harness import PropagatedRun, check_propagated_run
    wl = Workload("lp_p", "bf16", 3000, 2, 64, 64, 20, 60, 1984, 1992, 4, 50, usage="uniform",
                  value_std=1.0)
    print(f"[large-products] propagation: {wl}", flush=True)
    assert _phased("bf16", wl.n_keep, wl.d_v, wl.d_v)
    inp = make_inputs(wl, seed=23, device=DEV)
    fus = make_fusion(wl, 23, 512, device=DEV)
    r = PropagatedRun(inp, fus, make_propagation(wl, 23, 1, device=DEV)).run()
    kept0 = r.kept[0].cpu().numpy()
    rep = check_propagated_run(r, tokens=np.unique(np.concatenate([kept0[:8], kept0[-8:],
                                                                   kept0[252:260]])))
    assert rep.ok, str(rep)


@pytest.mark.parametrize("dtype,n,hidden,P", [("bf16", 2100, 1024, 1496),
                                              ("f32", 6200, 352, 2200)])
def test_relevance_logits_on_large_tiles(dtype, n, hidden, P):
    """The relevance MLP's second layer where it is a product of its own (a
    width that the fused top-k does not take), with its bias, ragged edges."""
    from tests.harness import RelevanceRun, check_relevance_run
    wl = Workload("lp_r", dtype, n, 1, 64, 64, 9, P, 64, 64, 8, 10, usage="uniform")
    print(f"[large-products] relevance: {wl} hidden {hidden}", flush=True)
    assert _phased(dtype, n, P, hidden)
    inp = make_inputs(wl, seed=25, device=DEV)
    r = RelevanceRun(inp, make_relevance(wl, 25, hidden, device=DEV)).run()
    toks = np.unique(np.concatenate([np.arange(8), np.arange(n - 8, n), np.arange(250, 262),
                                     np.random.default_rng(25).choice(n, 60, replace=False)]))
    rep = check_relevance_run(r, tokens=toks)
    assert rep.ok, str(rep)


def _table(dtype, S, P, d_v, k, g):
    from paper_2607_16305_amd import lookme as lk
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    rn = lambda *s, std=1.0: (torch.randn(s, generator=g, device=DEV) * std).to(dt)
    return lk.Table(rn(S, 64), rn(S, P, 64), rn(S * P, d_v), k), rn, dt


def _lookup(M, n, S, P, k, g):
    scene = torch.randint(0, S, (M, n), generator=g, device=DEV, dtype=torch.int32)
    prim = torch.randint(0, P, (M, n, k), generator=g, device=DEV, dtype=torch.int32)
    w = torch.softmax(torch.randn((M, n, k), generator=g, device=DEV), 2)
    return scene, prim, w


def _kept(n, opens, g):
    kept = torch.full((len(opens), n), -1, dtype=torch.int32, device=DEV)
    for l, m in enumerate(opens):
        kept[l, :m] = torch.randperm(n, generator=g, device=DEV)[:m].sort()[0].int()
    return kept, torch.tensor(opens, dtype=torch.int32, device=DEV)


# 8400 rows of capacity take the phased kernel in both types; live tiles of 256
# x 256 and 64 x 64: 7 and 25 (a CU each), 21 and 275 (pairs, the last half
# empty), 63
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("m", [0, 1, 30, 700, 2100])
def test_counted_queries_of_any_count(dtype, m):
    """Gated multi-scale injection of m of 8400 rows against float64: q =
    round(H[kept] W) decides the weights alpha.  u: half the spacing of the
    stored type, or for float32 the bound K 2^-24 of a sum.  q errs by u (|H|
    |W|), the scores by that times |R| / sqrt(d_v) and R's own rounding, alpha
    by twice the score's error, and the stored row by u once more."""
    n, d_v, d_h, M, S, P, k = 8400, 1544, 1600, 2, 6, 50, 4
    print(f"[large-products] counted queries {dtype} {m}", flush=True)
    assert _phased(dtype, n, d_v, d_h)
    g = torch.Generator(DEV).manual_seed(m + 1)
    tab, rn, dt = _table(dtype, S, P, d_v, k, g)
    w_he = rn(d_v, d_h, std=d_h ** -0.5)
    tab.set_multiscale(M, w_he)
    scene, prim, w = _lookup(M, n, S // M, P, k, g)
    kept, count = _kept(n, [m], g)
    h0 = rn(n, d_h)
    h = h0.clone()
    tab.inject_multiscale_gated(kept, count, scene, prim, w, h)
    torch.cuda.synchronize()
    t = kept[0, :m].long()
    V, H, W = tab.tensors[2].double(), h0.double(), w_he.double()
    R = torch.stack([(w[s, t].double()[:, :, None] *
                      V[(scene[s, t].long() + s * (S // M))[:, None] * P + prim[s, t].long()]
                      ).sum(1).to(dt).double() for s in range(M)])
    q = (H[t] @ W.T).to(dt).double()
    a = torch.softmax((q[None] * R).sum(2) / d_v ** 0.5, 0)
    want = H.clone()
    want[t, :d_v] += (a[:, :, None] * R).sum(0)
    other = torch.ones(n, dtype=torch.bool, device=DEV)
    other[t] = False
    assert torch.equal(h[other], h0[other])
    if m == 0:
        return
    u = 2.0 ** -8 if dtype == "bf16" else d_h * 2.0 ** -24
    eq = u * (H[t].abs() @ W.abs().T)
    es = (eq[None] * R.abs() + u * q.abs()[None] * R.abs()).sum(2).max(0)[0] / d_v ** 0.5
    tol = (2 * es)[:, None] * R.abs().sum(0) + u * (want[t, :d_v].abs() + R.abs().sum(0))
    err = (h[t, :d_v].double() - want[t, :d_v]).abs()
    assert bool((err <= tol).all()), float((err / tol).max())
    # the bound is loose in each row; over all rows the error is a rounding's
    assert float(err.norm() / want[t, :d_v].norm()) <= (2.0 ** -8 if dtype == "bf16" else 1e-5)


@pytest.mark.parametrize("dtype,opens", [
    # live 64 x 64 tiles: gate/up 34 and down 33, with an empty layer
    ("f32", [40, 0]), ("f32", [1, 65]),
    # 9 row blocks of 64: 306 and 297, pairs
    ("f32", [300, 250]), ("bf16", [60]), ("bf16", [560]),
])
def test_counted_fusion_of_few_rows(dtype, opens):
    """Gated fused injection where a launch chosen for 8400 rows finds few:
    against float64 by the roundings on the way (R, U and the stored row; u as
    above), and over all rows within one rounding."""
    n, d_v, d_ff, d_h, S, P, k = 8400, 1088, 1088, 2080, 6, 50, 4
    L = len(opens)
    print(f"[large-products] counted fusion {dtype} {opens}", flush=True)
    assert _phased(dtype, n, d_ff, d_v, L, 128) and _phased(dtype, n, d_h, d_ff, L)
    g = torch.Generator(DEV).manual_seed(sum(opens))
    tab, rn, dt = _table(dtype, S, P, d_v, k, g)
    wg, wu = rn(L, d_ff, d_v, std=d_v ** -0.5), rn(L, d_ff, d_v, std=d_v ** -0.5)
    wd = rn(L, d_h, d_ff, std=d_ff ** -0.5)
    tab.set_fusion(wg, wu, wd)
    scene, prim, w = _lookup(L, n, S, P, k, g)
    kept, count = _kept(n, opens, g)
    h0 = rn(L, n, d_h)
    h = h0.clone()
    tab.inject_fused_gated(kept, count, scene, prim, w, h, layers=L)
    torch.cuda.synchronize()
    V = tab.tensors[2].double()
    u = 2.0 ** -8 if dtype == "bf16" else d_v * 2.0 ** -24
    for l, m in enumerate(opens):
        t = kept[l, :m].long()
        other = torch.ones(n, dtype=torch.bool, device=DEV)
        other[t] = False
        assert torch.equal(h[l][other], h0[l][other])
        if m == 0:
            continue
        R = (w[l, t].double()[:, :, None] *
             V[scene[l, t].long()[:, None] * P + prim[l, t].long()]).sum(1).to(dt).double()
        G, U, D = wg[l].double(), wu[l].double(), wd[l].double()
        gate, up = R @ G.T, R @ U.T
        act = gate / (1 + torch.exp(-gate))
        inner = (act * up).to(dt).double()
        want = h0[l, t].double() + inner @ D.T
        # |silu'| < 1.1
        eg, eu = u * (R.abs() @ G.abs().T), u * (R.abs() @ U.abs().T)
        ei = 2 * (1.1 * eg * up.abs() + act.abs() * eu) + u * inner.abs()
        tol = ei @ D.abs().T + u * (want.abs() + inner.abs() @ D.abs().T)
        err = (h[l, t].double() - want).abs()
        assert bool((err <= tol).all()), float((err / tol).max())
        assert float(err.norm() / want.norm()) <= (2.0 ** -8 if dtype == "bf16" else 1e-5)
