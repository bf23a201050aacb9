"""Products large enough for the phased matrix-core kernel (256 x 256 tiles),
at the sizes where its tiling can go wrong: one K stage and an odd number of
them, ragged row and column edges, batches whose tiles all lie in the cut last
round and ones with whole tiles before it, float32, and counted kept lists
(tiles numbered from the device's counts).  Against the oracle, with the bounds
of the fused checks.  Each case says which of its products the phased kernel takes, and that is
asserted: a moved rule does not empty the test."""

import ctypes

import numpy as np
import pytest
import torch

from synth import Workload, make_fusion, make_gate, make_inputs

pytestmark = pytest.mark.gpu

DEV = "cuda"
ES = {"bf16": 2, "f32": 4}


def _phased(dtype, rows, cols, k, batches=1, tile_cols=256):
    """Whether the library runs this product on 256-row tiles."""
    from paper_2607_16305_amd import lookme as lk
    f = lk.load()._ZN6lookme14product_phasedEill
    f.argtypes = [ctypes.c_int, ctypes.c_int64, ctypes.c_int64]
    f.restype = ctypes.c_bool
    return f(1 if dtype == "bf16" else 0, -(-rows // 256) * -(-cols // tile_cols) * batches,
             k * ES[dtype])


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
