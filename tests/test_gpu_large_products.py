"""Products large enough for the phased matrix-core kernel (at least 48 tiles
of 256 x 256), at the sizes where its tiling can go wrong: one K stage and an
odd number of them, ragged row and column edges, batches whose tiles all lie
in the cut last round and ones with whole tiles before it, float32, and
counted kept lists (tiles numbered from the device's counts).  Against the
oracle, with the bounds of the fused checks."""

import numpy as np
import pytest
import torch

from synth import Workload, make_fusion, make_gate, make_inputs

pytestmark = pytest.mark.gpu

DEV = "cuda"

CASES = {
    # name: (workload, d_ff, counted).  Gate/up tiles are 256 x 128 outputs,
    # down tiles 256 x 256.
    # 4.1 row blocks, d_ff 8.5 and d_h 4.03 column tiles, 3 K stages; 90 and
    # 50 tiles, all cut in quarters
    "bf16_ragged_cut": (Workload("lp_a", "bf16", 2100, 2, 64, 64, 20, 60, 192, 1032, 8, 50,
                                 usage="uniform", value_std=1.0), 1088, False),
    # one K stage; 264 tiles in both products: 256 whole, 8 cut
    "bf16_whole_and_cut": (Workload("lp_b", "bf16", 8200, 1, 64, 64, 20, 60, 64, 2048, 4, 100,
                                    usage="uniform", value_std=1.0), 1024, False),
    "f32_ragged": (Workload("lp_c", "f32", 1500, 2, 64, 64, 12, 40, 96, 840, 3, 60,
                            usage="uniform", value_std=1.0), 1056, False),
    # counts near half of the rows, another for each layer
    "bf16_counted_l3": (Workload("lp_d", "bf16", 2300, 3, 64, 64, 20, 60, 128, 776, 8, 50,
                                 usage="uniform", value_std=1.0), 832, True),
}


@pytest.mark.parametrize("name", list(CASES))
def test_fused_injection_on_large_tiles(name):
    from tests.harness import FusedRun, GatedRun, check_fused_run, check_gated_run
    wl, d_ff, counted = CASES[name]
    print(f"[large-products] {name}: {wl} d_ff {d_ff}", flush=True)
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
