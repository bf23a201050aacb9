"""Routing of large batches against the plain arg max on small-integer
queries, keys and biases (every score exact, many exact ties, the lowest scene
wins), at the sizes where the tile kernel can go wrong: fewer scenes than a
key tile, ragged last tiles and row blocks, one and several key tiles a
workgroup, split and unsplit ranges, one K stage and several, and on either
side of the rule that gives many rows over few scenes to the scoring kernel;
and projections of the middle sizes, on either side of the rules that give
them 64 x 64 tiles or one round of 256 x 256 ones."""

import pytest
import torch

pytestmark = pytest.mark.gpu

DEV = "cuda"

CASES = [
    # rows, scenes, key width (bf16), bias
    (4096, 1, 64, False), (4097, 200, 64, False), (4351, 256, 128, False),
    (5000, 257, 64, False), (9001, 700, 192, False), (23040, 1024, 64, False),
    (33000, 1000, 128, False), (40000, 4100, 64, False), (70001, 513, 64, False),
    (4100, 300, 64, True), (23040, 1024, 64, True), (40000, 5000, 64, True),
    # the scoring kernel's shared mode from 65409 rows, the tile kernel below
    (65408, 64, 128, False), (65409, 64, 128, True), (70001, 300, 64, False),
    (66000, 300, 256, True),
]


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("rows,S,d_e,with_bias", CASES)
def test_routing_is_the_lowest_arg_max(rows, S, d_e, with_bias, dtype):
    from paper_2607_16305_amd import lookme as lk
    print(f"[route-tiles] {dtype} rows {rows} S {S} d_e {d_e} bias {with_bias}", flush=True)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator(DEV).manual_seed(rows + S)
    x = torch.randint(-2, 3, (1, rows, d_e), generator=g, device=DEV).to(dt)
    keys = torch.randint(-2, 3, (S, d_e), generator=g, device=DEV).to(dt)
    bias = torch.randint(-4, 5, (S,), generator=g, device=DEV).float() if with_bias else None
    tab = lk.Table(keys, torch.zeros((S, 1, d_e), dtype=dt, device=DEV),
                   torch.zeros((S, 64), dtype=dt, device=DEV), 1, scene_bias=bias)
    q = torch.empty((1, rows, d_e), dtype=dt, device=DEV)
    scene = torch.full((1, rows), -7, dtype=torch.int32, device=DEV)
    for _ in range(2):   # the arrival counters of split ranges are left at zero
        scene.fill_(-7)
        tab.route(x[0], None, q, scene)
        torch.cuda.synchronize()
        for r in range(0, rows, 8192):
            sc = x[0, r:r + 8192].float() @ keys.float().T
            if with_bias:
                sc = sc + bias
            best = sc.max(1, keepdim=True)[0]
            want = torch.where(sc == best, torch.arange(S, device=DEV), S).min(1)[0]
            assert torch.equal(scene[0, r:r + 8192].long(), want), r


@pytest.mark.parametrize("n,layers,d_e,d_in", [(513, 1, 512, 256), (1024, 1, 512, 192),
                                               (1025, 1, 512, 64), (2001, 3, 96, 320),
                                               (700, 2, 608, 128)])
def test_projection_of_middle_sizes(n, layers, d_e, d_in):
    """q = round(x W): bf16 integer inputs whose exact sums are bf16 values."""
    from paper_2607_16305_amd import lookme as lk
    print(f"[route-tiles] projection n {n} layers {layers} d_e {d_e} d_in {d_in}", flush=True)
    g = torch.Generator(DEV).manual_seed(n)
    dt = torch.bfloat16
    x = torch.randint(-1, 2, (n, d_in), generator=g, device=DEV).to(dt)
    wt = torch.randint(-1, 2, (layers, d_e, d_in), generator=g, device=DEV).to(dt)
    keys = torch.randint(-2, 3, (3, d_e), generator=g, device=DEV).to(dt)
    tab = lk.Table(keys, torch.zeros((3, 1, d_e), dtype=dt, device=DEV),
                   torch.zeros((3, 64), dtype=dt, device=DEV), 1)
    q = torch.full((layers, n, d_e), 7.0, dtype=dt, device=DEV)
    scene = torch.empty((layers, n), dtype=torch.int32, device=DEV)
    tab.route(x, wt, q, scene, layers=layers)
    torch.cuda.synchronize()
    want = torch.stack([x.float() @ wt[l].float().T for l in range(layers)])
    assert torch.equal(q, want.to(dt))   # |sums| < 256: bf16 holds them exactly


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("n,layers,d_e,d_in", [
    (7900, 3, 480, 64), (8192, 4, 512, 320),     # 186 and 256 tiles of 256 x 256
    (7930, 4, 480, 192),                         # 248, ragged both ways, 3 (6) K stages
    (4200, 4, 512, 512),                         # 136, K of 1 KiB: bf16 on large tiles
])
def test_projection_of_one_round(n, layers, d_e, d_in, dtype):
    from paper_2607_16305_amd import lookme as lk
    print(f"[route-tiles] projection {dtype} n {n} layers {layers} d_e {d_e} d_in {d_in}",
          flush=True)
    g = torch.Generator(DEV).manual_seed(n)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    x = torch.randint(-1, 2, (n, d_in), generator=g, device=DEV).to(dt)
    wt = torch.randint(-1, 2, (layers, d_e, d_in), generator=g, device=DEV).to(dt)
    keys = torch.randint(-2, 3, (3, d_e), generator=g, device=DEV).to(dt)
    tab = lk.Table(keys, torch.zeros((3, 1, d_e), dtype=dt, device=DEV),
                   torch.zeros((3, 64), dtype=dt, device=DEV), 1)
    q = torch.full((layers, n, d_e), 7.0, dtype=dt, device=DEV)
    scene = torch.empty((layers, n), dtype=torch.int32, device=DEV)
    tab.route(x, wt, q, scene, layers=layers)
    torch.cuda.synchronize()
    for l in range(layers):   # |sums| < 256: bf16 holds them exactly
        assert torch.equal(q[l], (x.float() @ wt[l].float().T).to(dt)), l
