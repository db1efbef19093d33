"""Batched sparse step with few sequences: two and four row tiles per workgroup (four and two key parts), last
iterations that leave key parts without a tile, fewer tiles than key parts, index windows that are refilled; and fewer still, which the single-sequence kernel takes with a sequence dimension (channels in
four, two parts and unsplit, one and more passes)."""
import zlib

import numpy as np
import pytest

from paper_2602_14209_amd.workloads import Workload, make_layer

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("case", [
    # name, n_seq, Hq, Hkv, d, L, B, k
    ("f1", 2, 2, 2, 128, 40, 1, 1),          # a single key position per part, most parts empty
    ("f2", 3, 4, 2, 64, 500, 8, 24),         # k + B = 32: exactly one tile
    ("f3", 2, 14, 2, 64, 900, 5, 257),       # 35 rows, odd tile count
    ("f4", 2, 28, 4, 128, 2600, 32, 2300),   # entries beyond one index window, one row tile per workgroup
    ("f5", 5, 28, 4, 128, 700, 32, 300),     # two row tiles
    ("f6", 12, 28, 4, 128, 700, 31, 301),    # four row tiles, the last one of a unit half empty
    ("f7", 9, 32, 8, 64, 2400, 16, 2200),    # d = 64, refilled windows, two row tiles
    ("f8", 32, 8, 8, 128, 300, 3, 100),      # 256 units of three rows
    ("f9", 32, 8, 8, 128, 700, 3, 600),      # the same with more keys: the kernel for many units
    ("s1", 3, 3, 1, 128, 900, 7, 633),       # one KV head; channels in four parts, one full pass
    ("s2", 5, 6, 3, 64, 1100, 8, 1016),      # 15 units of one row tile, two channel parts, sixteen wavefronts
    ("s3", 9, 14, 2, 128, 700, 16, 300),     # 18 units x 7 row tiles: two channel parts
    ("s4", 6, 40, 5, 128, 800, 16, 700),     # 30 units x 8 row tiles: channels unsplit, two passes
    ("s5", 30, 8, 8, 64, 300, 5, 120),       # 240 units
    ("s6", 4, 16, 8, 128, 1500, 9, 1015),    # 32 units x 2 row tiles, four channel parts, sixteen wavefronts of four tiles
])
def test_few_sequences(oracle_mod, case):
    import torch
    import paper_2602_14209_amd.binding as mb
    from gpu_util import check_out, to_device
    name, n, Hq, Hkv, d, L, B, k = case
    w = Workload(name, "bf16", Hq=Hq, Hkv=Hkv, d=d, L=L, B=B, ks=(k,), T=2, heavy_frac=0.02, heavy_scale=3.0)
    rng = np.random.default_rng(zlib.crc32(name.encode()))
    xs = [make_layer(w, 100 + i, steps=2) for i in range(n)]
    idx = np.stack([np.stack([np.sort(rng.choice(L, k, replace=False)) for _ in range(Hkv)]) for _ in range(n)]).astype(np.int32)
    stack = lambda f: to_device(np.stack([f(x) for x in xs]), "bf16")
    q, kc, vc = stack(lambda x: x["q"][1]), stack(lambda x: x["k_cache"]), stack(lambda x: x["v_cache"])
    kb, vb = stack(lambda x: x["k_blk"][1]), stack(lambda x: x["v_blk"][1])
    out = torch.full((n, B, Hq, d), float("nan"), device="cuda")
    lse = torch.full((n, B, Hq), float("nan"), device="cuda")
    s = mb.make_shape(B, Hq, Hkv, d, L, k, "bf16")
    print(f"[parity] few sequences {case}", flush=True)
    for blk in (True, False):
        mb.check(mb.mage_sparse_attn_batched(s, n, q, kc, vc, torch.from_numpy(idx).cuda(), kb if blk else None, vb if blk else None, out, lse))
        torch.cuda.synchronize()
        for i, x in enumerate(xs):
            o_ref, l_ref = oracle_mod.sparse_attn(x["q"][1], x["k_cache"], x["v_cache"], idx[i], x["k_blk"][1] if blk else None,
                                                  x["v_blk"][1] if blk else None)
            check_out(out[i].cpu().numpy(), o_ref, lse[i].cpu().numpy(), l_ref, "bf16")
