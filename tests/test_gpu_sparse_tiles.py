"""Sparse step at the key counts where the number of tiles per wavefront, of wavefronts and of passes changes."""
import zlib

import numpy as np
import pytest

from paper_2602_14209_amd.workloads import Workload, make_layer

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("keys", [128, 129, 256, 257, 384, 385, 640, 641, 768, 769, 1024, 1025, 1280, 1281, 1536, 1537])
@pytest.mark.parametrize("Hq, Hkv, d, B", [(14, 2, 128, 8), (8, 2, 64, 16), (40, 20, 128, 56)])      # channels in four, two parts, unsplit
def test_key_counts(oracle_mod, keys, Hq, Hkv, d, B):
    from gpu_util import Problem, check_out
    k = keys - B
    w = Workload("tiles", "bf16", Hq=Hq, Hkv=Hkv, d=d, L=k + 50, B=B, ks=(k,), T=2, heavy_frac=0.02, heavy_scale=3.0)
    seed = zlib.crc32(f"{keys}{d}{B}".encode()) % 1000
    x = make_layer(w, seed, steps=2)
    rng = np.random.default_rng(seed)
    idx = np.stack([np.sort(rng.choice(w.L, k, replace=False)) for _ in range(Hkv)]).astype(np.int32)
    print(f"[parity] sparse, {keys} key positions, d={d} B={B}", flush=True)
    p = Problem(x["q"][1], x["k_cache"], x["v_cache"], x["k_blk"][1], x["v_blk"][1], k, "bf16")
    o, l = p.sparse(idx)
    o_ref, l_ref = oracle_mod.sparse_attn(x["q"][1], x["k_cache"], x["v_cache"], idx, x["k_blk"][1], x["v_blk"][1])
    check_out(o, o_ref, l, l_ref, "bf16")
