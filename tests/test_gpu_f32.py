"""fp32 kernels at the edges of their tiling: 16-row tiles (one or two per workgroup), 16-key tiles dealt to key
slices and splits, 32-key units of the column sums; gathered, dense and fused entry points against the oracle."""
import zlib

import numpy as np
import pytest

from paper_2602_14209_amd.workloads import Workload, make_layer

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("case", [
    # name, Hq, Hkv, d, L, B, k
    ("e1", 1, 1, 64, 1, 1, 1),               # one row, one key
    ("e2", 4, 1, 64, 15, 4, 15),             # 16 rows, a ragged first tile, fewer tiles than key slices
    ("e3", 17, 1, 128, 17, 1, 3),            # 17 rows: two row tiles
    ("e4", 6, 2, 128, 129, 11, 128),         # 33 rows: three row tiles
    ("e5", 5, 1, 64, 2049, 13, 700),         # 65 rows: five row tiles; gathered keys in several splits
    ("e6", 8, 4, 128, 3001, 16, 531),        # several splits everywhere
    ("e7", 2, 2, 64, 33, 7, 16),             # block tiles only in some slices
    ("e8", 24, 8, 64, 1400, 11, 700),        # 33 rows and more than one round of workgroups: two row tiles each, the last one empty
    ("e9", 4, 1, 64, 1000, 4, 380),          # gathered: one round per split, the last split with the block tile only
])
def test_f32_edges(oracle_mod, case):
    from gpu_util import Problem, check_alpha, check_index_sets, check_out
    name, Hq, Hkv, d, L, B, k = case
    w = Workload(name, "f32", Hq=Hq, Hkv=Hkv, d=d, L=L, B=B, ks=(k,), T=2, heavy_frac=0.02, heavy_scale=3.0)
    seed = zlib.crc32(name.encode()) % 1000 + 5
    x = make_layer(w, seed, steps=2)
    print(f"[parity] f32 {case}", flush=True)
    p = Problem(x["q"][0], x["k_cache"], x["v_cache"], x["k_blk"][0], x["v_blk"][0], k, "f32")
    ref = oracle_mod.select(x["q"][0], x["k_cache"], k)
    o_ref, l_ref = oracle_mod.exact_attn(x["q"][0], x["k_cache"], x["v_cache"], x["k_blk"][0], x["v_blk"][0])
    idx, alpha = p.select()
    check_alpha(alpha, ref["alpha32"])
    check_index_sets(idx, ref["idx"], ref["alpha32"], L)
    check_out(*_pair(p.exact(), (o_ref, l_ref)), "f32")
    p.out.fill_(float("nan")); p.idx.fill_(-1); p.alpha.fill_(float("nan"))
    o, l, idx, alpha = p.step1()
    check_out(o, o_ref, l, l_ref, "f32")
    check_alpha(alpha, ref["alpha32"])
    check_index_sets(idx, ref["idx"], ref["alpha32"], L)
    np.testing.assert_allclose(p.block_probs().reshape(Hkv, Hq // Hkv, L).mean(axis=1), ref["alpha"], rtol=2e-4, atol=1e-9)
    p.set_q(x["q"][1]); p.set_blk(x["k_blk"][1], x["v_blk"][1])
    ref_sp = oracle_mod.sparse_attn(x["q"][1], x["k_cache"], x["v_cache"], ref["idx"], x["k_blk"][1], x["v_blk"][1])
    check_out(*_pair(p.sparse(ref["idx"]), ref_sp), "f32")


def _pair(got, want):
    return got[0], want[0], got[1], want[1]
