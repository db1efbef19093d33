"""Top-k at the edges of its routes: rows of one sweep and of several, binned directly or through the group filter, hit
lists that fit the registers and that do not, rows longer than the position bitmap, clustered heavy keys (the bound
from the group maxima is octaves below rank k), values that leave the histogram's range."""
import numpy as np
import pytest

from paper_2602_14209_amd.workloads import bf16_to_f32, round_to_bf16

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L, k, layout", [
    (16, 16, "plain"), (511, 1, "plain"), (8192, 700, "plain"), (8193, 700, "plain"),
    (16384, 256, "plain"), (16385, 256, "plain"), (16385, 257, "plain"),      # one sweep; the filter's first length; too large k for it
    (20003, 1500, "plain"),                 # two direct sweeps
    (70001, 1000, "plain"),                 # more hits than the registers hold
    (140000, 2048, "plain"),                # the filter's largest k
    (140000, 2049, "plain"),                # several direct sweeps
    (50000, 512, "cluster"),                # all heavy keys in one run: 16 per group
    (50000, 300, "steep"),                  # rank k below 2^-64: radix route
    (270001, 400, "plain"),                 # longer than the bitmap
    (270001, 2049, "plain"),                # ... and k beyond the filter
])
def test_topk_routes(oracle_mod, L, k, layout):
    from gpu_util import Problem, check_index_sets
    rng = np.random.default_rng(L + k)
    B, Hq, Hkv, d = 2, 2, 2, 64
    q = np.zeros((B, Hq, d), np.float32)
    q[:, :, 0] = 8.0
    q[1, :, 1] = 1.0                        # two different rows per head
    K = rng.standard_normal((L, Hkv, d)).astype(np.float32)
    if layout == "cluster":
        K[1000:1000 + k + 40, :, 0] += 12.0
    elif layout == "steep":
        K[:100, :, 0] += 80.0
    K = bf16_to_f32(round_to_bf16(K))
    p = Problem(q, K, K, None, None, k, "bf16")
    print(f"[topk] L={L} k={k} {layout}", flush=True)
    idx, _ = p.select()
    ref = oracle_mod.select(q, K, k)
    # far below 1 neighbouring fp32 results are one rounding apart more often: judge the set on the oracle's own values
    check_index_sets(idx, ref["idx"], ref["alpha32"], L)
