"""The fp64 re-score of near-ties at rank k: several key splits with references of their own, fp32 inputs, more than 256
query rows (two passes over the rows), and page rows, where the queries are split by sign."""
import numpy as np
import pytest
import torch

from paper_2602_14209_amd.workloads import bf16_to_f32, round_to_bf16

pytestmark = pytest.mark.gpu


def _plant(oracle_mod, q, K, k, h, rng, bf16):
    """Replace a key of head h by a slightly changed copy of another one, so that the two are at ranks k and k+1 with a gap of
    1.5e-6 .. 3.5e-6."""
    def gap(b, new):
        trial = K.copy()
        trial[b, h] = new
        s = np.sort(oracle_mod.select(q, trial, k)["alpha"][h])[::-1]
        return trial, (s[k - 1] - s[k]) / s[k - 1]

    order = np.argsort(-oracle_mod.select(q, K, k)["alpha"][h], kind="stable")
    pairs = ((b, a) for b in order[k + 5:k + 60] for a in order[k - 8:k + 3])      # (the change of key b moves the others a little)
    b, a = next((b, a) for b, a in pairs if gap(b, K[a, h])[1] < 1e-12)
    for _ in range(200):
        if bf16:                                     # one unit in the last place of a few channels
            new = K[a, h].copy()
            c = rng.choice(K.shape[2], 3, replace=False)
            new[c] *= 1 + rng.choice([-1, 1], 3) * 2.0 ** -8
            new = bf16_to_f32(round_to_bf16(new.astype(np.float32)))
        else:
            new = (K[a, h] * (1 + rng.uniform(-1, 1) * 10 ** rng.uniform(-6, -4))).astype(np.float32)
        trial, g = gap(b, new)
        if 1.5e-6 < g < 3.5e-6:
            return trial
    return None


@pytest.mark.parametrize("seed", [0, 1, 2])
@pytest.mark.parametrize("kind, Hq, Hkv, d, B, L, k", [
    ("bf16", 8, 2, 64, 8, 4200, 70),         # several splits
    ("f32", 4, 2, 64, 4, 1500, 50),
    ("f32", 20, 1, 128, 14, 300, 40),        # 280 rows
    ("pages", 8, 2, 128, 8, 900, 60),        # pages of one position: the estimate is the exact score
])
def test_near_ties(oracle_mod, kind, Hq, Hkv, d, B, L, k, seed):
    from gpu_util import Problem, check_index_sets, to_device
    rng = np.random.default_rng(100 * seed + k)
    dtype = "f32" if kind == "f32" else "bf16"
    rnd = (lambda x: x.astype(np.float32)) if dtype == "f32" else (lambda x: bf16_to_f32(round_to_bf16(x.astype(np.float32))))
    q = rng.standard_normal((1, Hq, d)) + 0.1 * rng.standard_normal((B, Hq, d))
    if kind == "pages" or dtype == "bf16":
        q[:, :, ::4] *= 2.0 ** -7                    # channels whose change moves a score by little
    q, K = rnd(q), rnd(rng.standard_normal((L, Hkv, d)))
    planted = 0
    for h in range(Hkv):
        got = _plant(oracle_mod, q, K, k, h, rng, dtype == "bf16")
        if got is not None:
            K, planted = got, planted + 1
    print(f"[near-tie] {kind} d={d} L={L} seed={seed}: {planted} planted", flush=True)
    assert planted >= 1
    ref = oracle_mod.select(q, K, k)
    if kind == "pages":
        import paper_2602_14209_amd.binding as mb
        shape = mb.make_shape(B, Hq, Hkv, d, L, k, dtype)
        kd, qd = to_device(K, dtype), to_device(q, dtype)
        summ = torch.zeros((L, Hkv, 2, d), dtype=kd.dtype, device="cuda")
        mb.check(mb.mage_page_summary(shape, 1, kd, summ))
        ws = torch.empty(mb.mage_quest_workspace_bytes(shape, 1), dtype=torch.uint8, device="cuda")
        idx = torch.full((Hkv, k), -1, dtype=torch.int32, device="cuda")
        mb.check(mb.mage_quest_select(shape, 1, qd, summ, idx, None, ws))
        torch.cuda.synchronize()
        check_index_sets(idx.cpu().numpy(), ref["idx"], ref["alpha32"], L)
        return
    p = Problem(q, K, rnd(rng.standard_normal((L, Hkv, d))), None, None, k, dtype)
    check_index_sets(p.select()[0], ref["idx"], ref["alpha32"], L)
    check_index_sets(p.step1()[2], ref["idx"], ref["alpha32"], L)
