"""The static checks of tests/test_code_objects.py for the batched kernel of few sequences (csrc/sparse_few_bf16.hip)."""
from test_code_objects import _code_object, _demangle, _early_uses, _sgpr_hazards


def test_few_sequences_kernels(tmp_path):
    meta, kernels = _code_object(str(tmp_path), "sparse_few_bf16")
    assert len(meta) == 4
    for sym, m in meta.items():
        name, ins = _demangle(sym), kernels[sym]
        assert m["scratch"] == 0 and m["vspill"] == 0 and m["vgpr"] + m["agpr"] <= 256 and m["lds"] <= 160 * 1024, (name, m)
        assert not any(x.startswith("s_swappc") for x in ins), name
        assert not _sgpr_hazards(ins) and not _early_uses(ins), (name, _early_uses(ins)[:3])
        # hand-counted LDS waits: no scalar load between the first fragment read and the last MFMA
        first, last = next(i for i, s in enumerate(ins) if s.startswith("ds_read_b128")), max(i for i, s in enumerate(ins) if s.startswith("v_mfma"))
        assert not [s for s in ins[first:last] if s.startswith(("s_load", "s_buffer_load", "s_mem"))], name
