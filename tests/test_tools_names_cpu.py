"""Profiles of kernels that take the mapping as an argument: their names carry no
variant, so a sweep's counters are matched by launch order."""
import json

import pytest

import paper_2511_02132_amd as pa
from paper_2511_02132_amd import rocprof_counters as rc
from paper_2511_02132_amd import sweep

NS = "void attn::(anonymous namespace)::"
MIXED = NS + "attn_fwd_mixed_kernel<64, 56, true>(attn::KernelArgs, int)"
GRADS = NS + "attn_bwd_grads_kernel<true>(attn::BwdArgs, int, int)"
PP = NS + "attn_fwd_pp_kernel<true, 2, 1>(attn::KernelArgs)"


def _run(tmp_path, kernels, variants):
    with open(tmp_path / "run_counter_collection.csv", "w") as f:
        f.write("Dispatch_Id,Kernel_Name,Grid_Size,Counter_Name,Counter_Value\n")
        for i, (name, hit) in enumerate(kernels):
            f.write('%d,"%s",131072,TCC_HIT,%r\n' % (i, name, hit))
            f.write('%d,"%s",131072,TCC_MISS,%r\n' % (i, name, 100.0 - hit))
    cfg = {"B": 1, "Hq": 128, "Hkv": 128, "S": 2048}
    man = tmp_path / "m.json"
    man.write_text(json.dumps([{"config": cfg, "variant": v} for v in variants]))
    got = sweep.l2_by_launch(str(tmp_path), str(man))
    return [got[(1, 128, 128, 2048, v)] for v in variants]


def test_variants_by_launch_order(tmp_path):
    names = [n for n, _ in pa.variants(True, 56)][:3]
    assert _run(tmp_path, list(zip([MIXED] * 3, (10.0, 20.0, 30.0))), names) == \
        [pytest.approx(x) for x in (0.1, 0.2, 0.3)]


def test_gradients_in_one_launch(tmp_path):
    names = [pa.variant_name(2), pa.variant_name(0x12)]
    launches = [(PP, 1.0), (GRADS, 40.0), (GRADS, 50.0)]   # the forward is left out
    assert _run(tmp_path, launches, names) == [pytest.approx(0.4), pytest.approx(0.5)]
    assert rc.kernel_of(GRADS) == "dK/dV and dQ"


def test_a_named_variant_is_still_checked(tmp_path):
    with pytest.raises(ValueError):
        _run(tmp_path, [(PP, 1.0)], [pa.variant_name(2)])
