"""The budget of tests/test_kernel_resources.py for the kernels that default calls run
beside k_loglik_grad: the gradient kernels that choose a form per node, the value
kernels, the deep stacks' scan with determinants, and the split units that count
nodes per lane."""
import os
from concurrent.futures import ThreadPoolExecutor

import pytest

from test_kernel_resources import HIPCC, _remarks


def select(lmax, split):
    return f"_ZN2nr13k_grad_selectILi{lmax}ELb{split}EEEvNS_10KernelArgsE"


def value(precision, op, split, few, forms):
    return (f"_ZN2nr7k_valueINS_3{precision}ELi{op}ELb{split}ELb{few}ELb{forms}EE"
            "EvNS_10KernelArgsE")


def scan_select(levels, waves):
    return f"_ZN2nr18k_grad_scan_selectILi{levels}ELi{waves}EEEvNS_10KernelArgsE"


def per_lane(precision, lmax, store, res):
    return (f"_ZN2nr13k_loglik_gradINS_7PerLaneINS_3{precision}EEELi{lmax}ELb{store}ELb0ELb{res}"
            "ELb1EEEvNS_10KernelArgsE")


# (translation unit, defines) -> kernel: (VGPRs, AGPRs, scratch bytes per lane, waves
# per SIMD, LDS bytes)
BUDGET = {
    ("nr_kernels_f64.hip", ()): {
        select(6, 0): (193, 0, 0, 2, 17168),
        select(10, 0): (256, 0, 36, 2, 20240),
        select(10, 1): (253, 0, 0, 2, 20240),
        select(12, 0): (252, 0, 0, 2, 20240),
        select(12, 1): (256, 0, 12, 2, 20240),
        value("F64", 0, 0, 0, 1): (95, 0, 0, 5, 2832),
        value("F64", 1, 1, 0, 1): (100, 0, 0, 4, 2832),
        value("F64", 1, 1, 1, 1): (122, 0, 0, 4, 2832),
        value("F64", 1, 0, 0, 0): (83, 0, 0, 5, 2832),
        per_lane("F64", 4, 1, 0): (254, 4, 0, 1, 18192),
    },
    ("nr_kernels_bucket.hip", ("F64", 14)): {
        select(14, 0): (256, 0, 108, 2, 20240),
        select(14, 1): (256, 0, 116, 2, 20240),
    },
    ("nr_kernels_bucket.hip", ("F64", 20)): {
        select(20, 0): (256, 168, 0, 1, 40720),
        select(20, 1): (256, 174, 0, 1, 40720),
    },
    ("nr_kernels_bucket.hip", ("F64", 36)): {
        select(36, 0): (256, 256, 232, 1, 40720),
        per_lane("F64", 36, 0, 0): (256, 256, 616, 1, 40720),
    },
    ("nr_kernels_f32.hip", ()): {
        value("F32", 0, 0, 0, 0): (29, 0, 0, 8, 2832),
        value("F32", 1, 1, 1, 0): (45, 0, 0, 8, 2832),
        per_lane("F32", 6, 1, 0): (207, 0, 0, 2, 13584),
    },
    ("nr_kernels_bucket.hip", ("F32", 20)): {
        per_lane("F32", 20, 0, 0): (256, 0, 404, 2, 20240),
    },
    ("nr_kernels_bucket.hip", ("F32", 40)): {
        per_lane("F32", 40, 0, 1): (256, 256, 540, 1, 40720),
    },
    ("nr_scan_select.hip", ()): {
        scan_select(1, 1): (147, 0, 0, 3, 2832),
        scan_select(8, 1): (256, 0, 68, 2, 19216),
        scan_select(8, 2): (256, 0, 68, 2, 35824),
        scan_select(8, 4): (256, 0, 96, 2, 68816),
    },
}


@pytest.mark.slow
def test_register_scratch_lds_budget_of_the_default_forms(tmp_path):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    jobs = list(BUDGET)
    with ThreadPoolExecutor(max_workers=min(len(jobs), os.cpu_count() or 4)) as ex:
        found = list(ex.map(lambda j: _remarks(j, str(tmp_path)), jobs))
    bad = []
    for job, rem in zip(jobs, found):
        for name, want in BUDGET[job].items():
            r = rem.get(name)
            assert r is not None, f"{name} not compiled in {job}"
            got = tuple(int(r[f]) for f in ("VGPRs", "AGPRs", "ScratchSize [bytes/lane]",
                                            "Occupancy [waves/SIMD]", "LDS Size [bytes/block]"))
            if got != want:
                bad.append(f"{name}: (VGPR, AGPR, scratch, waves, LDS) = {got}, expected {want}")
    assert not bad, "\n".join(bad)
