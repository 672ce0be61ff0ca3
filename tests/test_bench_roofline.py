"""bench.py's roofline block (host only): the bytes of the launches that a timed
call makes, not of its steps, which may share launches on D2Q9."""
import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

import bench  # noqa: E402
from paper_1904_00866_amd import elbm  # noqa: E402


def _block(box, storage, mode, ms, steps, arith="fp64", traffic=None):
    return bench.roofline(elbm, box, storage, mode, arith, elbm.DIAG_COUNTS, ms, steps, traffic)


def test_single_steps():
    """512^3 FP32: 28.99 GB in 5 ms; counter traffic passed on."""
    r = _block(("d3q27", (512,) * 3), "f32", "closed", 5.0, 200, traffic=29)
    assert r["steps_per_launch"] == 1 and r["traffic"] == 29
    assert r["algorithmic_bytes_per_launch"] == 2 * 27 * 4 * 512 ** 3
    assert r["achieved"] == pytest.approx(28.99e9 / 5e-3 / 1e9, rel=1e-3)
    assert r["kernel"] == "k_step<3,Storef32,closed,fp64>"


def test_steps_that_share_launches():
    """FP64 LBGK 4096^2 at 171 us a step: three steps a launch and the recording one
    alone move 20 / 3 + 1 launches' worth, 4.9 TB/s, not the 14.1 of 20."""
    r = _block(("d2q9", (4096, 4096, 1)), "f64", "bgk", 0.171, 20, traffic=1)
    launches = elbm.batch_launches([elbm.make_config("d2q9", 4096, 4096, storage="f64",
                                                     mode="bgk", diag=elbm.DIAG_COUNTS)], [20])
    assert launches == 8 and r["steps_per_launch"] == 2.5
    assert r["traffic"] is None and r["kernel"].startswith("k_fused<")
    assert r["achieved"] == pytest.approx(2 * 9 * 8 * 4096 ** 2 * 8 / (20 * 0.171e-3) / 1e9, rel=1e-4)
    assert r["frac"] < 1


def test_the_hash_covers_every_step_kernel_that_is_timed():
    assert {"elbm_step_d2.hip", "elbm_step_d3.hip", "elbm_step_fused.hip",
            "elbm_step_impl.hpp"} <= set(bench.STEP_KERNEL_SOURCES)
