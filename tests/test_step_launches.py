"""How many kernel launches steps take (host only: no device work)."""
import pytest

from paper_1904_00866_amd import elbm


def launches(boxes, steps, lattice="d2q9", **kw):
    cfgs = [elbm.make_config(lattice, *b, **kw) for b in boxes]
    return elbm.batch_launches(cfgs, steps)


def test_one_launch_per_step_where_nothing_is_fused():
    """Lattices, modes and entropies without a fused kernel; a step that records."""
    for lattice, box in (("d1q3", (640,)), ("d3q27", (8, 8, 8)), ("d3q19", (8, 8, 8))):
        assert launches([box], [7], lattice) == 7
    for kw in (dict(mode="newton"), dict(mode="secant"), dict(entropy="burg")):
        assert launches([(64, 64)], [7], **kw) == 7
    assert launches([(64, 64)], [1], diag=elbm.DIAG_COUNTS) == 1
    assert launches([(64, 64)], [0]) == 0 and launches([], []) == 0


def test_fused_steps_share_launches():
    """64^2: five steps a launch (six would have to come in pairs); the recording
    last step is a launch of its own."""
    assert launches([(64, 64)], [10], storage="f64") == 2
    assert launches([(64, 64)], [11], storage="f64", diag=elbm.DIAG_COUNTS) == 3
    assert launches([(64, 64)], [12], storage="f64") == 2  # six and six


def test_batch_of_different_lengths():
    """Simulations that record and end at different steps; more than sixteen
    share no launch."""
    d = elbm.DIAG_COUNTS
    assert launches([(8, 8, 8)] * 3, [2, 5, 0], "d3q27", diag=d) == 5
    assert launches([(8, 8, 8)] * 17, [4] * 17, "d3q27") == 8


@pytest.mark.parametrize("n,kw", [(64, dict(storage="f32")),
                                  (128, dict(storage="f16dev", fp64="mixed")),
                                  (128, dict(storage="f32", fp64="mixed")),
                                  (128, dict(storage="f64"))])
def test_groups_of_sixteen_choose_for_themselves(n, kw):
    """Sixteen simulations share a launch: more of them change no group's choice."""
    one = launches([(n, n)] * 16, [60] * 16, **kw)
    assert launches([(n, n)] * 64, [60] * 64, **kw) == 4 * one
    rest = launches([(n, n)] * 8, [60] * 8, **kw)
    assert launches([(n, n)] * 40, [60] * 40, **kw) == 2 * one + rest


THIN = [((1, 100000), dict(storage="f64")), ((2, 500000), dict(storage="f64")),
        ((4, 100000), dict(storage="f64")), ((16, 8000), dict(storage="f64")),
        ((32, 8192), dict(storage="f64")), ((1, 100000), dict(storage="f64", mode="bgk")),
        ((2, 500000), dict(mode="bgk")), ((8, 200000), dict(mode="bgk")),
        ((32, 8192), dict(mode="bgk")), ((8, 200000), dict(fp64="fp32")),
        ((1, 100000), dict(fp64="mixed")), ((2, 500000), dict(fp64="mixed")),
        ((16, 100000), dict(fp64="mixed")), ((32, 32768), dict(fp64="mixed")),
        ((128, 3000), dict(fp64="mixed")), ((2, 500000), dict()), ((32, 32768), dict()),
        ((32768, 32), dict()), ((64, 65536), dict()), ((64, 65536), dict(fp64="mixed")),
        ((1, 12000), dict()), ((4, 11000), dict()),
        ((64, 65536), dict(storage="f16dev", mode="bgk")),
        ((64, 65536), dict(storage="f16dev", fp64="mixed")),
        ((1, 100000), dict(storage="f16dev", fp64="mixed")),
        ((2, 500000), dict(storage="f32dev", fp64="mixed"))]


@pytest.mark.parametrize("box,kw", THIN)
def test_thin_boxes_take_single_steps(box, kw):
    """Boxes of which a region holds little more than a few sites: fused, its other
    sites would be computed for nothing (up to 15 times the time of single steps)."""
    assert launches([box], [60], **dict(dict(storage="f32"), **kw)) == 60


SQUARE = [((1001, 601), 20, dict(storage="f64", mode="bgk")),
          ((2048, 2048), 30, dict(storage="f64")), ((4096, 4096), 30, dict(storage="f64")),
          ((1024, 1024), 20, dict(mode="bgk")), ((1001, 601), 30, dict(fp64="fp32")),
          ((640, 640), 30, dict(fp64="mixed")), ((4096, 4096), 30, dict(fp64="mixed")),
          ((365, 365), 20, dict(fp64="mixed")), ((512, 512), 30, dict(fp64="mixed")),
          ((901, 901), 30, dict()), ((2048, 2048), 30, dict()), ((1001, 601), 60, dict()),
          ((4096, 4096), 60, dict()), ((2048, 2048), 30, dict(storage="f16dev", mode="bgk")),
          ((1450, 1447), 30, dict(storage="f16dev", fp64="mixed")),
          ((620, 620), 30, dict(storage="f16dev", fp64="mixed")),
          ((64, 8192), 20, dict(storage="f64", mode="bgk")),
          ((64, 65536), 30, dict(storage="f64")),
          ((64, 4096), 30, dict(storage="f16dev", fp64="mixed")), ((2, 6000), 20, dict()),
          ((1, 2000), 12, dict()), ((8, 9000), 20, dict())]


@pytest.mark.parametrize("box,want,kw", SQUARE)
def test_other_boxes_fuse(box, want, kw):
    """Near-square boxes on either side of each type's lines, and thin ones where
    the regions are worth it."""
    assert launches([box], [60], **dict(dict(storage="f32"), **kw)) == want


def test_invalid_batches():
    cfg = elbm.make_config("d2q9", 64, 64)
    with pytest.raises(elbm.ElbmError, match="nsteps < 0"):
        elbm.batch_launches([cfg], [-1])
    with pytest.raises(elbm.ElbmError, match="differ"):
        elbm.batch_launches([cfg, elbm.make_config("d2q9", 64, 64, storage="f64")], [1, 1])
    bad = elbm.make_config("d2q9", 64, 64)
    bad.reserved = 1
    with pytest.raises(elbm.ElbmError, match="reserved"):
        elbm.batch_launches([bad], [1])
