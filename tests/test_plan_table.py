"""Launch-plan selection on the host (no GPU): candidates, pins and the table of measured plans.

Which plan runs a conv pass changes how its sums are tiled and split, never
what they are; the GPU parity of every candidate plan is in
test_gpu_kernels.py.  Here: the candidate list holds the cost model's choice,
pins take effect and come off, invalid pins are refused, and every entry of
the compiled-in table is a candidate of its shape and is what the planner
picks for it.
"""
import os
import re

import pytest

from paper_2101_07968_amd import _lib as D
from paper_2101_07968_amd import nets as PN

INC = os.path.join(os.path.dirname(D.__file__), "csrc", "plan_table.inc")


def _table():
    rows = []
    for line in open(INC):
        m = re.match(r"\s*\{([-\d,\s]+)\},", line)
        if m:
            v = [int(t) for t in m.group(1).split(",")]
            assert len(v) == 14, line
            rows.append((v[0], tuple(v[1:11]), tuple(v[11:14])))
    return rows


SHAPES = [(32, 14, 14, 256, 256, 3, 3, 1, 1, 1), (32, 17, 17, 224, 256, 7, 1, 1, 3, 0),
          (32, 224, 224, 3, 64, 3, 3, 1, 1, 1), (32, 1, 1, 4096, 1000, 1, 1, 1, 0, 0),
          (2, 9, 9, 4, 8, 3, 3, 2, 1, 1)]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("pas", [0, 1, 2])
def test_candidates_hold_the_model_choice_and_pins_apply(shape, pas):
    D.conv_set_plan(shape, pas, -1)
    try:
        model = D.conv_plan_info(shape, pas)
        cands = D.conv_plan_candidates(shape, pas)
        assert model[:3] in cands and model[7] == 0
        assert len(set(cands)) == len(cands)
        for mt, nt, sp in cands:
            assert (mt, nt) in ((128, 128), (128, 64), (64, 128), (64, 64)) and sp >= 1
        for plan in (cands[0], cands[-1]):
            D.conv_set_plan(shape, pas, *plan)
            info = D.conv_plan_info(shape, pas)
            assert info[:3] == plan and info[7] == 2
            assert info[3:7] == model[3:7]   # the GEMM itself does not change
        with pytest.raises(D.DcError):
            D.conv_set_plan(shape, pas, 96, 64, 1)
        with pytest.raises(D.DcError):
            D.conv_set_plan(shape, pas, 64, 64, 10 ** 6)
    finally:
        D.conv_set_plan(shape, pas, 0)


def test_workspace_follows_the_pinned_plan():
    shape = (32, 14, 14, 512, 512, 3, 3, 1, 1, 1)
    import ctypes
    sh = D.ConvShape(*shape)
    try:
        D.conv_set_plan(shape, 0, 128, 128, 1)
        D.conv_set_plan(shape, 1, 128, 128, 1)
        D.conv_set_plan(shape, 2, 128, 128, 1)
        small = D.lib().dc_conv2d_workspace_bytes(ctypes.byref(sh))   # bias-gradient scratch only
        assert small < 32 * 14 * 14 * 512 * 4
        big = max(D.conv_plan_candidates(shape, 0), key=lambda p: p[2])
        D.conv_set_plan(shape, 0, *big)
        assert D.lib().dc_conv2d_workspace_bytes(ctypes.byref(sh)) >= big[2] * 32 * 14 * 14 * 512 * 4
    finally:
        for p in range(3):
            D.conv_set_plan(shape, p, 0)


def test_table_entries_are_candidates_and_are_picked():
    rows = _table()
    keys = set()
    for pas, g, plan in rows:
        assert (pas, g) not in keys, (pas, g)
        keys.add((pas, g))
        assert plan in D.conv_plan_candidates(g, pas), (pas, g, plan)
        info = D.conv_plan_info(g, pas)
        assert info[:3] == plan and info[7] == 1, (pas, g, info)
        # pinning the cost model bypasses the table
        D.conv_set_plan(g, pas, -1)
        try:
            assert D.conv_plan_info(g, pas)[7] == 0
        finally:
            D.conv_set_plan(g, pas, 0)


def test_table_covers_only_workload_shapes():
    """Entries are keyed on the workloads' own geometries at their own batch sizes."""
    known = set()
    for name, wl in PN.WORKLOADS.items():
        ops, hwc, _ = PN.build(name)
        for _i, g, _first in PN.conv_geoms(ops, hwc, wl["batch"]):
            known.add(tuple(g))
    for pas, g, _plan in _table():
        assert g in known, g


RGB = [((32, 224, 224, 3, 64, 3, 3, 1, 1, 1), True), ((32, 299, 299, 3, 32, 3, 3, 2, 0, 0), True),
       ((128, 32, 32, 3, 64, 3, 3, 1, 1, 1), True), ((2, 9, 9, 3, 128, 3, 3, 1, 1, 1), True),
       ((2, 9, 9, 3, 70, 3, 3, 1, 1, 1), False), ((2, 9, 9, 3, 160, 3, 3, 1, 1, 1), False),
       ((2, 9, 9, 3, 16, 3, 3, 1, 1, 1), False), ((32, 224, 224, 3, 64, 7, 7, 2, 3, 3), False),
       ((2, 9, 9, 4, 64, 3, 3, 1, 1, 1), False), ((2, 9, 1, 3, 64, 3, 3, 1, 1, 1), False)]


@pytest.mark.parametrize("shape,direct", RGB, ids=[str(s) for s, _ in RGB])
def test_rgb_layer_takes_the_direct_kernels(shape, direct):
    """Three input channels, a 3 x 3 filter and 32 to 128 output channels in blocks of 32
    (and output rows of at least two pixels): forward and filter gradient report plan source 4,
    the data gradient stays on the implicit GEMM; a pinned plan overrides the direct kernels."""
    src = [D.conv_plan_info(shape, p)[7] for p in range(3)]
    assert (src[0] == 4, src[2] == 4) == (direct, direct), src
    assert src[1] != 4
    if direct:
        mt, nt, sp = D.conv_plan_candidates(shape, 0)[0]
        D.conv_set_plan(shape, 0, mt, nt, sp)
        try:
            assert D.conv_plan_info(shape, 0)[7] == 2
        finally:
            D.conv_set_plan(shape, 0, 0)
        assert D.conv_plan_info(shape, 0)[7] == 4


def test_plan_split_names_the_form():
    """Operands are split from 5e8 flops and a reduction of 96 on, where they are read as float4s; the kernels
    of plan sources 3 and 4 never split."""
    big = (8, 28, 28, 96, 128, 3, 3, 1, 1, 1)            # 1.4e9 flops
    assert [D.conv_plan_split(big, p) for p in range(3)] == [True, True, True]
    assert [D.conv_plan_split((2,) + big[1:], p) for p in range(3)] == [False] * 3   # 3.5e8 flops
    short = (64, 28, 28, 64, 256, 1, 1, 1, 0, 0)         # forward reduction of 64
    assert [D.conv_plan_split(short, p) for p in range(3)] == [False, True, True]
    odd = (8, 28, 28, 96, 126, 3, 3, 1, 1, 1)            # 126 filters: dy is not read as float4s
    assert [D.conv_plan_split(odd, p) for p in range(3)] == [True, False, False]
    assert not D.conv_plan_split((32, 1, 1, 25088, 4096, 1, 1, 1, 0, 0), 1)
    assert not D.conv_plan_split((32, 224, 224, 3, 64, 3, 3, 1, 1, 1), 0)
    with pytest.raises(D.DcError):
        D.conv_plan_split(big, 3)


def test_forward_plans_fit_the_static_scratch():
    """The entry without a workspace argument takes every forward shape whose padded copies (c % 4 != 0) alone
    fit its 64 MiB, under the model's plan: its split-K factor leaves room for them."""
    import random
    rng = random.Random(4)

    def r256(b):
        return (b + 255) // 256 * 256

    shapes = [(59, 15, 15, 181, 1616, 5, 5, 2, 2, 2), (8, 132, 132, 26, 48, 11, 11, 1, 5, 5)]
    while len(shapes) < 4000:
        r = rng.choice([1, 3, 3, 5, 7, 11])
        st = rng.choice([1, 1, 2])
        hw = int(2 ** rng.uniform(2, 8))
        if hw >= r:
            shapes.append((rng.randint(1, 128), hw, hw, int(2 ** rng.uniform(2, 10)), int(2 ** rng.uniform(3, 11)),
                           r, r, st, r // 2, r // 2))
    split = 0
    for g in shapes:
        n, h, w, c, k, r, s, *_ = g
        if n * h * w * max(c, k) >= 2 ** 31:   # refused as a shape
            continue
        _mt, _nt, sp, m, ng, _kg, _ph, src = D.conv_plan_info(g, 0)
        if src > 0:
            continue
        cp = (c + 3) // 4 * 4
        pads = (r256(4 * n * h * w * cp) + r256(4 * k * r * s * cp)) if c % 4 else 0
        sums = r256(4 * sp * m * ng) if sp > 1 else 0
        if D.conv_plan_split(g, 0) and pads <= 64 << 20:
            assert sums + pads <= 64 << 20, (g, sp)
            split += c % 4 != 0 and sp > 1
    assert split > 20


# (pass, shape): relative 2-norm error against 64 bits of the float32 form under the plan that it had, on the
# inputs of perf/cases.py (mean of two seeds)
PRECISE = {
    (1, (4, 16, 16, 8, 16, 3, 3, 1, 1, 1)): 1.514e-7,
    (0, (32, 14, 14, 16, 48, 5, 5, 1, 2, 2)): 1.736e-7,
    (0, (32, 7, 7, 48, 128, 5, 5, 1, 2, 2)): 1.546e-7,
    (0, (32, 17, 17, 192, 224, 1, 7, 1, 0, 3)): 2.285e-7,
    (0, (32, 14, 14, 512, 512, 3, 3, 1, 1, 1)): 2.959e-7,
    (2, (64, 14, 14, 512, 512, 3, 3, 2, 1, 1)): 2.455e-7,
    (2, (32, 14, 14, 128, 256, 3, 3, 1, 1, 1)): 1.500e-7,
    (2, (32, 14, 14, 528, 256, 1, 1, 1, 0, 0)): 1.547e-7,
    (2, (32, 35, 35, 192, 224, 3, 3, 1, 1, 1)): 3.185e-7,
    (2, (32, 71, 71, 192, 192, 3, 3, 2, 0, 0)): 3.305e-7,
    (2, (32, 224, 224, 64, 64, 3, 3, 1, 1, 1)): 5.169e-7,
}


def test_precise_plans_are_picked():
    """Plans kept for their precision come before the table of the fastest ones and are not listed there; the
    tuner that writes the table skips them."""
    from paper_2101_07968_amd import tune
    assert tune.precise_passes() == set(PRECISE)
    listed = {(pas, g) for pas, g, _ in _table()}
    for pas, g in PRECISE:
        assert (pas, g) not in listed
        info = D.conv_plan_info(g, pas)
        assert info[7] == 1 and info[2] > 1 and info[:3] in D.conv_plan_candidates(g, pas), (pas, g, info)
