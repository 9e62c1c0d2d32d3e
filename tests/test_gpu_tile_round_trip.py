"""get_tile says what a sweep is launched with, and set_tile gives it back: the
same shape (the library's own rule, compiled for the host), in every precision
and mode, also where a tile of as many pencils would not fit a workgroup."""
import numpy as np
import pytest
import torch

import gpu_cases as GC
from paper_1607_02214_amd import inputs as I
from sweep_plan import plan

pytestmark = pytest.mark.gpu


def _context(n, tracing=0):
    from paper_1607_02214_amd import ppmlr
    return ppmlr.Context([I.uniform_faces(k) for k in n], (1, 1, 1), (1, 1, 1), tracing=tracing)


@pytest.mark.parametrize("n", [(256, 192, 192), (32, 32, 32), (97, 61, 83), (1000, 8, 8), (512, 384, 384), (24, 200, 200)])
@pytest.mark.parametrize("tracing", [0, 1])
def test_what_is_launched_comes_back(n, tracing):
    from paper_1607_02214_amd import ppmlr
    ctx = _context(n, tracing)
    for axis in range(3):
        for dtype, elem in ((ppmlr.F32, 4), (ppmlr.F64, 8)):
            ctx.set_tile(axis, 0)
            if ctx.get_segments(axis, dtype) != 1:
                continue
            want = plan(n, axis, elem, 0, tracing)
            got = ctx.get_tile(axis, dtype)
            assert got == want[0]
            ctx.set_tile(axis, got)                         # and with the segments that are reported
            ctx.set_segments(axis, ctx.get_segments(axis, dtype))
            assert ctx.get_tile(axis, dtype) == got
            assert plan(n, axis, elem, got, tracing) == want
            ctx.set_segments(axis, 0)


def test_other_counts_that_fit_no_workgroup_stay_refused():
    from paper_1607_02214_amd import ppmlr
    ctx = _context((256, 192, 192))
    for axis in range(3):
        auto = {plan((256, 192, 192), axis, e, 0, 0, g)[0] for e, g in ((4, 0), (8, 0), (4, 1))}
        for P in range(1, 70):
            fits = (P * (ctx.n[axis] + 14) + 63) // 64 * 64 <= 1024
            if fits or P in auto:
                ctx.set_tile(axis, P)
            else:
                with pytest.raises(ppmlr.PPMLRError):
                    ctx.set_tile(axis, P)
        ctx.set_tile(axis, max(auto))
        with pytest.raises(ppmlr.PPMLRError):               # 1024 lanes of whole pencils: none march
            ctx.set_tile(axis, 64)
        assert ctx.get_tile(axis) == max(auto)


# a z axis that marches 4 pencils of 248 zones, more than a tile holds: sweeps
# with the count given back are the same, and the harvest mode, which takes
# tiles, still runs
def test_sweeps_after_the_round_trip():
    from paper_1607_02214_amd import ppmlr
    n = (64, 64, 300)
    case = GC.smooth_case(shape=n[::-1], seed=3)
    start = torch.from_numpy(case.U).to("cuda", torch.float32).contiguous()
    auto, back = case.context(), case.context()
    for axis in range(3):
        back.set_tile(axis, auto.get_tile(axis))
    P, C, _, _ = plan(n, 2, 4, 0, 0, 0, 1)
    assert back.get_tile(2) == P and C >= 3 and P * 314 > 1024
    a, b = start.clone(), start.clone()
    auto.advance(a, 2, 0.4)
    back.advance(b, 2, 0.4)
    assert torch.equal(a, b)
    rec = torch.zeros((1000, 28), device="cuda")
    cnt = torch.zeros(1, dtype=torch.int64, device="cuda")
    for ctx, u in ((auto, a), (back, b)):
        ctx.set_harvest(rec, cnt)
        ctx.set_guess(ppmlr.GUESS_HARVEST)
        ctx.advance(u, 1, 0.4)
    assert torch.equal(a, b) and auto.get_tile(2) == back.get_tile(2) and P != back.get_tile(2)


def test_autotune_returns_what_it_keeps():
    from paper_1607_02214_amd import ppmlr
    n = (64, 64, 300)
    case = GC.smooth_case(shape=n[::-1], seed=3)
    u = torch.from_numpy(case.U).to("cuda", torch.float32).contiguous()
    ctx, other = case.context(), case.context()
    tiles = ctx.autotune(u, reps=1)
    for axis in range(3):
        assert tiles[axis] == ctx.get_tile(axis)
        other.set_segments(axis, ctx.get_segments(axis))
        other.set_tile(axis, tiles[axis])
        assert other.get_tile(axis) == tiles[axis]
    v = u.clone()
    ctx.advance(u, 2, 0.4)
    other.advance(v, 2, 0.4)
    assert torch.equal(u, v)
    assert np.all(np.asarray(tiles) > 0)
