"""Whole pencils swept in chunks by one workgroup (the path of a context without
pencil segments): bit for bit the result of the segmented tile path, whose own
results the oracle tests pin, at the sizes where chunks begin and end."""
import numpy as np
import pytest
import torch

from tests import gpu_cases as GC
from paper_1607_02214_amd import inputs as I

pytestmark = pytest.mark.gpu


def _faces(n, seed):
    rng = np.random.default_rng(seed)
    f = [np.concatenate([[0.0], np.cumsum(rng.uniform(0.7, 1.3, k))]) for k in n]
    return [x / x[-1] for x in f]


def _case(kind, n, tracing):
    nx, ny, nz = n
    if kind == "dipole":
        case = GC.dipole_case(nx=nx, ny=ny, nz=nz)
    elif kind == "blast":
        case = GC.blast_case(n=n)
    else:
        case = GC.Case("smooth", _faces(n, 7), I.random_smooth_state((nz, ny, nx), seed=9))
    case.tracing = tracing
    return case


def _run(case, dtype, segments, tile=0):
    ctx = case.context()
    for axis in range(3):
        n = ctx.n[axis]
        ctx.set_segments(axis, min(segments, n // 7) if segments > 1 else 0)
        ctx.set_tile(axis, tile)
    u = torch.from_numpy(case.U).to("cuda", dtype).contiguous()
    ctx.advance(u, 3, 0.4)                     # both sweep orders, the fused signal speed
    return u, ctx.stats(), ctx.time(u)


# axis sizes around one, two and more chunks of 25 to 121 zones, one zone more
# or less than full chunks, pencil counts that leave the last workgroup short
@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("kind,n", [
    ("smooth", (14, 18, 16)), ("smooth", (43, 69, 93)), ("smooth", (17, 118, 44)),
    ("blast", (50, 21, 68)), ("blast", (171, 19, 67)),
    ("dipole", (64, 43, 28)), ("dipole", (121, 32, 45)),
])
def test_march_equals_segments(kind, n, dtype):
    case = _case(kind, n, 0)
    ref, st, t = _run(case, dtype, 2)
    got, st2, t2 = _run(case, dtype, 1)
    assert torch.equal(got, ref) and st2 == st and t2 == t


@pytest.mark.parametrize("tile", [1, 2, 3, 8])
def test_march_of_given_pencils(tile):
    case = _case("smooth", (40, 53, 61), 0)
    ref, st, _ = _run(case, torch.float32, 3)
    got, st2, _ = _run(case, torch.float32, 1, tile)
    assert torch.equal(got, ref) and st2 == st


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_march_characteristic(dtype):
    case = _case("dipole", (96, 43, 60), 1)
    ref, st, _ = _run(case, dtype, 2)
    got, st2, _ = _run(case, dtype, 1)
    assert torch.equal(got, ref) and st2 == st


def test_march_in_a_graph():
    # nothing of the path allocates or synchronises: captured once, replayed on
    # new states, with eager work between the replays
    case = _case("blast", (40, 33, 30), 0)
    ctx = case.context()
    start = torch.from_numpy(case.U).to("cuda", torch.float32).contiguous()
    dt = ctx.cfl_dt(start, 0.4)
    u = start.clone()
    ctx.sweep(u, dt, 0)                        # loads the kernels
    s = torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        for axis in range(3):
            ctx.sweep(u, dt, axis)
    for k in range(3):
        u.copy_(start * (1.0 + 0.25 * k))
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        ref = start * (1.0 + 0.25 * k)
        for axis in range(3):
            ctx.sweep(ref, dt, axis)
        torch.cuda.synchronize()
        assert torch.equal(u, ref)


# An ensemble's marches: members of one chunk and of many, fewer tiles than
# XCDs, periodic and other ends together, more members than lanes of a wave;
# with one member cut into segments, its axis goes by tiles for all.
@pytest.mark.parametrize("dtype,cut", [(torch.float32, False), (torch.float64, False), (torch.float32, True)])
def test_march_of_an_ensemble(dtype, cut):
    from paper_1607_02214_amd import ppmlr
    kinds = [_case("smooth", (14, 18, 16), 0), _case("blast", (171, 19, 67), 0), _case("smooth", (43, 8, 93), 0),
             _case("dipole", (64, 43, 28), 0)]
    want = [_run(c, dtype, 2) for c in kinds]
    pick = [0] * 35 + [1, 3, 2] + [0] * 29 + [2, 1, 3]
    ctxs = [kinds[k].context() for k in pick]
    us = [torch.from_numpy(kinds[k].U).to("cuda", dtype).contiguous() for k in pick]
    if cut:
        ctxs[36].set_segments(1, 3)
    ppmlr.ensemble_run(ctxs, us, 3, 0.4, block=512)     # (0 is what an autotune of the process left)
    for k, c, u in zip(pick, ctxs, us):
        ref, st, t = want[k]
        assert torch.equal(u, ref) and c.time(u) == t and c.stats() == st


# The learned guess: its list of faces in the rows of the edges, from a few
# faces to every lane (gate 0), against segment tiles of another lane order.
@pytest.mark.parametrize("gate", [0.1, 0.0])
@pytest.mark.parametrize("kind,n", [("blast", (50, 21, 68)), ("blast", (171, 19, 67)), ("smooth", (43, 69, 93))])
def test_march_learned(kind, n, gate):
    from paper_1607_02214_amd import ppmlr
    case = _case(kind, n, 0)
    theta = torch.from_numpy(I.mlp_init(2, scale=0.5)).cuda()
    out = []
    for segments, tile in ((2, 0), (1, 0), (1, 3)):
        ctx = case.context()
        for axis in range(3):
            ctx.set_segments(axis, segments)
            ctx.set_tile(axis, tile)
        ctx.set_guess(ppmlr.GUESS_LEARNED, theta)
        ctx.set_gate(gate, gate)
        u = torch.from_numpy(case.U).to("cuda", torch.float32).contiguous()
        ctx.advance(u, 3, 0.4)
        out.append((u, ctx.stats(), ctx.time(u)))
    assert out[0][1]["guess_faces"] > 0 or gate > 0
    for u, st, t in out[1:]:
        assert torch.equal(u, out[0][0]) and st == out[0][1] and t == out[0][2]


# FP64 rows of 208 slots: two pencils of 95 and 96 zones, and two whose lanes or
# slots are more than those workgroups take
@pytest.mark.parametrize("kind,nx", [("smooth", 169), ("blast", 171), ("smooth", 175), ("smooth", 177)])
def test_march_rows_of_208(kind, nx):
    case = _case(kind, (nx, 9, 11), 0)
    ref, st, t = _run(case, torch.float64, 2)
    got, st2, t2 = _run(case, torch.float64, 1, 2)
    assert torch.equal(got, ref) and st2 == st and t2 == t
