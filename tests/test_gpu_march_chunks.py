"""Marches of many chunks: every case here is swept in three chunks or more along
its long axis (the shape is asserted), against pencil segments, whose results
the oracle tests pin, bit for bit.  Chunk counts of both parities, last chunks
of all, all but one and fewer of a chunk's zones; pencil counts that leave the
last workgroup short, up to 10 pencils per workgroup."""
import pytest
import torch

import gpu_cases as GC
from paper_1607_02214_amd import inputs as I
from sweep_plan import plan

F32, F64 = torch.float32, torch.float64
# pencils per workgroup (0: chosen), zones along the long axis and across, precision,
# tracing mode.  (FP32 needs more pencils than fit the chip at once as tiles.)
CASES = [(9, 73, (50, 46), F32, 0), (9, 78, (50, 46), F32, 0), (9, 79, (50, 46), F32, 0), (9, 82, (50, 46), F32, 0),
         (0, 250, (64, 64), F32, 0), (8, 93, (19, 17), F64, 0), (10, 72, (19, 17), F64, 0), (10, 88, (19, 17), F64, 0),
         (8, 52, (50, 46), F32, 1), (8, 69, (50, 46), F32, 1), (8, 93, (19, 17), F64, 1), (8, 98, (19, 17), F64, 1)]


def _size(axis, n, across):
    size = list(across)
    size.insert(axis, n)
    return size


def _case(kind, axis, n, across, tracing):
    size = _size(axis, n, [max(k, 28) for k in across] if kind == "dipole" else across)
    if kind == "dipole":
        case = GC.dipole_case(nx=size[0], ny=size[1], nz=size[2])
    elif kind == "blast":
        case = GC.blast_case(n=tuple(size))
    else:
        case = GC.smooth_case(shape=tuple(size[::-1]), seed=n)
    case.tracing = tracing
    return case


def _shape(case, axis, pencils, dtype, learned=0):
    n = [len(f) - 1 for f in case.faces]
    return plan(n, axis, 4 if dtype == F32 else 8, pencils, case.tracing, learned, int(case.bc_hi[axis] == 0))


def test_the_cases_reach_every_kind_of_last_chunk():
    seen = set()
    for pencils, n, across, dtype, tracing in CASES:
        for axis in range(3):
            P, C, L, _ = plan(_size(axis, n, across), axis, 4 if dtype == F32 else 8, pencils, tracing)
            assert C >= 3 and pencils in (0, P)
            last = n + 7 - (C - 1) * L
            seen |= {"odd" if C % 2 else "even", max(last - L, -2)}
    assert seen == {"odd", "even", 0, -1, -2}


def _advance(case, axis, dtype, segments, pencils, prepare=None):
    ctx = case.context()
    for a in range(3):
        if segments > 1:
            ctx.set_segments(a, min(segments, ctx.n[a] // 7))
    ctx.set_tile(axis, pencils)
    if prepare:
        prepare(ctx)
    u = torch.from_numpy(case.U).to("cuda", dtype).contiguous()
    ctx.advance(u, 3, 0.4)                     # both sweep orders, the fused signal speed
    return u, ctx.stats(), ctx.time(u)


@pytest.mark.gpu
@pytest.mark.parametrize("axis", [0, 1, 2])
@pytest.mark.parametrize("k", range(len(CASES)))
def test_march_of_many_chunks(k, axis):
    pencils, n, across, dtype, tracing = CASES[k]
    kind = ("smooth", "blast", "dipole")[(k + axis) % 3]
    case = _case(kind, axis, n, across, tracing)
    shape = _shape(case, axis, pencils, dtype)
    GC.log(f"[march] {kind} axis {axis} n {n} {dtype} tracing {tracing}: pencils, chunks, zones, stride {shape}")
    assert pencils in (0, shape[0]) and shape[1] >= 3
    ref = _advance(case, axis, dtype, 2, 0)
    got = _advance(case, axis, dtype, 1, pencils)
    assert torch.equal(got[0], ref[0]) and got[1] == ref[1] and got[2] == ref[2]


@pytest.mark.gpu
@pytest.mark.parametrize("axis", [0, 1, 2])
@pytest.mark.parametrize("n,gate", [(73, 0.1), (78, 0.0)])
def test_learned_march_of_many_chunks(n, gate, axis):
    from paper_1607_02214_amd import ppmlr
    case = _case("blast", axis, n, (50, 46), 0)
    shape = _shape(case, axis, 9, F32, 1)
    assert shape[0] == 9 and shape[1] >= 3
    theta = torch.from_numpy(I.mlp_init(2, scale=0.5)).cuda()

    def learned(ctx):
        ctx.set_guess(ppmlr.GUESS_LEARNED, theta)
        ctx.set_gate(gate, gate)
    ref = _advance(case, axis, F32, 2, 0, learned)
    got = _advance(case, axis, F32, 1, 9, learned)
    assert ref[1]["guess_faces"] > 0
    assert torch.equal(got[0], ref[0]) and got[1] == ref[1] and got[2] == ref[2]


@pytest.mark.gpu
def test_march_of_many_chunks_in_a_graph():
    # captured once and replayed on new states, with eager work between the replays
    case = _case("blast", 1, 78, (50, 46), 0)
    assert _shape(case, 1, 9, F32)[1] >= 3
    ctx = case.context()
    ctx.set_tile(1, 9)
    start = torch.from_numpy(case.U).to("cuda", F32).contiguous()
    dt = ctx.cfl_dt(start, 0.4)
    u = start.clone()
    ctx.sweep(u, dt, 1)                        # loads the kernel
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=torch.cuda.Stream()):
        for axis in (0, 1, 2, 1):
            ctx.sweep(u, dt, axis)
    for k in range(3):
        u.copy_(start * (1.0 + 0.25 * k))
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        ref = start * (1.0 + 0.25 * k)
        for axis in (0, 1, 2, 1):
            ctx.sweep(ref, dt, axis)
        torch.cuda.synchronize()
        assert torch.equal(u, ref)


# an ensemble's axes: tiles where every member is one chunk (FP32), marches
# where one is not, next to members of one chunk
@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [F32, F64])
def test_ensemble_axes_of_one_chunk_and_of_many(dtype):
    from paper_1607_02214_amd import ppmlr
    cases = [GC.smooth_case(shape=(17, 33, 300), seed=1), GC.blast_case(n=(40, 33, 30)), GC.c1_case(32)]
    for block in (256, 512):
        if block == 256 and max(len(f) for c in cases for f in c.faces) + 13 > block:
            use = cases[1:]
        else:
            use = cases
        ctxs = [c.context() for c in use]
        us = [torch.from_numpy(c.U).to("cuda", dtype).contiguous() for c in use]
        ppmlr.ensemble_run(ctxs, us, 3, 0.4, block=block)
        for c, ctx, u in zip(use, ctxs, us):
            solo = c.context()
            for a in range(3):
                solo.set_segments(a, 2)
            w = torch.from_numpy(c.U).to("cuda", dtype).contiguous()
            solo.advance(w, 3, 0.4)
            assert torch.equal(u, w) and ctx.time(u) == solo.time(w)
