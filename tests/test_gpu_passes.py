"""Fused passes of split steps beyond what the forward comparisons show: that
the fused path is the one that runs (kernels of a captured call), transposed
steps bitwise the transposed sweeps in two and more dimensions, and the time of
a pass at displacements of many cells against the sweeps it replaces."""
import ctypes

import numpy as np
import pytest

from gpu_helpers import have_gpu
from test_gpu_strang import _bits, _seq, _state

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sl():
    if not have_gpu():
        pytest.skip("no HIP device")
    import paper_1603_07008_amd as sl
    sl.lib()
    return sl


def _kernels(stream, fn):
    """Nodes of the graph that fn's launches on `stream` capture to."""
    hip = ctypes.CDLL("libamdhip64.so")
    graph, n = ctypes.c_void_p(), ctypes.c_size_t()
    st = ctypes.c_void_p(stream.cuda_stream)
    assert hip.hipStreamBeginCapture(st, 1) == 0           # thread-local
    try:
        fn()
    finally:
        assert hip.hipStreamEndCapture(st, ctypes.byref(graph)) == 0
    assert hip.hipGraphGetNodes(graph, None, ctypes.byref(n)) == 0
    assert hip.hipGraphDestroy(graph) == 0
    return n.value


@pytest.mark.parametrize("ns,steps,fused,single", [((75, 41), 5, 1, 3), ((64,), 7, None, 1)])
@pytest.mark.parametrize("adjoint", [False, True])
def test_fused_launches(sl, ns, steps, fused, single, adjoint):
    """X V X: one launch a step instead of three; a 1D plan's steps: one launch
    in all (after the tables' one)."""
    import torch
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        plan = sl.Plan(ns, 2, "fp32", stream=stream.cuda_stream)
        a, b = plan.empty_state(), plan.empty_state()
        seq = _seq(ns, 2, 1, 3.0, 0.4, 1) if len(ns) > 1 else \
            [(0, 0, torch.full((1,), 0.3, dtype=torch.float64, device="cuda"))]
        run = plan.split_steps_adjoint if adjoint else plan.split_steps
        stream.synchronize()
        for fuse, want in ((True, 1 if fused is None else steps * fused), (False, steps * single)):
            plan.set_fusion(fuse)
            assert _kernels(stream, lambda: run(seq, steps, a, b)) == want + 1
        stream.synchronize()
        plan.close()


@pytest.mark.parametrize("ns,k,tier,fused", [
    ((4, 1024, 64), 2, "fp32", False), ((8, 512, 64), 3, "bf16", False),
    ((16, 64, 256), 3, "fp32", False), ((30, 100, 64), 3, "bf16", True),
    ((16, 64, 256), 2, "fp64", True), ((8, 500), 3, "bf16", True), ((4, 4096), 2, "fp32", True)])
def test_x_v_x_of_short_lines(sl, ns, k, tier, fused):
    """Full-chip grids of lines that fill few lanes run sweep by sweep (4 x 1024 x
    64: a pass took 2.5 times the sweeps); the others in one pass."""
    import torch
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        plan = sl.Plan(ns, k, tier, stream=stream.cuda_stream)
        a, b = plan.empty_state(), plan.empty_state()
        seq = _seq(ns, 2, 1, 3.0, 0.4, 1)
        stream.synchronize()
        n = _kernels(stream, lambda: plan.split_steps(seq, 2, a, b))
        assert n == (3 if fused else 7)
        stream.synchronize()
        plan.close()


def _adjoint_both(sl, ns, k, tier, seq, nsteps, ndouble=1):
    import torch
    plan = sl.Plan(ns, k, tier, ndouble=ndouble)
    st = _state(plan, 11)
    a = tuple(t.clone() for t in st)
    b = tuple(torch.full_like(t, float("nan")) for t in st)
    got = (a, b)[plan.split_steps_adjoint(seq, nsteps, a, b)]
    buf, cur = [tuple(t.clone() for t in st), plan.empty_state()], 0
    for _ in range(nsteps):
        for dim, mask, shift in reversed(seq):
            plan.advect_dim_adjoint(dim, shift, mask, *buf[cur], *buf[1 - cur])
            cur = 1 - cur
    torch.cuda.synchronize()
    for x, y in zip(got, buf[cur]):
        assert torch.equal(_bits(x), _bits(y)), (ns, k, tier)
    plan.close()


@pytest.mark.parametrize("tier", ["fp64", "fp32", "bf16", "fp16"])
@pytest.mark.parametrize("k", [1, 2, 3])
@pytest.mark.parametrize("amp", [0.4, 25.0])
def test_transposed_x_v_x(sl, tier, k, amp):
    """One and two V shifts to a wave, and a shift of its own per column."""
    ns = (75, 41)
    _adjoint_both(sl, ns, k, tier, _seq(ns, 2, 1, 9.0, amp, k), 3, ndouble=k % 2)


@pytest.mark.parametrize("ns,mask_x,mask_v", [((1, 9), 2, 1), ((130, 1), 2, 1), ((66, 9), 0, 0),
                                              ((21, 6, 5), 0b110, 0b101),
                                              ((10, 6, 4, 3), 0b1010, 0b0101)])
def test_transposed_masks_and_higher_dimensions(sl, ns, mask_x, mask_v):
    for tier, k in (("fp32", 1), ("fp64", 2)):
        _adjoint_both(sl, ns, k, tier, _seq(ns, mask_x, mask_v, 3.0, 40.0, 5), 2)


@pytest.mark.parametrize("n0", [1, 2, 63, 64, 65, 200])
@pytest.mark.parametrize("tier,k", [("fp32", 3), ("fp16", 2), ("bf16", 3)])
def test_spread_shifts(sl, n0, tier, k):
    """Smooth fields of many cells, whose waves hold runs of equal shifts, over
    lines of less than one tile to several; odd and even numbers of rows."""
    import torch
    for n1 in (1, 5, 50):
        ns = (n0, n1)
        seq = _seq(ns, 2, 1, 1.5 * n0, 0.0, n0)
        u = torch.arange(n0, dtype=torch.float64, device="cuda") / n0
        seq[1] = (1, 1, 11.3 * torch.sin(2 * np.pi * u + 0.3))
        plan = sl.Plan(ns, k, tier)
        st = _state(plan, 5)
        out = []
        for fuse in (False, True):
            plan.set_fusion(fuse)
            a = tuple(t.clone() for t in st)
            b = tuple(torch.full_like(t, float("nan")) for t in st)
            out.append((a, b)[plan.split_steps(seq, 2, a, b)])
        torch.cuda.synchronize()
        for x, y in zip(*out):
            assert torch.equal(_bits(x), _bits(y)), ns
        plan.close()


def _time(plan, seq, nsteps, a, b):
    import torch
    plan.split_steps(seq, nsteps, a, b)
    best = float("inf")
    for _ in range(5):
        e0, e1 = torch.cuda.Event(True), torch.cuda.Event(True)
        e0.record()
        plan.split_steps(seq, nsteps, a, b)
        e1.record()
        torch.cuda.synchronize()
        best = min(best, e0.elapsed_time(e1))
    return best


@pytest.mark.parametrize("k,tier", [(2, "fp32"), (3, "bf16"), (3, "fp64")])
@pytest.mark.parametrize("amp", [3.0, 10.0, 30.0])
def test_x_v_x_of_many_cells_costs_no_more_than_the_sweeps(sl, k, tier, amp):
    """Measured ratios 0.5 to 1.2 (1.2: k = 3 at 30 cells); evaluating each
    distinct shift of a wave by itself took 1.5 to 9 times the sweeps."""
    import torch
    ns = (512, 512)
    plan = sl.Plan(ns, k, tier)
    a, b = plan.empty_state(), plan.empty_state()
    for t in (*a, *b):
        t.zero_()
    u = torch.arange(512, dtype=torch.float64, device="cuda") / 512
    sx = 4.0 * (2.0 * u - 1.0)
    seq = [(0, 2, sx), (1, 1, amp * torch.sin(2 * np.pi * u)), (0, 2, sx)]
    t = []
    for fuse in (False, True):
        plan.set_fusion(fuse)
        t.append(_time(plan, seq, 10, a, b))
    assert t[1] <= 1.4 * t[0], t
    plan.close()


@pytest.mark.parametrize("graph", [False, True])
def test_batch_with_problems_outside_the_pass(sl, graph):
    """A batch that fills the chip: its problems of short lines run sweep by sweep
    beside the others' passes, bitwise each problem's sweeps."""
    import torch
    from paper_1603_07008_amd.batch import Batch
    grids = [((8, 9000), 3), ((130, 3000), 2), ((6, 4000), 1), ((40, 50), 3), ((10, 37), 2)]
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        seqs = [_seq(ns, 2, 1, 3.0, 2.5, i) for i, (ns, _) in enumerate(grids)]
        plans = [sl.Plan(ns, k, "fp32", stream=stream.cuda_stream) for ns, k in grids]
        states = [_state(p, i) for i, p in enumerate(plans)]
        b = Batch([g[0] for g in grids], [g[1] for g in grids], "fp32", stream=stream.cuda_stream)
        s0 = [tuple(t.clone() for t in st) for st in states]
        s1 = [tuple(torch.full_like(t, float("nan")) for t in st) for st in states]
        b.bind(s0, s1)
        b.set_sequence([(seqs[0][q][0], [(s[q][1], s[q][2]) for s in seqs]) for q in range(3)])
        res = b.run(3, use_graph=graph)
        for i, plan in enumerate(plans):
            plan.set_fusion(False)
            x = tuple(t.clone() for t in states[i])
            y = plan.empty_state()
            want = (x, y)[plan.split_steps(seqs[i], 3, x, y)]
            stream.synchronize()
            for got, ref in zip((s0, s1)[res][i], want):
                assert torch.equal(_bits(got), _bits(ref)), grids[i]
            plan.close()
        b.close()


def _pair_both(sl, ns, k, tier, d, mask, shifts, ndouble=1, nsteps=1, fused=True):
    import torch
    plan = sl.Plan(ns, k, tier, ndouble=ndouble)
    st = _state(plan, 7)
    seq = [(d, mask, shifts[0]), (d + 1, mask, shifts[1])]
    out = []
    for fuse in (False, True):
        plan.set_fusion(fuse)
        a = tuple(t.clone() for t in st)
        b = tuple(torch.full_like(t, float("nan")) for t in st)
        plan.timing_enable(True)
        out.append((a, b)[plan.split_steps(seq, nsteps, a, b)])
        assert plan.timing_read(-2)[0] == (2 - (fuse and fused)) * nsteps
        plan.timing_enable(False)
    torch.cuda.synchronize()
    for x, y in zip(*out):
        assert torch.equal(_bits(x), _bits(y)), (ns, k, tier)
    plan.close()


def _uniform(n, amp, seed):
    import torch
    return torch.from_numpy(np.random.default_rng(seed).uniform(-amp, amp, n)).cuda()


@pytest.mark.parametrize("tier", ["fp64", "fp32", "bf16", "fp16"])
@pytest.mark.parametrize("k", [1, 2, 3])
@pytest.mark.parametrize("amp", [1.5, 30.0])
def test_pair_of_spread_shifts(sl, tier, k, amp):
    """Shifts of four values over a wave and of any, in states that always take
    the fused pass (each lane its own rows) and in larger ones, which run the
    sweeps one by one through lines in LDS where the shifts are spread."""
    for ndouble in (0, 1):
        for ns in ((60, 11, 13), (48 if k < 3 else 64, 170, 175 if k == 1 else 90)):
            _pair_both(sl, ns, k, tier, 1, 1, [_uniform(ns[0], amp, 1), _uniform(ns[0], amp, 2)],
                       ndouble=ndouble, nsteps=2)


@pytest.mark.parametrize("ns,d,mask,k,tier,fused", [
    ((304, 50, 59), 1, 1, 2, "bf16", True),            # 128 columns a tile, the last short
    ((300, 50, 59), 1, 1, 2, "bf16", False),           # rows across cache lines, in the caches
    ((300, 5, 59), 1, 1, 2, "bf16", True), ((300, 170, 59), 1, 1, 2, "bf16", True),
    ((64, 3, 600), 1, 1, 3, "fp64", True),             # 8 columns a tile
    ((64, 3, 700), 1, 1, 3, "fp64", False),            # lines too long for LDS
    ((64, 900, 8), 1, 1, 2, "fp32", True), ((64, 150, 200), 1, 1, 1, "fp16", True),
    ((16, 7, 36, 47), 2, 3, 2, "fp32", True), ((48, 29, 36, 7), 1, 1, 2, "bf16", True),
    ((48, 9, 26, 27), 2, 1, 1, "fp32", True), ((16, 3, 13, 14, 15), 2, 2, 2, "bf16", True)])
def test_lines_in_lds(sl, ns, d, mask, k, tier, fused):
    n = int(np.prod([ns[e] for e in range(len(ns)) if mask >> e & 1]))
    _pair_both(sl, ns, k, tier, d, mask, [_uniform(n, 50.0, 1), _uniform(n, 9.0, 2)], fused=fused)


@pytest.mark.parametrize("k,tier", [(2, "fp32"), (2, "bf16"), (1, "fp64")])
@pytest.mark.parametrize("amp", [3.0, 10.0])
def test_pair_of_many_cells_costs_no_more_than_the_sweeps(sl, k, tier, amp):
    """Measured ratios 0.7 to 1.2; the fused pass alone took 1 to 4.6 times the
    sweeps."""
    import torch
    ns = (36, 36, 36, 36)
    plan = sl.Plan(ns, k, tier)
    a, b = plan.empty_state(), plan.empty_state()
    for t in (*a, *b):
        t.zero_()
    u = torch.arange(36, dtype=torch.float64, device="cuda") / 36
    e = torch.sin(2 * np.pi * u)[None, :] + 0.5 * torch.sin(2 * np.pi * (u[None, :] + u[:, None]))
    seq = [(2, 3, (amp * e).reshape(-1).contiguous()), (3, 3, (amp * e.t()).reshape(-1).contiguous())]
    t = []
    for fuse in (False, True):
        plan.set_fusion(fuse)
        t.append(_time(plan, seq, 4, a, b))
    assert t[1] <= 1.4 * t[0], t
    plan.close()


@pytest.mark.parametrize("ns,k,tier,want", [
    ((1024, 8, 10, 10), 3, "bf16", [(4, 1), (4, 1), (4, 1)]),     # 10 rows fill 8 + 2
    ((64, 64, 64, 3), 2, "bf16", [(8, 2), (8, 2), (4, 1)]),
    ((48, 48, 48, 48), 2, "bf16", [(8, 18)] * 3), ((48, 48, 48, 48), 2, "fp32", [(8, 2)] * 3),
    ((32, 32, 32, 27), 1, "fp16", [(8, 2), (8, 2), (4, 1)]),
    ((32, 32, 32, 27), 2, "fp16", [(8, 2)] * 3),
    ((24, 24, 24, 24), 2, "fp32", [(4, 1)] * 3), ((96, 96, 96), 2, "fp32", [(4, 1)] * 2)])
def test_default_shapes_of_uneven_grids(sl, ns, k, tier, want):
    plan = sl.Plan(ns, k, tier)
    assert [(s["rows"], s["colwaves"]) for s in plan.shapes()[1:]] == want
    plan.close()


@pytest.mark.parametrize("tier,k", [("fp64", 1), ("fp32", 2), ("bf16", 3), ("fp16", 2)])
@pytest.mark.parametrize("amp", [0.4, 1.5, 30.0])
def test_transposed_pair(sl, tier, k, amp):
    """The transpose of the sweeps d + 1, d is a pair along d, d + 1."""
    import torch
    ns = (64, 40, 90)
    seq = [(2, 1, _uniform(64, amp, 3)), (1, 1, _uniform(64, amp, 4))]
    _adjoint_both(sl, ns, k, tier, seq, 2)
    plan = sl.Plan(ns, k, tier)
    a, b = plan.empty_state(), plan.empty_state()
    for t in (*a, *b):
        t.zero_()
    plan.timing_enable(True)
    plan.split_steps_adjoint(seq, 2, a, b)
    assert plan.timing_read(-2)[0] == 2
    plan.timing_enable(False)
    torch.cuda.synchronize()
    plan.close()


@pytest.mark.parametrize("n1", [2, 3, 5, 6, 8, 9, 11, 13])
@pytest.mark.parametrize("n2", [4, 9, 23, 50])
def test_waves_of_a_pair_over_workgroups(sl, n1, n2):
    """The waves along d of one, two or four strips fill whole workgroups; the last
    group has fewer strips."""
    for k, tier in ((1, "fp16"), (2, "fp32"), (3, "bf16")):
        _pair_both(sl, (62, n1, n2), k, tier, 1, 1, [_uniform(62, 0.4, 1), _uniform(62, 0.4, 2)],
                   fused=k < 3 or n2 >= 8)
        _pair_both(sl, (8, 8, n1, n2), k, tier, 2, 1, [_uniform(8, 0.4, 1), _uniform(8, 6.0, 2)],
                   fused=k < 3 or n2 >= 8)


@pytest.mark.parametrize("ns,k,tier", [
    ((2938, 2, 74), 3, "bf16"), ((6995, 9, 33), 2, "bf16"), ((35, 11, 31, 48), 2, "bf16"),
    ((37, 99, 10, 7), 2, "fp32"), ((59, 53, 13, 16), 2, "bf16"), ((2731, 2, 24), 2, "fp64"),
    ((128, 100, 100), 2, "bf16"), ((626, 4, 116), 2, "fp64")])
def test_pair_of_any_grid_costs_no_more_than_the_sweeps(sl, ns, k, tier):
    """Displacements of less than half a cell: 0.7 to 1.0 of the sweeps, and with
    workgroups of idle waves 1.3 to 1.8."""
    import torch
    plan = sl.Plan(ns, k, tier)
    a, b = plan.empty_state(), plan.empty_state()
    for t in (*a, *b):
        t.zero_()
    d = len(ns) - 2
    n = int(np.prod(ns[:d]))
    seq = [(d + i, (1 << d) - 1, torch.linspace(-0.4, 0.4, n, dtype=torch.float64, device="cuda"))
           for i in range(2)]
    t = []
    for fuse in (False, True):
        plan.set_fusion(fuse)
        t.append(_time(plan, seq, 8, a, b))
    assert t[1] <= 1.15 * t[0], t
    plan.close()
