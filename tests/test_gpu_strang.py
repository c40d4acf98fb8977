"""X V X passes (sweeps along dimensions 0, 1, 0 fused by sldg_split_steps,
section II splitting; section II-A update): bitwise the three sweeps run one
by one, over line lengths around the tile size, rows with
displacements of their own along dimension 0, columns with any displacement
along dimension 1, dependence on higher dimensions, every tier and degree."""
import numpy as np
import pytest

from gpu_helpers import have_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sl():
    if not have_gpu():
        pytest.skip("no HIP device")
    import paper_1603_07008_amd as sl
    sl.lib()
    return sl


def _bits(t):
    import torch
    return t.view({8: torch.int64, 4: torch.int32, 2: torch.int16}[t.element_size()])


def _state(plan, seed):
    import torch
    import paper_1603_07008_amd as sl
    g = torch.Generator(device="cuda").manual_seed(seed)
    m = torch.randn((plan.n_lo, plan.cells), generator=g, device="cuda", dtype=torch.float64)
    h = torch.randn((plan.n_hi, plan.cells), generator=g, device="cuda", dtype=torch.float64)
    return (m.reshape(-1) if plan.n_lo == 1 else m), h.to(sl.hi_dtype(plan.tier))


def _seq(ns, mask_x, mask_v, amp_x, amp_v, seed):
    import torch
    rng = np.random.default_rng(seed)

    def field(mask, amp):
        n = int(np.prod([ns[e] for e in range(len(ns)) if mask >> e & 1] or [1]))
        return torch.from_numpy(rng.uniform(-amp, amp, n)).cuda()
    x0, x1 = field(mask_x, amp_x), field(mask_x, amp_x)
    return [(0, mask_x, x0), (1, mask_v, field(mask_v, amp_v)), (0, mask_x, x1)]


def _both(sl, ns, k, tier, seq, nsteps=1, ndouble=1, seed=3):
    import torch
    plan = sl.Plan(ns, k, tier, ndouble=ndouble)
    st = _state(plan, seed)
    out = []
    for fuse in (False, True):
        plan.set_fusion(fuse)
        a = tuple(t.clone() for t in st)
        b = tuple(torch.full_like(t, float("nan")) for t in st)
        r = plan.split_steps(seq, nsteps, a, b)
        out.append((a, b)[r])
        assert r == (nsteps * len(seq)) % 2
    torch.cuda.synchronize()
    for x, y in zip(*out):
        assert torch.equal(_bits(x), _bits(y)), (ns, k, tier)
    plan.close()


@pytest.mark.parametrize("n0", [1, 2, 3, 61, 62, 63, 64, 65, 124, 125, 300, 641])
@pytest.mark.parametrize("tier,k", [("fp32", 2), ("bf16", 1)])
def test_line_lengths(sl, n0, tier, k):
    ns = (n0, 7)
    _both(sl, ns, k, tier, _seq(ns, 2, 1, 1.5 * n0, 1.3, n0))


@pytest.mark.parametrize("tier", ["fp64", "fp32", "bf16", "fp16"])
@pytest.mark.parametrize("k", [1, 2, 3])
@pytest.mark.parametrize("ndouble", [0, 1])
def test_tiers_and_degrees(sl, tier, k, ndouble):
    ns = (75, 41)
    _both(sl, ns, k, tier, _seq(ns, 2, 1, 9.0, 0.4, k), nsteps=3, ndouble=ndouble)


@pytest.mark.parametrize("n1", [1, 3, 46, 47, 93, 185, 371, 401])
def test_rows_per_wave(sl, n1):
    """Strips of every length, the last one short, over all rows per wave."""
    ns = (63 * 12, n1)
    _both(sl, ns, 1, "fp32", _seq(ns, 2, 1, 20.0, 0.6, n1), nsteps=2)


@pytest.mark.parametrize("ns,mask_x,mask_v", [
    ((37, 1), 2, 1), ((40, 2), 2, 1), ((66, 9), 0, 0), ((66, 9), 2, 0),
    ((21, 6, 5), 0b110, 0b101), ((21, 6, 5), 0b010, 0b100), ((400, 5, 3), 0b110, 0b101),
    ((10, 6, 4, 3), 0b1010, 0b0101)])
def test_masks_and_higher_dimensions(sl, ns, mask_x, mask_v):
    for tier, k in (("fp32", 1), ("fp64", 2)):
        _both(sl, ns, k, tier, _seq(ns, mask_x, mask_v, 3.0, 40.0, 5), nsteps=2)


def test_non_finite_displacements_and_values(sl):
    import torch
    ns = (70, 12)
    seq = _seq(ns, 2, 1, 2.0, 2.0, 9)
    seq[0][2][3] = float("nan")
    seq[1][2][20] = float("inf")
    plan = sl.Plan(ns, 2, "fp32")
    st = _state(plan, 4)
    st[1][2, 5] = float("inf")
    st[0][100] = float("nan")
    out = []
    for fuse in (False, True):
        plan.set_fusion(fuse)
        a = tuple(t.clone() for t in st)
        b = plan.empty_state()
        out.append((a, b)[plan.split_steps(seq, 1, a, b)])
    torch.cuda.synchronize()
    for x, y in zip(*out):
        assert torch.equal(torch.isnan(x), torch.isnan(y))
        ok = ~torch.isnan(x)
        assert torch.equal(x[ok], y[ok])
    plan.close()


@pytest.mark.parametrize("tier", ["fp64", "fp32", "bf16", "fp16"])
def test_batched_passes(sl, tier):
    """Batches: lines of one to ten tiles, strips that wrap, one and two V
    shifts per wave around zero and far from it and waves whose shifts are
    spread, eager and as a graph, against each problem's sweeps one by one."""
    import torch
    from paper_1603_07008_amd.batch import Batch
    grids = [((33, 40), 1, 0.3), ((64, 65), 2, 0.3), ((200, 1), 2, 0.4), ((256, 31), 3, 0.0),
             ((257, 70), 1, 0.3), ((400, 33), 2, 0.4), ((512, 18), 2, 0.2), ((300, 35), 3, 0.3),
             ((1, 50), 2, 0.3), ((5, 2), 1, 0.4), ((600, 20), 1, 0.3), ((48, 30), 2, 3.0)]
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        seqs, states = [], []
        for i, (ns, k, amp) in enumerate(grids):
            seq = _seq(ns, 2, 1, 1.2 * ns[0], amp, i)
            if i % 3 == 1:
                seq[1][2].add_(7.0 - 2.0 * i)
            states.append(_state(sl.Plan(ns, k, tier, stream=stream.cuda_stream), i))
            seqs.append(seq)
        b = Batch([g[0] for g in grids], [g[1] for g in grids], tier, stream=stream.cuda_stream)
        seq = [(seqs[0][q][0], [(s[q][1], s[q][2]) for s in seqs]) for q in range(3)]
        for graph in (False, True):
            s0 = [tuple(t.clone() for t in st) for st in states]
            s1 = [tuple(torch.full_like(t, float("nan")) for t in st) for st in states]
            b.bind(s0, s1)
            b.set_sequence(seq)
            for steps in (1, 2):
                res = b.run(steps, use_graph=graph)
                assert res == steps % 2
                if res:
                    for x, y in zip(s0, s1):
                        for t, u in zip(x, y):
                            t.copy_(u)
            stream.synchronize()
            for i, (ns, k, _) in enumerate(grids):
                plan = sl.Plan(ns, k, tier, stream=stream.cuda_stream)
                plan.set_fusion(False)
                x = tuple(t.clone() for t in states[i])
                y = plan.empty_state()
                want = (x, y)[plan.split_steps(seqs[i], 3, x, y)]
                stream.synchronize()
                for got, ref in zip(s0[i], want):
                    assert torch.equal(_bits(got), _bits(ref)), (ns, k, graph)
                plan.close()
        b.close()


@pytest.mark.parametrize("ns,k,tier", [((40, 90), 1, "fp32"), ((130, 33), 2, "bf16"),
                                       ((63, 63), 3, "fp64"), ((1100, 20), 1, "fp16")])
def test_self_consistent_steps(sl, ns, k, tier):
    """Vlasov-Poisson steps (V X X passes between field solves) are bitwise the
    sweeps and field solves one by one; N_x above and below the threads of the
    field solve."""
    import torch
    hx, hv, dt = 0.3, 0.2, 0.1
    plan = sl.Plan(ns, k, tier)
    st = _state(plan, 6)
    sx = _seq(ns, 2, 1, 4.0, 0.3, 8)[0][2]
    for nsteps in (1, 2, 5):
        a = tuple(t.clone() for t in st)
        b = plan.empty_state()
        got = (a, b)[plan.vlasov_poisson_steps(nsteps, sx, hx, hv, dt, a, b)]
        buf = [tuple(t.clone() for t in st), plan.empty_state()]
        cur = 0
        for _ in range(nsteps):
            for dim in (0, 1, 0):
                mask, s = (2, sx) if dim == 0 else (1, plan.poisson_shift(*buf[cur], hx, hv, dt))
                plan.advect_dim(dim, s, mask, *buf[cur], *buf[1 - cur])
                cur = 1 - cur
        torch.cuda.synchronize()
        for x, y in zip(got, buf[cur]):
            assert torch.equal(_bits(x), _bits(y)), nsteps
    plan.close()


@pytest.mark.parametrize("ns", [(12, 9, 5, 7), (9, 6, 4, 5), (8, 8, 1, 1)])
def test_self_consistent_steps_2d2v(sl, ns):
    """2D-2V Vlasov-Poisson steps with the (x1, x2) sweeps fused (and where they
    cannot be, or the tables do not fit together) are bitwise the unfused ones."""
    import torch
    plan = sl.Plan(ns, 2, "fp32")
    st = _state(plan, 2)
    seq = [torch.linspace(-2.0, 2.0, ns[d], dtype=torch.float64, device="cuda") for d in (2, 3)]
    out = []
    for fuse in (False, True):
        plan.set_fusion(fuse)
        a = tuple(t.clone() for t in st)
        b = plan.empty_state()
        r = plan.vlasov_poisson_steps_2d2v(2, *seq, (0.3, 0.4, 0.2, 0.25), 0.1, a, b)
        out.append((a, b)[r])
    torch.cuda.synchronize()
    for x, y in zip(*out):
        assert torch.equal(_bits(x), _bits(y))
    plan.close()
