"""What a batch holds and when it waits: X V X passes take no more device memory
than the sweeps they replace, and setting a sequence on a fresh batch does not
wait for the stream."""
import numpy as np
import pytest

from gpu_helpers import have_gpu
from test_gpu_strang import _bits, _seq, _state

pytestmark = pytest.mark.gpu

GRIDS = {
    "2d": [((33, 40), 1), ((64, 65), 2), ((200, 1), 2), ((256, 31), 3), ((64, 3000), 1), ((1, 9), 3)],
    "narrow": [((63, 5000), 1)] * 3,
    "3d": [((64, 30, 5), 2), ((20, 9, 7), 3), ((100, 64, 3), 1)],
    "4d": [((64, 16, 4, 3), 2), ((12, 10, 3, 2), 1)],
}


@pytest.fixture(scope="module")
def sl():
    if not have_gpu():
        pytest.skip("no HIP device")
    import paper_1603_07008_amd as sl
    sl.lib()
    return sl


def _batch(grids, dims, seqs, states):
    from paper_1603_07008_amd.batch import Batch
    b = Batch([g[0] for g in grids], [g[1] for g in grids], "fp32")
    s0 = [tuple(t.clone() for t in st) for st in states]
    s1 = [tuple(t.clone() for t in st) for st in states]
    b.bind(s0, s1)
    b.set_sequence([(d, [(s[q][1], s[q][2]) for s in seqs]) for q, d in enumerate(dims)])
    return b, s0, s1


@pytest.mark.parametrize("name", sorted(GRIDS))
def test_passes_fit_where_the_sweeps_do(sl, name):
    """The sequence 0, 1, 0 under a limit of what its sweeps need: the bytes of
    the sequences 0, 1 and 0 (which have no pass) less one empty batch."""
    import torch
    grids = GRIDS[name]
    seqs = [_seq(ns, 2, 1, 2.0, 0.4, i) for i, (ns, _) in enumerate(grids)]
    plans = [sl.Plan(ns, k, "fp32") for ns, k in grids]
    states = [_state(p, i) for i, p in enumerate(plans)]
    held = sl.device_alloc_bytes()
    need = 0
    for dims in ((0, 1), (0,)):
        b, _, _ = _batch(grids, dims, seqs, states)
        need += sl.device_alloc_bytes() - held
        b.close()
    from paper_1603_07008_amd.batch import Batch
    b = Batch([g[0] for g in grids], [g[1] for g in grids], "fp32")
    need -= sl.device_alloc_bytes() - held
    b.close()
    out = []
    for limit in (None, held + need):
        sl.set_device_alloc_limit(limit)
        try:
            b, s0, s1 = _batch(grids, (0, 1, 0), seqs, states)
        finally:
            sl.set_device_alloc_limit(None)
        out.append((s0, s1)[b.run(1)])
        torch.cuda.synchronize()
        b.close()
    for x, y in zip(*out):
        for t, u in zip(x, y):
            assert torch.equal(_bits(t), _bits(u))
    for p in plans:
        p.close()


def test_set_sequence_does_not_wait(sl):
    import torch
    from paper_1603_07008_amd.batch import Batch
    grids = GRIDS["2d"]
    seqs = [_seq(ns, 2, 1, 2.0, 0.4, i) for i, (ns, _) in enumerate(grids)]
    torch.cuda.synchronize()
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        b = Batch([g[0] for g in grids], [g[1] for g in grids], "fp32", stream=stream.cuda_stream)
        torch.cuda._sleep(300_000_000)
        b.set_sequence([(d, [(s[q][1], s[q][2]) for s in seqs]) for q, d in enumerate((0, 1, 0))])
        busy = not stream.query()
        stream.synchronize()
        assert busy
        b.close()


def test_more_tables_than_a_launch_holds(sl):
    """150 problems of one degree: three launches of tables, the results those of
    the single plans."""
    import torch
    rng = np.random.default_rng(3)
    grids = [((int(n0), int(n1)), 1) for n0, n1 in rng.integers(1, 12, (150, 2))]
    seqs = [_seq(ns, 2, 1, 2.0, 0.7, i) for i, (ns, _) in enumerate(grids)]
    plans = [sl.Plan(ns, k, "fp32") for ns, k in grids]
    states = [_state(p, i) for i, p in enumerate(plans)]
    for i in range(0, 150, 2):                              # one field for both X sweeps
        seqs[i][2] = seqs[i][0]
    b, s0, s1 = _batch(grids, (0, 1, 0), seqs, states)
    got = (s0, s1)[b.run(1)]
    for i, p in enumerate(plans):
        x, y = tuple(t.clone() for t in states[i]), p.empty_state()
        want = (x, y)[p.split_steps(seqs[i], 1, x, y)]
        torch.cuda.synchronize()
        for t, u in zip(got[i], want):
            assert torch.equal(_bits(t), _bits(u)), grids[i]
        p.close()
    b.close()


def test_pass_tuning(sl, tmp_path):
    """The tuner times the launches that run: the pass, no class of its sweeps; its
    rows change speed, not results, and come back from a cache."""
    import torch
    grids = GRIDS["2d"]
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        seqs = [_seq(ns, 2, 1, 2.0, 0.4, i) for i, (ns, _) in enumerate(grids)]
        states = [_state(sl.Plan(ns, k, "fp32"), i) for i, (ns, k) in enumerate(grids)]
        b, s0, s1 = _batch(grids, (0, 1, 0), seqs, states)
        ref = None
        for rows in (0, 4, 8, 16):
            b.set_pass_tuning(0, rows)
            for st, init in zip(s0, states):
                for t, u in zip(st, init):
                    t.copy_(u)
            res = b.run(2, use_graph=rows == 8)
            got = [t.clone() for st in (s0, s1)[res] for t in st]
            ref = ref or got
            for t, u in zip(got, ref):
                assert torch.equal(_bits(t), _bits(u)), rows
        with pytest.raises(sl.SldgError):
            b.set_pass_tuning(0, 5)
        assert "pass" not in b.tuning()[1] and b.tuning()[0]["pass"]["rows"] == 16
        shapes, cached = b.tune_cached(str(tmp_path / "t.json"))
        assert not cached
        assert shapes[0]["pass"]["ms"] > 0 and shapes[0]["pass"]["tiles"] > 0
        assert all(not s["classes"] for s in shapes)
        assert abs(sum(s["ms"] for s in shapes) - shapes[0]["pass"]["ms"]) < 1e-9
        b.set_pass_tuning(0, 0)
        again, cached = b.tune_cached(str(tmp_path / "t.json"))
        assert cached and b.tuning()[0]["pass"]["rows"] == shapes[0]["pass"]["rows"]
        stream.synchronize()
        b.close()
