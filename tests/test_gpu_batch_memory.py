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
