"""Self-consistent steps: displacement buffers that overlap, and where the result
lies when the caller does not ask."""
import ctypes

import pytest

from gpu_helpers import have_gpu
from test_gpu_strang import _bits, _state

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sl():
    if not have_gpu():
        pytest.skip("no HIP device")
    import paper_1603_07008_amd as sl
    sl.lib()
    return sl


def _ptr(t):
    return ctypes.c_void_p(t.data_ptr())


def test_x_displacements_under_the_field_1d1v(sl):
    """shift_v over shift_x: every field solve replaces the x displacements, as the
    sweeps one by one read them."""
    import torch
    ns, hx, hv, dt, nsteps = (40, 30), 0.3, 0.2, 0.1, 3
    plan = sl.Plan(ns, 2, "fp32")
    st = _state(plan, 1)
    both = torch.linspace(-1.0, 1.0, 40, dtype=torch.float64, device="cuda")
    a, b = tuple(t.clone() for t in st), plan.empty_state()
    res = ctypes.c_int(-1)
    rc = sl.lib().sldg_vlasov_poisson_steps(
        plan._h, nsteps, _ptr(both), ctypes.c_double(hx), ctypes.c_double(hv), ctypes.c_double(dt),
        _ptr(both), *[_ptr(t) for t in (*a, *b)], ctypes.byref(res))
    assert rc == 0
    got = (a, b)[res.value]
    s = torch.linspace(-1.0, 1.0, 40, dtype=torch.float64, device="cuda")
    buf, cur = [tuple(t.clone() for t in st), plan.empty_state()], 0
    for _ in range(nsteps):
        for dim in (0, 1, 0):
            if dim:
                s.copy_(plan.poisson_shift(*buf[cur], hx, hv, dt))
            plan.advect_dim(dim, s if dim else s[:30].contiguous(), 1 if dim else 2, *buf[cur],
                            *buf[1 - cur])
            cur = 1 - cur
    torch.cuda.synchronize()
    for x, y in zip(got, buf[cur]):
        assert torch.equal(_bits(x), _bits(y))
    plan.close()


@pytest.mark.parametrize("which", [0, 1])
def test_x_displacements_under_the_field_2d2v(sl, which):
    import torch
    ns, h, dt, nsteps = (12, 9, 6, 7), (0.3, 0.4, 0.2, 0.25), 0.1, 2
    plan = sl.Plan(ns, 2, "fp32")
    st = _state(plan, 2)
    nv = ns[0] * ns[1]

    def start():
        v = [torch.zeros(nv, dtype=torch.float64, device="cuda") for _ in range(2)]
        x = [torch.linspace(-2.0, 2.0, ns[d], dtype=torch.float64, device="cuda") for d in (2, 3)]
        v[1][:ns[2 + which]] = x[which]
        return x, v
    x, v = start()
    xs = list(x)
    xs[which] = v[1]                                  # x displacements at the start of shift_v2
    a, b = tuple(t.clone() for t in st), plan.empty_state()
    res = ctypes.c_int(-1)
    rc = sl.lib().sldg_vlasov_poisson_steps_2d2v(
        plan._h, nsteps, _ptr(xs[0]), _ptr(xs[1]), (ctypes.c_double * 4)(*h), ctypes.c_double(dt),
        _ptr(v[0]), _ptr(v[1]), *[_ptr(t) for t in (*a, *b)], ctypes.byref(res))
    assert rc == 0
    got = (a, b)[res.value]
    x, v = start()
    buf, cur = [tuple(t.clone() for t in st), plan.empty_state()], 0

    def sweep(d, s, mask):
        nonlocal cur
        plan.advect_dim(d, s, mask, *buf[cur], *buf[1 - cur])
        cur = 1 - cur
    for _ in range(nsteps):
        for half in range(2):
            for d in (0, 1):
                sweep(d, v[1][:ns[2 + d]].contiguous() if d == which else x[d], 4 << d)
            if half == 0:
                rc = sl.lib().sldg_poisson_shift_2d(plan._h, *[_ptr(t) for t in buf[cur]],
                                                    (ctypes.c_double * 4)(*h), ctypes.c_double(dt),
                                                    _ptr(v[0]), _ptr(v[1]), None)
                assert rc == 0
                sweep(2, v[0], 3)
                sweep(3, v[1], 3)
    torch.cuda.synchronize()
    for p, q in zip(got, buf[cur]):
        assert torch.equal(_bits(p), _bits(q))
    plan.close()


@pytest.mark.parametrize("nsteps", [1, 2, 3])
def test_2d2v_result_buffer_not_asked_for(sl, nsteps):
    """With a NULL result_buffer the result is in buffer 0, also after an odd number
    of steps, whose (v1, v2) pairs take one pass each."""
    import torch
    ns, h, dt = (12, 8, 6, 7), (0.3, 0.4, 0.2, 0.25), 0.1
    plan = sl.Plan(ns, 1, "fp32")
    st = _state(plan, 3)
    x = [torch.linspace(-2.0, 2.0, ns[d], dtype=torch.float64, device="cuda") for d in (2, 3)]
    v = [torch.zeros(ns[0] * ns[1], dtype=torch.float64, device="cuda") for _ in range(2)]
    out = []
    for fuse in (False, True):
        plan.set_fusion(fuse)
        a, b = tuple(t.clone() for t in st), plan.empty_state()
        plan.timing_enable(True)
        rc = sl.lib().sldg_vlasov_poisson_steps_2d2v(
            plan._h, nsteps, _ptr(x[0]), _ptr(x[1]), (ctypes.c_double * 4)(*h), ctypes.c_double(dt),
            _ptr(v[0]), _ptr(v[1]), *[_ptr(t) for t in (*a, *b)], None)
        assert rc == 0
        pairs = nsteps - nsteps % 2 if fuse else 0
        higher = plan.timing_read(-2)[0]                 # x2 sweeps not in a fused pass, v1, v2
        assert higher == (0 if fuse else 2 * nsteps) + 2 * nsteps - pairs
        plan.timing_enable(False)
        out.append(a)
    torch.cuda.synchronize()
    for p, q in zip(*out):
        assert torch.equal(_bits(p), _bits(q))
    plan.close()
