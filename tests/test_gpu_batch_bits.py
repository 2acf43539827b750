"""A field of a batch gets, bit for bit, what it gets alone: solve, step and pullback. The
batch decides how many lines an FFT workgroup takes and with which instance, whether the 2D
row kernels run and how a z-march is cut, none of which may show in the result."""
import pytest
import torch

import synth as S

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _compare(s, one, scheme="rk4", vjp=True):
    torch.manual_seed(1)
    u = torch.randn(s.vel_shape, dtype=s.dtype, device="cuda")
    ub = torch.randn_like(u)
    r = torch.randn(s.scal_shape, dtype=s.pdtype, device="cuda")
    s.project(u, out=u)
    for k in (0, s.batch - 1):
        uk, rk, bk = u[k].contiguous(), r[k].contiguous(), ub[k].contiguous()
        assert torch.equal(s.poisson_solve(r)[k], one.poisson_solve(rk))
        assert torch.equal(s.step(u, 1e-3, scheme=scheme)[k], one.step(uk, 1e-3, scheme=scheme))
        if vjp:
            assert torch.equal(s.step_vjp(u, ub, 1e-3, scheme=scheme)[k], one.step_vjp(uk, bk, 1e-3, scheme=scheme))
    s.close()
    one.close()


# row kernels alone and separate kernels in the batch; other line counts; ragged line batches
PERIODIC = [((64, 64), 64), ((128, 128), 16), ((256, 256), 4), ((256, 256), 16), ((250, 126), 12), ((96, 70), 9),
            ((400, 300), 3), ((512, 512), 2), ((24, 20, 14), 40), ((48, 40, 54), 8), ((96, 90, 84), 4), ((150, 126, 98), 2)]


# the all-float32 comparison mode steps with RK4 and has no pullback
@pytest.mark.parametrize("scheme,precision", [("rk4", "fp64"), ("wray3", "fp64"), ("rk4", "fp32"), ("wray3", "fp32"),
                                              ("rk4", "fp32_all")])
@pytest.mark.parametrize("n,batch", PERIODIC)
def test_periodic(n, batch, scheme, precision):
    from paper_2604_18536_amd import Solver

    _compare(Solver(n, batch=batch, nu=0.01, precision=precision), Solver(n, nu=0.01, precision=precision), scheme,
             precision != "fp32_all")


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("tanh", [False, True])
@pytest.mark.parametrize("n,batch", [((64, 40), 8), ((32, 24, 20), 6), ((64, 33, 54), 2), ((96, 50, 84), 3), ((128, 64, 64), 2)])
def test_channel(n, batch, tanh, precision):
    from paper_2604_18536_amd import Solver

    lo, hi = S.channel_box(n)
    s, one = (Solver(n, batch=b, nu=0.01, precision=precision, lo=lo, hi=hi, bc="walls") for b in (batch, 1))
    if tanh:
        for q in (s, one):
            q.set_y_faces(S.tanh_faces(n[1], lo[1], hi[1], 1.4))
    _compare(s, one)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("n,batch", [((64, 64), 64), ((32, 32, 32), 8), ((96, 50, 84), 2)])
def test_eddy_viscosity(n, batch, precision):
    from paper_2604_18536_amd import Solver

    s, one = (Solver(n, batch=b, nu=0.01, precision=precision) for b in (batch, 1))
    for q in (s, one):
        q.set_eddy(0.17)
    _compare(s, one)


def test_learned_closure():
    from paper_2604_18536_amd import Solver
    from paper_2604_18536_amd.les import init_params

    torch.manual_seed(2)
    th = init_params(0)
    th[30304:30304 + 2592].uniform_(-0.02, 0.02)
    s, one = (Solver((96, 50, 84), batch=b, nu=0.01, precision="fp32") for b in (2, 1))
    for q in (s, one):
        q.set_closure(th)
    _compare(s, one)
