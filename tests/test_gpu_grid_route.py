"""GPU parity of the sphere-grid kernels at large degrees.

A plan that leaves grid and cover open runs the direct contraction, so the
tests with default plans no longer reach these kernels; a grid or cover of the
caller's choice does.  The forward (complex and real basis), channels and
gradients on one global grid of 2 L + 2 rings and with the alternate cover, at
degrees whose blocks take few pairs per work-group, many ring groups and
nearly all of a CU's LDS.  Bars: as for the same calls elsewhere, per path
(gradients: per degree) relative L2 error 1e-4 in fp32 and 1e-10 in fp64."""
import pytest

import cgtp_inputs as wl
import oracle
import oracle.channels as oc
from test_gpu_backward import _check as check_gradients, _grads
from test_gpu_parity import TOL, _lib, _torch, check_against_oracle, per_path_rel_err, run_gpu

pytestmark = pytest.mark.gpu


def _grid(L, which):
    return {"n_theta": 2 * L + 2} if which == "grid" else {"cover": _lib().CGTP_COVER_ALTERNATE}


@pytest.mark.parametrize("L,N,dtype,which", [(16, 21, "fp32", "grid"), (16, 21, "fp32", "alternate"),
                                             (20, 7, "fp32", "grid"), (32, 4, "fp32", "grid"),
                                             (16, 3, "fp64", "grid"), (19, 3, "fp64", "alternate")])
def test_forward(L, N, dtype, which):
    print("case L=%d N=%d %s %s" % (L, N, dtype, which), flush=True)
    x1, x2 = wl.draw(L, N, dtype, seed=2000 + L)
    _, _, _, out = run_gpu(L, x1, x2, dtype, **_grid(L, which))
    check_against_oracle(L, x1, x2, out.double().cpu().numpy(), dtype)


@pytest.mark.parametrize("L,N,which", [(16, 9, "grid"), (16, 9, "alternate"), (32, 3, "grid")])
def test_real_basis(L, N, which):
    torch = _torch()
    print("case L=%d N=%d %s" % (L, N, which), flush=True)
    x1, x2 = wl.draw(L, N, "fp32", seed=2100 + L)
    out = _lib().Plan(L, **_grid(L, which)).forward_real(x1.cuda(), x2.cuda())
    torch.cuda.synchronize()
    ref = oracle.cgtp_real(L, x1.double().numpy(), x2.double().numpy())
    err, path = per_path_rel_err(L, out.cpu().double().numpy(), ref)
    print("worst per-path rel L2 %.3e at %s" % (err, path), flush=True)
    assert err <= TOL["fp32"], (err, path)


@pytest.mark.parametrize("L,N,C,shared,which", [(8, 10, 7, True, "grid"), (8, 5, 3, False, "alternate"),
                                                (16, 2, 5, True, "grid")])
def test_channels(L, N, C, shared, which):
    torch = _torch()
    print("case L=%d N=%d C=%d %s" % (L, N, C, which), flush=True)
    x1, x2, w = wl.channel_inputs(L, N, C, shared, "pair", "fp32", seed=2200 + L)
    got = _lib().Plan(L, **_grid(L, which)).forward_weighted(x1.cuda(), x2.cuda(), w.cuda())
    torch.cuda.synchronize()
    ref = oc.cgtp_channels(L, x1.double().numpy(), x2.double().numpy(), w.double().numpy())
    nout = (L + 1) ** 4
    err, path = per_path_rel_err(L, got.cpu().double().numpy().reshape(N * C, nout), ref.reshape(N * C, nout))
    print("worst per-path rel L2 %.3e at %s" % (err, path), flush=True)
    assert err <= TOL["fp32"], (err, path)


@pytest.mark.parametrize("L,N,which", [(8, 19, "grid"), (16, 9, "grid"), (16, 9, "alternate"), (32, 3, "grid")])
def test_gradients(L, N, which):
    print("case L=%d N=%d %s" % (L, N, which), flush=True)
    _, host, _, got = _grads(L, N, "fp32", seed=2300 + L, **_grid(L, which))
    check_gradients(L, host, got, "fp32", what=which)


@pytest.mark.parametrize("call", ["forward", "forward_real", "backward"])
def test_rows_do_not_depend_on_the_number_of_pairs(call):
    """Work-groups of several pairs and several tiles of them (the first pairs of 300 against a call of their own)."""
    torch = _torch()
    L, N = 12, 300
    x1, x2 = (v.cuda() for v in wl.draw(L, N, "fp32", seed=5))
    plan = _lib().Plan(L, n_theta=2 * L + 2)
    rows = [x1, x2] + ([wl.draw_rows((L + 1) ** 4, N, "fp32", seed=6)[0].cuda()] if call == "backward" else [])
    many, few = (getattr(plan, call)(*(r[:n] for r in rows)) for n in (N, 5))
    for a, b in zip(few, many) if call == "backward" else [(few, many)]:
        assert torch.equal(a, b[:5])
