"""The direct contraction (plans without a grid or cover of the caller's choice).

CPU: the plan's work lists run by a host model (direct_model.cpp) that checks
every index and compares with the oracle's coefficients.  GPU: parity with the
fp64 oracle where tiles of pairs, chunks of k steps, row groups and stages end,
and agreement with the sphere-grid route, which an explicit grid selects.

Bounds: a sum of at most 65 products of 32-bit numbers with 32-bit
coefficients is off by a few 2^-24 of its terms' norm; 1e-6 relative L2 per
call (1e-14 in 64 bits) is about ten times that."""
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
TOL = {"fp32": 1e-6, "fp64": 1e-14}


@pytest.fixture(scope="module")
def model(tmp_path_factory):
    if shutil.which("g++") is None or shutil.which("gcc") is None:
        pytest.skip("no host compiler")
    out = tmp_path_factory.mktemp("direct")
    obj, exe = str(out / "oracle.o"), str(out / "direct_model")
    subprocess.run(["gcc", "-O2", "-std=c11", "-fopenmp", "-c", os.path.join(ROOT, "oracle", "cgtp_oracle.c"), "-o", obj],
                   check=True)
    subprocess.run(["g++", "-O2", "-std=c++17", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                    "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROOT, "tests", "sanitize"), "-I", "/opt/rocm/include",
                    "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2602_21466_amd", "csrc"),
                    os.path.join(ROOT, "tests", "direct_model.cpp"), obj, "-fopenmp", "-lm", "-o", exe], check=True)
    return lambda *a: float(subprocess.run([exe] + [str(v) for v in a], check=True, capture_output=True,
                                           text=True).stdout)


def test_coefficients_match_the_racah_formula(model):
    """Every 12th block (la <= lb) up to degree 32, every order and degree."""
    assert model("cg", 32) < 5e-14


@pytest.mark.parametrize("dtype,L", [("fp32", 0), ("fp32", 1), ("fp32", 2), ("fp32", 4), ("fp32", 7), ("fp32", 11),
                                     ("fp32", 16), ("fp64", 0), ("fp64", 3), ("fp64", 8),
                                     ("backward", 0), ("backward", 3), ("backward", 8), ("backward", 17),
                                     # the largest degrees; gradients of blocks in several parts (from 21)
                                     ("fp32", 24), ("fp32", 32), ("fp64", 14), ("fp64", 19), ("backward", 21),
                                     ("backward", 24), ("backward", 32)])
def test_work_lists_cover_every_output_once(model, dtype, L):
    assert model(dtype, L) < TOL.get(dtype, 1e-6)


# one launch takes fewer than 2^32 work-items: 2^23 - 1 work-groups of 512 threads
@pytest.mark.parametrize("L,n", [(1, 1), (9, 1), (23, 2), (26, 9), (31, 257)])
def test_launches_cover_every_work_group(model, L, n):
    assert model("launches", L) == n


def _rel(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


def _rows(torch, n, cols, dtype, seed):
    g = torch.Generator("cpu").manual_seed(seed)
    return torch.randn(n, cols, dtype=torch.float64, generator=g).to({"fp32": torch.float32, "fp64": torch.float64}[dtype])


# ragged tiles of 16 (fp32) and 32 (fp64) pairs; degrees whose blocks end inside and at the end of
# row groups, chunks of 8 / 16 k steps, groups of 8 / 4 orders, and with one or several stages
@pytest.mark.gpu
@pytest.mark.parametrize("L,N,dtype", [(0, 1, "fp32"), (1, 15, "fp32"), (2, 16, "fp32"), (3, 17, "fp32"), (5, 33, "fp32"),
                                       (8, 3, "fp32"), (13, 18, "fp32"), (20, 2, "fp32"), (0, 33, "fp64"),
                                       (2, 31, "fp64"), (4, 32, "fp64"), (9, 5, "fp64"),
                                       (27, 3, "fp32"), (32, 2, "fp32"), (14, 33, "fp64"), (19, 3, "fp64")])
def test_forward_and_real_match_oracle(L, N, dtype):
    import torch
    import oracle
    import paper_2602_21466_amd as lib
    print("case L=%d N=%d %s" % (L, N, dtype), flush=True)
    x1, x2 = _rows(torch, N, (L + 1) ** 2, dtype, L), _rows(torch, N, (L + 1) ** 2, dtype, 100 + L)
    a, b = x1.double().numpy(), x2.double().numpy()
    plan = lib.Plan(L, dtype=dtype)
    z = plan.forward(x1.cuda(), x2.cuda()).double().cpu().numpy()
    r = plan.forward_real(x1.cuda(), x2.cuda()).double().cpu().numpy()
    assert _rel(z, oracle.cgtp(L, a, b)) < TOL[dtype]
    assert _rel(r, oracle.cgtp_real(L, a, b)) < TOL[dtype]
    plan.close()


# ragged tiles of 16 and 8 pairs; the three classes of blocks (largest degrees up to 6, 16 and above)
@pytest.mark.gpu
@pytest.mark.parametrize("L,N", [(0, 1), (1, 17), (3, 15), (6, 33), (11, 16), (13, 9), (16, 8), (18, 5),
                                 # blocks in several parts
                                 (21, 9), (27, 3), (32, 2)])
def test_gradients_match_oracle(L, N):
    import torch
    import oracle
    import paper_2602_21466_amd as lib
    print("case L=%d N=%d" % (L, N), flush=True)
    x1, x2 = _rows(torch, N, (L + 1) ** 2, "fp32", L), _rows(torch, N, (L + 1) ** 2, "fp32", 100 + L)
    g = _rows(torch, N, (L + 1) ** 4, "fp32", 200 + L)
    plan = lib.Plan(L)
    a = plan.backward(x1.cuda(), x2.cuda(), g.cuda())
    b = plan.backward(x1.cuda(), x2.cuda(), g.cuda())
    ref = oracle.cgtp_backward(L, x1.double().numpy(), x2.double().numpy(), g.double().numpy())
    for u, v, r in zip(a, b, ref):
        assert torch.equal(u, v)   # every sum has a fixed order
        assert _rel(u.double().cpu().numpy(), r) < TOL["fp32"]
    plan.close()


# one tile of pairs and a few, which take the short lists of groups and stages, against
# more pairs than those are taken for
@pytest.mark.gpu
@pytest.mark.parametrize("L,N,dtype", [(2, 25000, "fp32"), (5, 4500, "fp32"), (8, 900, "fp32"), (13, 200, "fp32"),
                                       (19, 40, "fp32"), (3, 17000, "fp64"), (6, 2100, "fp64"), (12, 260, "fp64")])
def test_outputs_do_not_depend_on_the_number_of_pairs(L, N, dtype):
    import torch
    import paper_2602_21466_amd as lib
    print("case L=%d N=%d %s" % (L, N, dtype), flush=True)
    nin = (L + 1) ** 2
    x1, x2 = _rows(torch, N, nin, dtype, L).cuda(), _rows(torch, N, nin, dtype, 100 + L).cuda()
    w = _rows(torch, N, lib.cgtp_num_paths(L), dtype, 200 + L).cuda()
    g = _rows(torch, N, nin ** 2, dtype, 300 + L).cuda() if dtype == "fp32" else None
    plan = lib.Plan(L, dtype=dtype)

    def calls(n):
        z = [plan.forward(x1[:n], x2[:n]), plan.forward_real(x1[:n], x2[:n]),
             plan.forward_weighted(x1[:n, None].contiguous(), x2[:n], w[:n, None].contiguous())[:, 0]]
        return z + list(plan.backward(x1[:n], x2[:n], g[:n]) if g is not None else ())
    many = calls(N)
    for n in (1, 17):
        for a, b in zip(calls(n), many):
            assert torch.equal(a, b[:n])
    plan.close()


@pytest.mark.gpu
def test_threads_share_a_plan():
    """One plan, two threads on streams of their own: few pairs (short list) and many (long list), which take
    different amounts of LDS above 64 KiB in fp64."""
    import threading
    import torch
    import paper_2602_21466_amd as lib
    L, N = 12, 400
    plan = lib.Plan(L, dtype="fp64")
    x1, x2 = _rows(torch, N, (L + 1) ** 2, "fp64", 1).cuda(), _rows(torch, N, (L + 1) ** 2, "fp64", 2).cuda()
    ref = plan.forward(x1, x2)
    torch.cuda.synchronize()
    wrong = []

    def work(n):
        try:
            s = torch.cuda.Stream()
            with torch.cuda.stream(s):
                z = torch.empty(n, (L + 1) ** 4, dtype=torch.float64, device="cuda")
                for _ in range(40):
                    plan.forward(x1[:n], x2[:n], z, stream=s)
                s.synchronize()
                if not torch.equal(z, ref[:n]):
                    wrong.append(n)
        except Exception as e:
            wrong.append(e)
    threads = [threading.Thread(target=work, args=(n,)) for n in (3, N, 17, N)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong, wrong
    plan.close()


@pytest.mark.gpu
@pytest.mark.parametrize("shared,weights", [(True, "channel"), (False, "pair"), (True, "none")])
def test_routes_agree(shared, weights):
    """The direct contraction and the sphere-grid kernels (explicit grid): plain, real, channels (bound: the sum of
    both routes' errors, the grid route's per-call error is below 1e-6 at this degree)."""
    import torch
    import cgtp_inputs
    import paper_2602_21466_amd as lib
    L, N, C = 6, 7, 5
    x1, x2, w = cgtp_inputs.channel_inputs(L, N, C, shared, weights, "fp32", seed=3)
    x1, x2, w = x1.cuda(), x2.cuda(), None if w is None else w.cuda()
    direct, grid = lib.Plan(L), lib.Plan(L, n_theta=2 * L + 2, n_phi=27)
    a, b = (p.forward_weighted(x1, x2, w).double().cpu().numpy() for p in (direct, grid))
    assert _rel(a, b) < 2e-6
    y1, y2 = x1.reshape(N * C, -1), x1.flip(0).reshape(N * C, -1).contiguous()
    for name in ("forward", "forward_real"):
        a, b = (getattr(p, name)(y1, y2).double().cpu().numpy() for p in (direct, grid))
        assert _rel(a, b) < 2e-6
    direct.close()
    grid.close()


@pytest.mark.gpu
def test_infinite_input_stays_in_its_blocks():
    """A degree holding an infinity spoils only the blocks that read it, and other pairs nothing at all."""
    import torch
    import paper_2602_21466_amd as lib
    L, N = 5, 19
    x1, x2 = _rows(torch, N, (L + 1) ** 2, "fp32", 1).cuda(), _rows(torch, N, (L + 1) ** 2, "fp32", 2).cuda()
    plan = lib.Plan(L)
    ref = plan.forward(x1, x2)
    l, n = 3, 4
    for which in (0, 1):
        y = [x1.clone(), x2.clone()]
        y[which][n, l * l + 2] = float("inf")
        z = plan.forward(*y)
        keep = torch.ones_like(z, dtype=torch.bool)
        for k in range(L + 1):
            l1, l2 = (l, k) if which == 0 else (k, l)
            o = lib.cgtp_path_offset(L, l1, l2, abs(l1 - l2))
            keep[n, o:o + (2 * l1 + 1) * (2 * l2 + 1)] = False
        assert torch.equal(z[keep], ref[keep])
    plan.close()


@pytest.mark.gpu
def test_more_pairs_than_one_launch_takes():
    """Degree 0 (outputs x1 x2, exact): pairs past the work-items of one launch, 16 pairs per work-group of 512
    (forward) and 256 (gradients) threads."""
    import torch
    import paper_2602_21466_amd as lib
    plan = lib.Plan(0)
    n = 2 ** 27 + 17
    print("case L=0 N=%d forward" % n, flush=True)
    x1, x2 = (torch.randn(n, 1, device="cuda") for _ in range(2))
    assert torch.equal(plan.forward(x1, x2), x1 * x2)
    assert torch.equal(plan.forward_real(x1, x2), x1 * x2)
    n = 2 ** 28 + 17
    print("case L=0 N=%d gradients" % n, flush=True)
    x1, x2, g = (torch.randn(n, 1, device="cuda") for _ in range(3))
    g1, g2 = plan.backward(x1, x2, g)
    assert torch.equal(g1, g * x2) and torch.equal(g2, g * x1)
    plan.close()
