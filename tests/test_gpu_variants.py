"""Every register variant of the block kernels at the edges of its range, with lists
long enough that each size bucket is launched by itself and that workgroups take
several blocks (more blocks than workgroups, so that the memory of a part of the
factor is used again).

A chain of 1-point blocks, then COPIES copies of every case: `own` points conditioned
on the last joint - own points of the chain.  The copies share coordinates and
observations, so that all must give the bits of the first, and the first is compared
with the FP64 oracle on the structure with one copy.

Block terms within tol (|l_i| + |d_i| + u_i): FP64 tol = 1e-10, FP32 tol = n_A 2^-24
(sigma^2 + tau^2) / tau^2 (backward error of the factorisation against pivots no
smaller than tau^2).  Gradients within 1e-8 max(|g|_inf, 1) in FP64; FP32 (nugget
0.1): backward error of the factorisation and of the two solves, 2 n_A 2^-24 (sigma^2
+ tau^2) / tau^2, of terms of order one per own point, summed over the blocks.
Simulated values within 1e-9 of the oracle's.
"""
import numpy as np
import pytest

import oracle as O
from helpers import block_tolerance, to_gpu
from paper_2504_12004_amd import synth

pytestmark = pytest.mark.gpu

# joint sizes per variant (tile capacity)
JOINT = {4: [1, 2, 15, 16, 17, 18, 31, 32, 33, 34, 47, 48, 49, 50, 63, 64],
         8: [65, 66, 79, 80, 81, 112, 127, 128],
         12: [129, 130, 143, 144, 145, 176, 191, 192],
         14: [193, 194, 207, 208, 209, 215, 223, 224],
         16: [225, 226, 239, 240, 241, 248, 255, 256],
         17: [257, 258, 260, 263, 264, 265, 271, 272]}
COPIES, LEAD = 130, 272
CASES = [(j, min(j, (1, 5, 17, 33)[i % 4])) for js in JOINT.values() for i, j in enumerate(js)]


@pytest.fixture(scope="module")
def sbv():
    from paper_2504_12004_amd import sbv as S
    return S


def _structure(copies, cases=CASES):
    """Structure and, for every point, its row in the inputs of the one-copy structure."""
    own = [1] * LEAD + [b for _, b in cases] * copies
    one = np.r_[0, np.cumsum(own[:LEAD + len(cases)])]
    rows = np.r_[np.arange(LEAD), np.tile(np.arange(LEAD, one[-1]), copies)]
    bp = np.r_[0, np.cumsum(own)]
    nn = [[]] * LEAD + [np.arange(LEAD - (j - b), LEAD) for j, b in cases] * copies
    S = O.Structure(int(bp[-1]), 0, 0, bp, np.arange(bp[-1]), np.r_[0, np.cumsum([len(v) for v in nn])],
                    np.concatenate(nn).astype(np.int64))
    return S, rows


def _inputs(d, tau2):
    n = LEAD + sum(b for _, b in CASES)
    X, th, xi = synth.random_spd_problem(n, d, 30 + d, beta=np.linspace(0.2, 0.5, d), tau2=tau2)
    return X, np.random.default_rng(d).standard_normal(n), th, xi


def _copies_equal(v):
    return np.all(v == v[:1])


def _handle(sbv, X, y):
    S, rows = _structure(COPIES)
    B = to_gpu(sbv, X[rows], None if y is None else y[rows], S)
    # every bucket by itself
    flops, tiles = sbv.sbv_plan_flops(B, 5)
    nA = np.diff(S.nn_ptr) + np.diff(S.block_ptr)
    cap = np.array([next(t for t in JOINT if a <= 16 * t) for a in nA])
    got = dict(zip((int(t) for t in tiles), flops))
    for t in JOINT:
        a = nA[cap == t].astype(float)
        assert abs(got[t] - np.sum(a ** 3 / 3 + a ** 2)) <= 1e-9 * got[t], t
    return B, rows


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("d,two_nu", [(3, 3), (10, 5)])
def test_values(sbv, d, two_nu, prec, monkeypatch):
    import torch
    X, y, th, _ = _inputs(d, 1e-3)
    S1, _ = _structure(1)
    _, ref, ud = O.sbv_loglik(X, y, S1, th, two_nu, blocks=True, parts=True)
    B, _ = _handle(sbv, X, y)
    total = sbv.sbv_loglik(B, th, two_nu, prec)[0]
    lb = sbv.sbv_blocks_terms(B)
    tail = lb[LEAD:].reshape(COPIES, len(CASES))
    assert _copies_equal(tail)
    sizes = np.diff(S1.nn_ptr) + np.diff(S1.block_ptr)
    tol = sizes * 2.0 ** -24 * (1.0 + np.exp(-th[d + 1])) if prec else np.full(S1.K, 1e-10)
    err = np.abs(lb[:S1.K] - ref) / block_tolerance(ref, ud, tol)
    print(f"largest error over its bound {err.max():.2e}", flush=True)
    assert np.all(err <= 1.0), [CASES[r - LEAD] for r in np.nonzero(err > 1.0)[0] if r >= LEAD]
    # the forms without memory for a part of the factor: the same bits
    thd, out = torch.tensor(th, device="cuda"), torch.zeros(1, dtype=torch.float64, device="cuda")
    sbv.sbv_loglik_noalloc_dev(B, thd, two_nu, out, prec=prec)
    assert out.item() == total
    # one launch of the largest variant for all blocks: the same bits
    monkeypatch.setenv("SBV_PERSISTENT", "1")
    assert sbv.sbv_loglik(B, th, two_nu, prec)[0] == total
    assert np.array_equal(sbv.sbv_blocks_terms(B), lb)
    B.free()


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("d,two_nu", [(2, 1), (3, 5), (12, 7)])
def test_gradients(sbv, d, two_nu, prec):
    X, y, th, _ = _inputs(d, 0.1 if prec else 1e-3)
    S1, _ = _structure(1)
    S0, _ = _structure(0)
    l1, g1 = O.sbv_loglik(X, y, S1, th, two_nu, grad=True)
    l0, g0 = O.sbv_loglik(X[:LEAD], y[:LEAD], S0, th, two_nu, grad=True)
    ref_l, ref_g = l0 + COPIES * (l1 - l0), g0 + COPIES * (g1 - g0)
    B, _ = _handle(sbv, X, y)
    l, g = sbv.sbv_loglik_grad(B, th, two_nu, prec)
    assert _copies_equal(sbv.sbv_blocks_terms(B)[LEAD:].reshape(COPIES, len(CASES)))
    again = sbv.sbv_loglik_grad(B, th, two_nu, prec)
    assert again[0][0] == l[0] and np.array_equal(again[1], g)
    B.free()
    bar32 = 2 * 2.0 ** -24 * 11 * (LEAD + COPIES * sum(j * b for j, b in CASES))
    bar_l, bar_g = (bar32, bar32) if prec else (1e-10 * abs(ref_l), 1e-8 * max(1.0, np.max(np.abs(ref_g))))
    print(f"l {l[0] - ref_l:.2e} of {bar_l:.2e}; g {np.max(np.abs(g - ref_g)):.2e} of {bar_g:.2e}", flush=True)
    assert abs(l[0] - ref_l) <= bar_l
    assert np.max(np.abs(g - ref_g)) <= bar_g


def test_simulation(sbv):
    X, _, th, xi = _inputs(5, 1e-3)
    S1, _ = _structure(1)
    ref = O.sample(X, S1, th, 5, xi)
    B, rows = _handle(sbv, X, None)
    y = sbv.sbv_sample(B, th, 5, xi[rows])
    B.free()
    assert _copies_equal(y[LEAD:].reshape(COPIES, -1))
    assert np.max(np.abs(y[:len(ref)] - ref)) <= 1e-9 * max(1.0, np.max(np.abs(ref)))


def test_captured_before_the_memory_exists(sbv):
    """A caller's capture of an FP64 value on a plan that has only served FP32 runs without
    the memory for a part of the factor; its replays equal the eager value, also after
    eager calls have allocated that memory."""
    import torch
    X, y, th, _ = _inputs(10, 1e-3)
    B, _ = _handle(sbv, X, y)
    thd = torch.tensor(th, device="cuda")
    out, eager = (torch.zeros(1, dtype=torch.float64, device="cuda") for _ in range(2))
    sbv.sbv_loglik_dev(B, thd, 5, out, prec=1, stream=torch.cuda.current_stream())
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        sbv.sbv_loglik_dev(B, thd, 5, out, stream=torch.cuda.current_stream())
    got = []
    for step in range(3):
        thd.copy_(torch.tensor(th + 0.01 * step, device="cuda"))
        g.replay()
        torch.cuda.synchronize()
        sbv.sbv_loglik_dev(B, thd, 5, eager, stream=torch.cuda.current_stream())
        torch.cuda.synchronize()
        got.append((out.item(), eager.item()))
    assert all(a == b and np.isfinite(a) for a, b in got) and len(set(got)) == 3, got
    del g
    B.free()
