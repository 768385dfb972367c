"""Ragged batches whose problems run as pairs of states on coded CSR terms:
problems of unequal degrees, batches of more than one group of states, and what
is reported of non-finite states.  MAGNUS_CODED=2 codes every call,
MAGNUS_PERSIST=0 keeps the small problems out of the one-workgroup kernel."""
import numpy as np
import pytest

from paper_1709_06483_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - collected only where a GPU exists
    pytest.skip("no GPU", allow_module_level=True)

from paper_1709_06483_amd import binding as B  # noqa: E402
from test_gpu_coded import csr, rel, terms  # noqa: E402


@pytest.fixture(autouse=True)
def coded(monkeypatch):
    monkeypatch.setenv("MAGNUS_CODED", "2")
    monkeypatch.setenv("MAGNUS_PERSIST", "0")


def problem(ctx, N, batch, scale=1.0, steps=1, seed=0):
    """Chain-like real terms of N rows times `scale`, with `batch` states and a field per state."""
    A1, A2 = terms("real", N)
    ham = B.magnus_spectral_bounds(ctx, B.DeviceHamiltonian.from_csr(csr(scale * A1), csr(scale * A2)))
    f = np.stack([np.full((steps, 2), 0.3 + 0.4 * b / batch) for b in range(batch)])
    return ham, torch.from_numpy(inputs.random_states(N, seed=N + seed, batch=batch)).cuda(), f


@pytest.mark.parametrize("order", [(0, 1), (1, 0)])
def test_a_problem_that_ends_before_the_others_is_checked(order):
    """Two problems, one of a single iteration an exponential and one of more: the last launch holds
    only the second, and no launch of the first is followed by one that looks at its norms."""
    batch, opts, tau = 4, B.leja_opts(1e-6), 0.05
    ctx = B.Context(max_dim=4000, max_batch=batch)
    both = [problem(ctx, 900, batch, scale=1e-9), problem(ctx, 2000, batch)]
    degree = []
    for p in both:
        st = B.magnus_propagate_ragged(ctx, [p], B.CF4, tau, opts=opts, stats=True)
        assert st["planned_iters"] % st["exponentials"] == 0 and st["substeps"] == st["exponentials"]
        degree.append(st["planned_iters"] // st["exponentials"])
    assert degree[0] == 1 < degree[1]
    B.magnus_propagate_ragged(ctx, [both[k] for k in order], B.CF4, tau, opts=opts, stats=True)
    both[0][1][3, 899] = float("nan")
    with pytest.raises(B.MagnusError) as e:
        B.magnus_propagate_ragged(ctx, [both[k] for k in order], B.CF4, tau, opts=opts, stats=True)
    assert e.value.code == B.ENAN
    ctx.close()


def both_ways(monkeypatch, run):
    out = []
    for mode in ("2", "0"):
        monkeypatch.setenv("MAGNUS_CODED", mode)
        out.append(run())
    return out


# one and two problems of one group, of groups of 32 and 8 states, of 32, 32 and 2, and of as many groups as a
# launch takes; tolerance: each side within the bound of its exponentials (2 steps of 2, 20 times the tolerance each)
@pytest.mark.parametrize("sizes,batch", [([700], 40), ([700, 2001], 40), ([300, 1001], 66), ([200, 333], 128)])
def test_batches_of_several_groups_match_csr_kernels(sizes, batch, monkeypatch):
    tol = 1e-12

    def run():
        ctx = B.Context(max_dim=sum(sizes), max_batch=batch)
        probs = [problem(ctx, N, batch, steps=2) for N in sizes]
        st = B.magnus_propagate_ragged(ctx, probs, B.CF4, 0.3, opts=B.leja_opts(tol), stats=True)
        ctx.close()
        return [p[1].cpu().numpy() for p in probs], st

    (a, sa), (b, sb) = both_ways(monkeypatch, run)
    assert sa["exponentials"] == sb["exponentials"]
    for x, y in zip(a, b):
        assert np.linalg.norm(x - y, axis=1).max() <= 2 * 4 * 20 * tol


def test_a_batch_whose_parameters_exceed_the_table_runs(monkeypatch):
    """5500 states, two exponentials of degree 26: more records than the device table holds when they are
    planned as one group."""
    N, batch, tol = 48, 5500, 1e-12

    def run():
        ctx = B.Context(max_dim=N, max_batch=batch)
        p = problem(ctx, N, batch)
        st = B.magnus_propagate_ragged(ctx, [p], B.CF4, 8.0, opts=B.leja_opts(tol), stats=True)
        ctx.close()
        return p[1].cpu().numpy(), st

    (a, sa), (b, _) = both_ways(monkeypatch, run)
    assert sa["max_degree_used"] * 2 * batch > 1 << 18
    assert np.linalg.norm(a - b, axis=1).max() <= 2 * 2 * 20 * tol


# a single problem, and four whose groups of two states were too many for one launch of the CSR kernels: without
# statistics too the call waits and reports, as batched propagations one after another do
@pytest.mark.parametrize("sizes,batch", [([900], 4), ([300, 700, 200, 500], 6)])
def test_problems_that_do_not_run_jointly_report_at_once(sizes, batch, monkeypatch):
    def run():
        ctx = B.Context(max_dim=sum(sizes) + 300, max_batch=batch)
        probs = [problem(ctx, N, batch) for N in sizes]
        probs[-1][1][1, 7] = float("inf")
        try:
            with pytest.raises(B.MagnusError) as e:
                B.magnus_propagate_ragged(ctx, probs, B.CF4, 0.1)
            return e.value.code
        finally:
            ctx.close()

    assert both_ways(monkeypatch, run) == [B.ENAN, B.ENAN]


@pytest.mark.parametrize("bad", [None, 0, 1])
def test_a_report_beside_small_states(bad, monkeypatch):
    """A problem of pairs that reports at once beside one in the one-workgroup kernel, launched before the wait."""
    monkeypatch.setenv("MAGNUS_PERSIST", "1")

    def run():
        ctx = B.Context(max_dim=6000, max_batch=4)
        probs = [problem(ctx, 300, 4), problem(ctx, 5500, 4)]
        if bad is not None:
            probs[bad][1][2, 7] = float("nan")
        try:
            B.magnus_propagate_ragged(ctx, probs, B.CF4, 0.1)
            return [p[1].cpu().numpy() for p in probs] if bad is None else 0
        except B.MagnusError as e:
            return e.code
        finally:
            ctx.close()

    a, b = both_ways(monkeypatch, run)
    if bad is None:
        assert all(rel(x, y) < 1e-9 for x, y in zip(a, b))
    else:
        assert [a, b] == [B.ENAN if bad else 0] * 2
