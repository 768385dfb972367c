"""The gradient on coded CSR terms, its block exponentials two pairs to a launch,
against the same call on the CSR arrays."""
import numpy as np
import pytest

from oracle import magnus as mg
from paper_1709_06483_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - collected only where a GPU exists
    pytest.skip("no GPU", allow_module_level=True)

from paper_1709_06483_amd import binding as B  # noqa: E402
from test_gpu_coded import csr, terms  # noqa: E402


def gradient(monkeypatch, coded, A1, A2, tau, f, df, every_k, tol):
    monkeypatch.setenv("MAGNUS_CODED", coded)
    N = A1.shape[0]
    ctx = B.Context(max_dim=N, max_batch=2)
    ham = B.magnus_spectral_bounds(ctx, B.DeviceHamiltonian.from_csr(csr(A1), csr(A2)))
    psi0, target = (torch.from_numpy(inputs.random_states(N, seed=N + k)).cuda() for k in (1, 2))
    loss, grad, st = B.magnus_propagate_adjoint(ctx, ham, tau, f, df, psi0, target, every_k=every_k,
                                                opts=B.leja_opts(tol, tol_mode=1), stats=True)
    radius = max(abs(ham.struct.H2.lam_min), abs(ham.struct.H2.lam_max))
    ctx.close()
    return loss, grad, st, radius


def allowed(tau, df, radius, tol):
    """Both sides: z within the budget of its run (20 times, as elsewhere), and each block exponential's coupling,
    of norm at most tau |H2| times the derivative of its field, within as much of that norm; the gradient is
    2 Re(conj(z) dz) with |z| <= 1."""
    w = np.abs([mg.CF4_ALPHA1, mg.CF4_ALPHA2])
    reach = tau * radius * np.sum(np.abs(df) * w.sum(), axis=(0, 1))
    return 2 * 2 * 20 * tol, 2 * 2 * 2 * 20 * tol * np.maximum(reach, 1.0)


def test_a_segment_that_fits_the_table_one_pair_at_a_time(monkeypatch):
    """Half steps of degrees so unequal that the two pairs of a step, which share the larger, need more
    records than the device table holds, and one after the other do not."""
    N, steps, tau, tol = 64, 4800, 0.02, 1e-9
    A1, A2 = terms("real", N)
    f = np.tile([9.0, 9.0 * -mg.CF4_ALPHA2 / mg.CF4_ALPHA1], (steps, 1))  # no field in the first half step
    df = np.cos(np.arange(2 * steps)).reshape(steps, 2, 1) / steps
    (l1, g1, s1, radius), (l0, g0, s0, _) = (gradient(monkeypatch, c, A1, A2, tau, f, df, steps, tol) for c in ("2", "0"))
    lt, gt = allowed(tau, df, radius, tol)
    assert abs(l1 - l0) <= lt and np.all(np.abs(g1 - g0) <= gt)
    assert s1["planned_iters"] == s0["planned_iters"]  # (one pair at a time on both sides)
    # what two pairs to a launch would take, and what one pair at a time takes
    assert 4 * s0["max_degree_used"] * steps > 1 << 18


# one number a value and two, one term imaginary, a diagonal in H2, blocks of rows that are read from the CSR
# arrays, rows of more rounds than are loaded ahead; partial slices and blocks; one substep and several (whose
# sums alternate between two buffers); segments recomputed
@pytest.mark.parametrize("tau", [0.05, 20.0])
@pytest.mark.parametrize("kind,N", [("real", 17), ("imaginary", 65), ("complex", 1000), ("too many", 300), ("too many", 4133),
                                    ("wide", 300), ("empty", 1000)])
def test_block_exponentials_of_all_kinds_of_terms(kind, N, tau, monkeypatch):
    steps, tol = 5, 1e-10
    A1, A2 = terms(kind, N)
    f = 0.3 + 0.1 * np.arange(2 * steps).reshape(steps, 2)
    df = np.cos(np.arange(4 * steps)).reshape(steps, 2, 2)
    (l1, g1, s1, radius), (l0, g0, s0, _) = (gradient(monkeypatch, c, A1, A2, tau, f, df, 2, tol) for c in ("2", "0"))
    lt, gt = allowed(tau, df, radius, tol)
    assert abs(l1 - l0) <= lt and np.all(np.abs(g1 - g0) <= gt)
    assert (s1["max_substeps_used"] > 1) == (tau > 1)
