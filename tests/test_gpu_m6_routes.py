"""Method M6 on the CSR arrays in two passes over H1, H2, K, P1 and P2 and in
three over H1, H2 and K, whichever the rows of P1 and P2 make the faster: terms
on either side of the rule at sizes on either side of its lines, with the stop
test fused and by the decide kernel (always past 32,768 rows), against the
oracle's nested commutators."""
import numpy as np
import pytest
import scipy.sparse as sp

from oracle import magnus as mg
from paper_1709_06483_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - collected only where a GPU exists
    pytest.skip("no GPU", allow_module_level=True)

from paper_1709_06483_amd import binding as B  # noqa: E402
from test_gpu_coded import bands, rel  # noqa: E402
from test_gpu_m6_passes import BUDGET, TAU, field, run  # noqa: E402
from test_gpu_small_routes import shifts  # noqa: E402


def commutator(A, C):
    K = sp.csr_matrix(A @ C - C @ A)
    K.eliminate_zeros()
    return K


def make(kind, N):
    d = np.random.default_rng(N).standard_normal(N)
    if kind == "short":  # at most ten entries of P1 and P2 a row
        return bands(N, [1], [0.6], d), bands(N, [1], [0.5j])
    return shifts(N, 6, 1) * 2.0, shifts(N, 4, 2) * 2.0  # about three times as many entries of P1 and P2 as of the others


@pytest.mark.parametrize("fuse", ["1", "0"])
@pytest.mark.parametrize("kind,N,two", [("short", 513, True), ("short", 20000, True), ("short", 40001, True),
                                        ("filled", 29, True), ("filled", 700, False), ("filled", 4133, False),
                                        ("filled", 33000, False)])
def test_passes_match_oracle(kind, N, two, fuse, monkeypatch):
    monkeypatch.setenv("MAGNUS_CODED", "0")
    monkeypatch.setenv("MAGNUS_FUSE", fuse)
    A1, A2 = make(kind, N)
    K = commutator(A1, A2)
    P = sum(commutator(A, K).nnz for A in (A1, A2))
    H = A1.nnz + A2.nnz + K.nnz
    # (the rule, with room on either side)
    assert P <= 9 * N or N <= 500 and P <= 60 * N if two else P > 2.5 * H
    fn = np.vectorize(field)(B.magnus_quadrature_nodes(B.M6, 0.0, TAU, 1))
    psi0 = inputs.random_states(N, seed=N + 1)
    out, _ = run(A1, A2, fn, TAU, psi0)
    ref = mg.propagate("M6", mg.two_term(A1, A2, field), TAU, 1, psi0, expm="taylor")
    assert rel(out, ref) <= BUDGET
