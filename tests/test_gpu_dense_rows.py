"""The dense iterations' split of the matrix: the rows in equal shares over at most
512 workgroups, the columns over the 256 lanes of each."""
import numpy as np
import pytest

from oracle import magnus as mg
from paper_1709_06483_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - collected only where a GPU exists
    pytest.skip("no GPU", allow_module_level=True)

from paper_1709_06483_amd import binding as B  # noqa: E402

BUDGET = 1e-10  # the tolerance asked of the propagation, far above 24 products' rounding (about 1e-14)


@pytest.mark.parametrize("rpw", ["1", "2", "4"])
@pytest.mark.parametrize("N", [3, 256, 511, 513, 1025])
def test_dense_row_and_column_remainders_match_oracle(N, rpw, monkeypatch):
    """One column step and one row per workgroup (up to 512 rows), and sizes where some
    workgroups have one row or column step more than others: two terms with a padded
    row stride, the assembled exponent and its fused first iteration, with M4's
    commutator too."""
    monkeypatch.setenv("MAGNUS_DENSE_RPW", rpw)
    H0 = inputs.powerlaw_hermitian(N, 1.5, seed=60)
    V = inputs.powerlaw_hermitian(N, 1.5, seed=61)
    f = inputs.sin_field(1.0, 2.0)
    psi0 = inputs.random_states(N, seed=62)
    tau, nsteps = 0.01, 3
    pads = [torch.full((N, N + 3), float("nan"), dtype=torch.complex128, device="cuda") for _ in range(2)]
    for p, h in zip(pads, (H0, V)):
        p[:, :N] = torch.from_numpy(np.ascontiguousarray(h)).cuda()
    for method, assembled in (("CF4", False), ("CF4", True), ("M4", True)):
        c = B.Context(max_dim=N)
        if assembled:
            c.reserve_dense(N)
        ham = B.magnus_spectral_bounds(c, B.DeviceHamiltonian.from_dense(pads[0][:, :N], pads[1][:, :N]))
        if method == "M4":
            B.magnus_dense_commutator(c, ham)
        fn = np.vectorize(f)(B.magnus_quadrature_nodes(B.METHODS[method], 0.0, tau, nsteps))
        psi = torch.from_numpy(np.ascontiguousarray(psi0)).cuda()
        B.propagate(c, ham, B.METHODS[method], tau, fn, psi, opts=B.leja_opts(BUDGET, tol_mode=1))
        out = psi.cpu().numpy()
        ref = mg.propagate(method, mg.two_term(H0, V, f), tau, nsteps, psi0, expm="eig")
        assert np.linalg.norm(out - ref) <= BUDGET * np.linalg.norm(ref), (method, assembled)
        c.close()
