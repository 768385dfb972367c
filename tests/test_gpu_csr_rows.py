"""The CSR iterations that give eight lanes to a row: two terms, the commutator
applied to vectors in two passes, and three terms with it assembled; real, complex
and empty rows, rows of more entries than one batch of loads holds, partial
workgroups, both workgroup sizes, and the decide kernel in place of the fused stop
test.  Tolerance: 20 times the tolerance of one exponential, as for the other CSR
kernels."""
import pytest

from paper_1709_06483_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - collected only where a GPU exists
    pytest.skip("no GPU", allow_module_level=True)

from paper_1709_06483_amd import binding as B  # noqa: E402
from test_gpu_coded import csr, oracle, rel, terms  # noqa: E402

TOL = 1e-12


def exponentials(A1, A2, v, assembled=True):
    """exp(-0.1 i (0.6 H1 - 0.4 H2 + kappa K)) v with kappa = 0, with K in two passes, and assembled."""
    ctx = B.Context(max_dim=len(v))
    ham = B.magnus_spectral_bounds(ctx, B.DeviceHamiltonian.from_csr(csr(A1), csr(A2)))
    vd = torch.from_numpy(v).cuda()
    out = []
    for kappa in (0.0, 0.02) + ((0.02,) if assembled else ()):
        if len(out) == 2:
            B.magnus_csr_commutator(ctx, ham)
        out.append(B.expmv_leja(ctx, ham, 0.6, -0.4, kappa, 0.1, vd, opts=B.leja_opts(TOL)).cpu().numpy())
    ctx.close()
    return out


@pytest.mark.parametrize("fuse", ["1", "0"])
@pytest.mark.parametrize("kind", ["real", "complex", "empty", "wide", "too wide"])
@pytest.mark.parametrize("N", [1, 7, 31, 33, 1000, 4133])
def test_eight_lane_rows_match_oracle(kind, N, fuse, monkeypatch):
    monkeypatch.setenv("MAGNUS_CODED", "0")
    monkeypatch.setenv("MAGNUS_FUSE", fuse)
    A1, A2 = terms(kind, N)
    v = inputs.random_states(N, seed=N + 5)
    got = exponentials(A1, A2, v, assembled="wide" not in kind)
    for w, kappa in zip(got, (0.0, 0.02, 0.02)):
        assert rel(w, oracle(A1, A2, 0.6, -0.4, kappa, 0.1, v)) <= 20 * TOL, kappa


# the sizes where the mapping changes, and its largest grids
@pytest.mark.parametrize("N", [28671, 28672, 49151, 49152, 65535, 65536, 65537, 131071, 131072, 131073])
def test_eight_lane_rows_match_other_mappings(N, monkeypatch):
    monkeypatch.setenv("MAGNUS_CODED", "0")
    A1, A2 = terms("complex", N)
    v = inputs.random_states(N, seed=4)
    runs = []
    for variant in ("0", "1", "5"):  # the rule, eight lanes (nonzero streaming past 131,072), wave tiles
        monkeypatch.setenv("MAGNUS_CSR_VARIANT", variant)
        runs.append(exponentials(A1, A2, v))
    for got in runs[:2]:
        for w, ref in zip(got, runs[2]):
            assert rel(w, ref) <= 1e-13
