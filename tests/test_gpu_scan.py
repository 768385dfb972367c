"""The scan of both CSR terms behind one wait: malformed arrays of either term
are refused (nothing reads past them, the coding that follows on the stream
included), the other term's enclosure is as it was before, and a sound pair
afterwards is scanned and coded as ever."""
import numpy as np
import pytest

from paper_1709_06483_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - collected only where a GPU exists
    pytest.skip("no GPU", allow_module_level=True)

from paper_1709_06483_amd import binding as B  # noqa: E402
from test_gpu_coded import csr, oracle, rel, terms  # noqa: E402

N = 3000


@pytest.mark.parametrize("which", [0, 1])
@pytest.mark.parametrize("fault", ["decreasing", "past the end", "negative", "short", "column", "negative column"])
def test_malformed_terms_are_refused(which, fault):
    A = terms("real", N)
    ctx = B.Context(max_dim=N)
    ham = B.DeviceHamiltonian.from_csr(csr(A[0]), csr(A[1]))
    rp, ci = ham.tensors[3 * which], ham.tensors[3 * which + 1]
    keep = rp.clone(), ci.clone()
    if fault == "decreasing":
        rp[1500], rp[1501] = rp[1501].item(), rp[1500].item() - 1
    elif fault == "past the end":
        rp[1500:] = 1 << 30
    elif fault == "negative":
        rp[7] = -5
    elif fault == "short":
        rp[N] = rp[N].item() - 3
    else:
        ci[4000] = N if fault == "column" else -1
    for T in (ham.struct.H1, ham.struct.H2):
        T.lam_min, T.lam_max = -99.0, 98.0
    with pytest.raises(B.MagnusError) as e:
        B.magnus_spectral_bounds(ctx, ham)
    assert e.value.code == B.EINVAL
    # term 1 sound: its enclosure is set before term 2 is refused
    assert (ham.struct.H1.lam_min != -99.0) == (which == 1) and ham.struct.H2.lam_min == -99.0
    rp.copy_(keep[0])
    ci.copy_(keep[1])
    B.magnus_spectral_bounds(ctx, ham)
    radius = [abs(M).sum(axis=1).max() for M in A]
    for T, r in zip((ham.struct.H1, ham.struct.H2), radius):
        assert max(-T.lam_min, T.lam_max) <= r * (1 + 1e-12)
    v = inputs.random_states(N, seed=1)
    w = B.expmv_leja(ctx, ham, 0.6, -0.4, 0.0, 0.1, torch.from_numpy(v).cuda(), opts=B.leja_opts(1e-12))
    assert rel(w.cpu().numpy(), oracle(A[0], A[1], 0.6, -0.4, 0.0, 0.1, v)) <= 20 * 1e-12
    ctx.close()
