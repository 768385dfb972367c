"""Where one small state of terms that fit neither registers nor the coded form
runs: in one workgroup while it reads at most 12,000 entries from memory (term 1
of up to 6,400 entries lies in LDS), on the grid from there on; each against the
oracle, and with term 1 in LDS bitwise as without."""
import ctypes as C

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
from test_gpu_coded import csr, oracle, rel  # noqa: E402

TOL = 1e-12


def shifts(N, per, seed):
    """Hermitian, `per` complex entries in every row, all different."""
    rng = np.random.default_rng(seed)
    M = sp.csr_matrix((N, N), dtype=np.complex128)
    for s in rng.choice(np.arange(1, (N + 1) // 2), per // 2, replace=False):
        v = 0.1 * (rng.standard_normal(N) + 1j * rng.standard_normal(N))
        U = sp.csr_matrix((v, (np.arange(N), (np.arange(N) + s) % N)), shape=(N, N))
        M = M + U + U.conj().T
    return sp.csr_matrix(M)


def run(A1, A2, f, psi0):
    ctx = B.Context(max_dim=len(psi0))
    ham = B.magnus_spectral_bounds(ctx, B.DeviceHamiltonian.from_csr(csr(A1), csr(A2)))
    psi = torch.from_numpy(psi0).cuda()
    B._check(B.lib().magnus_timing(ctx.handle, 1))
    B.propagate(ctx, ham, B.CF4, 0.05, f, psi, opts=B.leja_opts(TOL))
    ms, launches = C.c_double(), C.c_int64()
    B._check(B.lib().magnus_timing_read(ctx.handle, B.KERNEL_PERSIST, C.byref(ms), C.byref(launches)))
    out = psi.cpu().numpy()
    ctx.close()
    return out, launches.value


@pytest.mark.parametrize("N,per1,per2,small", [
    (400, 14, 8, True),      # 5,600 entries of term 1 in LDS, up to 512 rows
    (512, 10, 22, True),     # 11,264 read from memory
    (512, 12, 24, False),    # 12,288
    (512, 16, 8, False),     # 8,192 entries of term 1: too many for LDS, 12,288 read
    (1024, 6, 10, True),     # 513 to 1,024 rows, 6,144 in LDS and 10,240 read
    (1024, 6, 12, False),
    (1023, 8, 4, False)])
def test_one_small_state(N, per1, per2, small, monkeypatch):
    A1, A2 = shifts(N, per1, 1), shifts(N, per2, 2)
    f = np.array([[0.3, 0.5], [0.6, 0.2]])
    psi0 = inputs.random_states(N, seed=N)
    got, launches = run(A1, A2, f, psi0)
    assert (launches > 0) == small
    ref = psi0
    for n in range(2):
        for w in ((mg.CF4_ALPHA2, mg.CF4_ALPHA1), (mg.CF4_ALPHA1, mg.CF4_ALPHA2)):
            ref = oracle(A1, A2, 0.5, w[0] * f[n, 0] + w[1] * f[n, 1], 0.0, 0.05, ref)
    assert rel(got, ref) <= 4 * 20 * TOL
    if small:
        monkeypatch.setenv("MAGNUS_PERSIST_CACHE", "0")
        monkeypatch.setenv("MAGNUS_PERSIST", "2")
        assert np.array_equal(run(A1, A2, f, psi0)[0], got)

