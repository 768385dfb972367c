"""Leja iterations on coded CSR terms (a dictionary of (column - row, value)
pairs per block of rows and a byte per entry) against the CPU oracle and the
kernels that read the CSR arrays: real, imaginary and complex values, terms
with and without a diagonal, rows of up to 64 entries of a term and 128 of all
(more than the iteration loads ahead), blocks that do not fit the form, sizes
around the edges of slices and blocks, arrays rewritten in place between calls,
and the decide kernel in place of the fused stop test.  MAGNUS_CODED=2 codes
every call.  Tolerance: 20 times the tolerance of one exponential, as for the
other CSR kernels."""
import numpy as np
import pytest
import scipy.sparse as sp

from oracle import expm as oe
from oracle.linop import Mat
from oracle import magnus as mg
from paper_1709_06483_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - collected only where a GPU exists
    pytest.skip("no GPU", allow_module_level=True)

from paper_1709_06483_amd import binding as B  # noqa: E402


def rel(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


def bands(N, offsets, values, diag=None):
    """Hermitian: values[k] on the entries (r, r + offsets[k]), its conjugate below, diag (or none)."""
    M = sp.csr_matrix((N, N), dtype=np.complex128)
    for o, v in zip(offsets, values):
        if o < N:
            U = sp.diags([np.full(N - o, v)], [o], shape=(N, N), dtype=np.complex128)
            M = M + U + U.conj().T
    if diag is not None:
        M = M + sp.diags([np.asarray(diag, dtype=np.complex128)], [0])
    return sp.csr_matrix(M)


def csr(M):
    M = sp.csr_matrix(M)
    M.sort_indices()
    return inputs.CSR(M.indptr.astype(np.int32), M.indices.astype(np.int32), M.data.astype(np.complex128), M.shape[0])


def terms(kind, N):
    rng = np.random.default_rng(N)
    d = rng.standard_normal(N)
    if kind == "real":
        return bands(N, [1, 5], [0.7, -0.3], d), bands(N, [2, 40], [0.5, 0.25])
    if kind == "imaginary":  # H2 like a sigma^y field: one number a value, a rotated product
        return bands(N, [1, 3], [0.6, 0.2], d), bands(N, [1, 7], [0.5j, -0.4j], 0.1 * d)
    if kind == "complex":
        return bands(N, [1, 9], [0.5 + 0.3j, 0.2 - 0.6j], d), bands(N, [4], [0.3j + 0.1], d[::-1])
    if kind == "empty":  # no entry at all in H2, and half of H1's rows empty
        M = bands(N, [2], [0.8]).tolil()
        M[::2] = 0
        M[:, ::2] = 0
        return sp.csr_matrix(M), sp.csr_matrix((N, N), dtype=np.complex128)
    if kind == "wide":  # 62 entries of H1 and 20 of H2 a row: 21 rounds, past the words loaded ahead
        return (bands(N, list(range(1, 32)), list(0.02 * (1 + np.arange(31))), d),
                bands(N, list(range(3, 13)), list(0.05j * np.ones(10))))
    if kind == "too wide":  # 80 entries a row: no block fits
        return bands(N, list(range(1, 41)), list(0.01 * (1 + np.arange(40))), d), bands(N, [1], [0.5])
    if kind == "too many":  # rows 64 .. 127 all of different values: one block does not fit
        M = bands(N, [1, 3, 6], [0.4, 0.2, 0.1], d).tolil()
        for r in range(64, min(128, N - 6)):
            for o in (1, 3, 6):
                v = complex(*rng.standard_normal(2)) * 0.3
                M[r, r + o] = v
                M[r + o, r] = np.conj(v)
        return sp.csr_matrix(M), bands(N, [2], [0.5], d)
    raise ValueError(kind)


def oracle(A1, A2, a, b, kappa, tau, v):
    S = a * A1 + b * A2
    if kappa:
        S = S + kappa * 1j * (A1 @ A2 - A2 @ A1)
    return oe.expmv_taylor(Mat(-1j * tau * sp.csr_matrix(S)), v)


@pytest.mark.parametrize("kind", ["real", "imaginary", "complex", "empty", "wide", "too wide", "too many"])
@pytest.mark.parametrize("N", [1, 15, 16, 17, 64, 65, 1000, 4133])
def test_coded_exponentials_match_oracle(kind, N, monkeypatch):
    monkeypatch.setenv("MAGNUS_CODED", "2")
    A1, A2 = terms(kind, N)
    v = inputs.random_states(N, seed=N)
    tol = 1e-12
    ctx = B.Context(max_dim=N)
    ham = B.magnus_spectral_bounds(ctx, B.DeviceHamiltonian.from_csr(csr(A1), csr(A2)))
    vd = torch.from_numpy(v).cuda()
    for kappa in (0.0, 0.02):  # the commutator applied to vectors
        w = B.expmv_leja(ctx, ham, 0.6, -0.4, kappa, 0.1, vd, opts=B.leja_opts(tol)).cpu().numpy()
        assert rel(w, oracle(A1, A2, 0.6, -0.4, kappa, 0.1, v)) <= 20 * tol, kappa
    if "wide" not in kind:  # (its commutator is assembled too, three terms)
        B.magnus_csr_commutator(ctx, ham)
        w = B.expmv_leja(ctx, ham, 0.6, -0.4, 0.02, 0.1, vd, opts=B.leja_opts(tol)).cpu().numpy()
        assert rel(w, oracle(A1, A2, 0.6, -0.4, 0.02, 0.1, v)) <= 20 * tol
    ctx.close()


# blocks of 64, 128, 256 and 512 rows (one, two and four slices to a wave, several passes), ragged ends
@pytest.mark.parametrize("N", [65536, 65537, 131073, 262145, 300007])
@pytest.mark.parametrize("kind", ["real", "complex", "too many"])
def test_coded_propagation_matches_csr_kernels(N, kind, monkeypatch):
    A1, A2 = terms(kind, N)
    H1, H2 = csr(A1), csr(A2)
    v = inputs.random_states(N, seed=3)
    f = np.array([[0.3, 0.5], [0.6, 0.2]])
    out = []
    for coded, fuse in (("0", "1"), ("2", "1"), ("2", "0")):
        monkeypatch.setenv("MAGNUS_CODED", coded)
        monkeypatch.setenv("MAGNUS_FUSE", fuse)
        ctx = B.Context(max_dim=N)
        ham = B.magnus_spectral_bounds(ctx, B.DeviceHamiltonian.from_csr(H1, H2))
        psi = torch.from_numpy(v).cuda()
        _, st = B.propagate(ctx, ham, B.CF4, 0.05, f, psi, opts=B.leja_opts(1e-12), stats=True)
        out.append((psi.cpu().numpy(), st["iters"]))
        ctx.close()
    assert out[0][1] == out[1][1] == out[2][1]
    assert rel(out[1][0], out[0][0]) <= 1e-13
    assert rel(out[2][0], out[0][0]) <= 1e-13


@pytest.mark.parametrize("coded", ["1", "2"])
def test_terms_rewritten_in_place_are_coded_as_they_are(coded, monkeypatch):
    """The values of a term that fitted the form are replaced between calls, by others that fit it and
    by others that do not (all different); no call may use what an earlier one coded."""
    monkeypatch.setenv("MAGNUS_CODED", coded)
    N = 70001
    A1, A2 = terms("real", N)
    H1, H2 = csr(A1), csr(A2)
    ctx = B.Context(max_dim=N)
    ham = B.DeviceHamiltonian.from_csr(H1, H2)
    B.magnus_spectral_bounds(ctx, ham)
    for T in (ham.struct.H1, ham.struct.H2):
        T.lam_min, T.lam_max = 2 * T.lam_min, 2 * T.lam_max  # room for the new values
    v = inputs.random_states(N, seed=5)
    rng = np.random.default_rng(5)
    w = sp.triu(A1, 1).tocsr()
    w.data = rng.uniform(-0.5, 0.5, w.nnz).astype(np.complex128)
    changed = [A1, 0.5 * A1, w + w.conj().T + sp.diags(A1.diagonal())]
    for M in changed:
        H = csr(M)
        assert np.array_equal(H.indices, H1.indices)
        ham.tensors[2].copy_(torch.from_numpy(H.data))
        got = B.expmv_leja(ctx, ham, 0.5, 0.3, 0.0, 0.1, torch.from_numpy(v).cuda(), opts=B.leja_opts(1e-12))
        assert rel(got.cpu().numpy(), oracle(M, A2, 0.5, 0.3, 0.0, 0.1, v)) <= 20 * 1e-12
    ctx.close()


def test_coded_non_finite_state_is_reported(monkeypatch):
    monkeypatch.setenv("MAGNUS_CODED", "2")
    N = 5000
    A1, A2 = terms("real", N)
    ctx = B.Context(max_dim=N)
    ham = B.magnus_spectral_bounds(ctx, B.DeviceHamiltonian.from_csr(csr(A1), csr(A2)))
    x = inputs.random_states(N, seed=2)
    x[17] = np.inf
    with pytest.raises(B.MagnusError) as e:
        B.expmv_leja(ctx, ham, 1.0, 0.5, 0.0, 0.1, torch.from_numpy(x).cuda(), stats=True)
    assert e.value.code == B.ENAN
    ctx.close()


@pytest.mark.parametrize("comm", [False, True])
def test_coded_m4_run_matches_oracle(comm, monkeypatch):
    monkeypatch.setenv("MAGNUS_CODED", "2")
    n, steps, tau = 9, 4, 0.02
    H1, H2 = inputs.chain_terms(n)
    f = inputs.cos_field(2.0)
    psi0 = inputs.random_states(1 << n, seed=11)
    ctx = B.Context(max_dim=1 << n)
    ham = B.magnus_spectral_bounds(ctx, B.DeviceHamiltonian.from_csr(H1, H2))
    if comm:
        B.magnus_csr_commutator(ctx, ham)
    psi = torch.from_numpy(psi0).cuda()
    B.propagate(ctx, ham, B.M4, tau, np.vectorize(f)(B.magnus_quadrature_nodes(B.M4, 0.0, tau, steps)), psi,
                opts=B.leja_opts(1e-12))
    ref = mg.propagate("M4", mg.two_term(H1.to_scipy(), H2.to_scipy(), f), tau, steps, psi0, expm="taylor")
    assert rel(psi.cpu().numpy(), ref) <= 20 * 1e-12 * steps
    ctx.close()


def batch_run(monkeypatch, coded, H1, H2, psi0, f, tol=1e-12, widen=1.0):
    monkeypatch.setenv("MAGNUS_CODED", coded)
    monkeypatch.setenv("MAGNUS_PERSIST", "0")
    ctx = B.Context(max_dim=H1.dim, max_batch=psi0.shape[0])
    ham = B.magnus_spectral_bounds(ctx, B.DeviceHamiltonian.from_csr(H1, H2))
    for T in (ham.struct.H1, ham.struct.H2):
        c, r = 0.5 * (T.lam_min + T.lam_max), 0.5 * (T.lam_max - T.lam_min)
        T.lam_min, T.lam_max = c - widen * r, c + widen * r
    psi = torch.from_numpy(psi0).cuda()
    _, st = B.propagate(ctx, ham, B.CF4, 0.05, f, psi, opts=B.leja_opts(tol), stats=True)
    ctx.close()
    return psi.cpu().numpy(), st


# pairs, pairs and a single state, eight pairs (an XCD per pair) and more; each state with its own field, so
# with its own degree and stop; enclosures widened so that early termination cuts the a priori degree
@pytest.mark.parametrize("batch", [2, 3, 5, 16, 21])
@pytest.mark.parametrize("kind,N", [("real", 1000), ("imaginary", 65), ("complex", 1000), ("wide", 300), ("too many", 4133),
                                    ("empty", 17)])
def test_coded_batches_match_oracle(kind, N, batch, monkeypatch):
    A1, A2 = terms(kind, N)
    psi0 = inputs.random_states(N, seed=N + batch, batch=batch)
    f = np.stack([np.array([[0.2, 0.4], [0.5, 0.1]]) * (0.2 + b) for b in range(batch)])
    got, st = batch_run(monkeypatch, "2", csr(A1), csr(A2), psi0, f, widen=2.0)
    want, sw = batch_run(monkeypatch, "0", csr(A1), csr(A2), psi0, f, widen=2.0)
    if batch != 21:  # (20 + 1 states on coded terms, 16 + 4 + 1 else: a group shares the largest substep count)
        assert st["iters"] == sw["iters"] and st["planned_iters"] == sw["planned_iters"]
        assert rel(got, want) <= 1e-13
    for b in (0, batch - 1):
        ref = psi0[b]
        for n in range(2):
            for w in ((mg.CF4_ALPHA2, mg.CF4_ALPHA1), (mg.CF4_ALPHA1, mg.CF4_ALPHA2)):
                ref = oracle(A1, A2, 0.5, w[0] * f[b, n, 0] + w[1] * f[b, n, 1], 0.0, 0.05, ref)
        assert rel(got[b], ref) <= 20 * 1e-12 * 4


# one block of rows (several passes of a wave), blocks of 64 to 1024 rows
@pytest.mark.parametrize("N,batch", [(65536, 2), (70001, 4), (262145, 2), (262145, 16)])
def test_coded_batches_match_csr_kernels(N, batch, monkeypatch):
    A1, A2 = terms("real", N)
    psi0 = inputs.random_states(N, seed=1, batch=batch)
    f = np.array([[0.3, 0.5]])
    got, st = batch_run(monkeypatch, "1", csr(A1), csr(A2), psi0, f)
    want, sw = batch_run(monkeypatch, "0", csr(A1), csr(A2), psi0, f)
    assert st["iters"] == sw["iters"]
    assert rel(got, want) <= 1e-13


def test_coded_ragged_batch_matches_csr_kernels(monkeypatch):
    monkeypatch.setenv("MAGNUS_PERSIST", "0")
    sizes, batch = [("real", 300), ("complex", 5000), ("too many", 20011)], 6
    out = []
    for coded in ("2", "0"):
        monkeypatch.setenv("MAGNUS_CODED", coded)
        ctx = B.Context(max_dim=sum(N for _, N in sizes), max_batch=batch)
        probs = []
        for kind, N in sizes:
            ham = B.magnus_spectral_bounds(ctx, B.DeviceHamiltonian.from_csr(*map(csr, terms(kind, N))))
            f = np.stack([np.array([[0.2, 0.4], [0.5, 0.1], [0.3, 0.3]]) * (0.5 + b) for b in range(batch)])
            probs.append((ham, torch.from_numpy(inputs.random_states(N, seed=N, batch=batch)).cuda(), f))
        B.magnus_propagate_ragged(ctx, probs, B.CF4, 0.05, opts=B.leja_opts(1e-12))
        out.append([p.cpu().numpy() for _, p, _ in probs])
        ctx.close()
    # groups of 6 states against groups of 2, so other substep counts: each side within its six exponentials' bound
    for a, b in zip(*out):
        assert rel(a, b) <= 2 * 6 * 20 * 1e-12


def test_coded_batch_reports_a_non_finite_state(monkeypatch):
    monkeypatch.setenv("MAGNUS_CODED", "2")
    monkeypatch.setenv("MAGNUS_PERSIST", "0")
    N = 2000
    ctx = B.Context(max_dim=N, max_batch=4)
    ham = B.magnus_spectral_bounds(ctx, B.DeviceHamiltonian.from_csr(*map(csr, terms("real", N))))
    x = inputs.random_states(N, seed=2, batch=4)
    x[2, 1999] = np.nan
    with pytest.raises(B.MagnusError) as e:  # a plan of one iteration: only the check at the end sees it
        B.expmv_leja(ctx, ham, 1.0, 0.5, 0.0, 1e-7, torch.from_numpy(x).cuda(), opts=B.leja_opts(1e-6), stats=True)
    assert e.value.code == B.ENAN
    ctx.close()
