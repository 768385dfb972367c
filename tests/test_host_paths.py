"""The library's host code on the CPU, against a stand-in for the HIP runtime
(hip_stub.cpp: host memory for device memory, kernels logged and not run): which
kernels a call launches, what it allocates, and what it does when memory is
short.  Each test runs in a process of its own, so that the stand-in's symbols
come before the real runtime's."""
import os
import subprocess
import sys
import textwrap

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))

PRELUDE = """
import ctypes as C, sys
stub = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
stub.stub_live.restype = C.c_size_t
stub.stub_limit.argtypes = [C.c_size_t]
stub.stub_log.restype = C.c_char_p
stub.stub_cost.argtypes = [C.c_char_p, C.c_double]
stub.stub_watch.argtypes = [C.c_char_p, C.c_int]
stub.stub_fill.argtypes = [C.c_char_p, C.c_int, C.c_int, C.c_int]
import numpy as np
from paper_1709_06483_amd import binding as B
L = B.lib()
keep = []

def context(max_dim, max_batch=1):
    h = C.c_void_p()
    B._check(L.magnus_create(C.byref(h), max_dim, max_batch, 0))
    return h

def term(N, per=1, radius=1.0):
    # `per` entries in every row, all of column 0 (the values are zeros)
    rp = (np.arange(N + 1) * per).astype(np.int32); ci = np.zeros(max(N * per, 1), np.int32); va = np.zeros(2 * max(N * per, 1))
    keep.extend((rp, ci, va))
    return B.Term(B.CSR, 0, N, N * per, 0, rp.ctypes.data, ci.ctypes.data, va.ctypes.data, -radius, radius)

def ham(ctx, N, per=1, radius=1.0):
    h = B.Hamiltonian(term(N, per, radius), term(N, per, radius), -1.0, 1.0)
    B._check(L.magnus_spectral_bounds(ctx, C.byref(h), None))
    for t in (h.H1, h.H2):
        t.lam_min, t.lam_max = -radius, radius
    h.k_min, h.k_max = -2 * radius**2, 2 * radius**2
    return h

def vector(n):
    v = np.zeros(2 * n); keep.append(v)
    return v.ctypes.data

def opts(tol=1e-10):
    return C.byref(B.LejaOpts(tol, 64, 1 << 20, 1, 0))

def launched(f):
    # (names of the kernels that f launches, in order)
    stub.stub_clear()
    B._check(f())
    return stub.stub_log().decode().split()

def propagate(ctx, h, method=B.CF4, steps=2, batch=1, tau=0.1):
    f = np.linspace(0.2, 0.9, steps * L.magnus_method_nodes(method)); keep.append(f)
    return L.propagate(ctx, C.byref(h), method, tau, steps, B._dptr(f), 1, vector(h.H1.dim * batch), batch, None, 1,
                       opts(), None, None)
"""


@pytest.fixture(scope="session")
def stub(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("stub") / "libhipstub.so")
    subprocess.run(["g++", "-O1", "-shared", "-fPIC", "-std=c++17", "-o", out, os.path.join(HERE, "hip_stub.cpp")], check=True)
    return out


def run(stub, body, **env):
    p = subprocess.run([sys.executable, "-c", PRELUDE + textwrap.dedent(body), stub], cwd=os.path.dirname(HERE),
                       env={**os.environ, **env}, capture_output=True, text=True, timeout=300)
    assert p.returncode == 0, p.stdout + p.stderr


@pytest.mark.parametrize("N,single,two_pass", [
    (20000, "csr_rows_kernel", "csr_rows_kernel"), (28671, "csr_rows_kernel", "csr_rows_kernel"),
    (28672, "csr2_rowlane_kernel", "csr2_rowlane_kernel"), (49152, "csr2_rowlane_kernel", "csr2_rowlane_kernel"),
    (49153, "csr_rows_kernel", "csr_rows_kernel"), (65535, "csr_rows_kernel", "csr_rows_kernel"),
    (65536, "csr_rows_kernel", "csr2_wave_kernel"), (65537, "csr2_wave_kernel", "csr2_wave_kernel"),
    (131071, "csr2_wave_kernel", "csr2_wave_kernel"), (131072, "csr2_stream_kernel", "csr2_stream_kernel")])
def test_row_mapping_by_size(stub, N, single, two_pass):
    """The iteration of one CSR state on the arrays, and with a commutator applied to vectors."""
    run(stub, f"""
    ctx = context({N})
    h = ham(ctx, {N})
    for method, name in ((B.CF4, "{single}"), (B.M4, "{two_pass}")):
        names = [n for n in launched(lambda: propagate(ctx, h, method)) if "csr" in n]
        assert names and all(name in n for n in names), names
    """, MAGNUS_CODED="0")


def test_spectral_bounds_wait_once(stub):
    """Both terms' scans and the look whether they fit the coded form, behind one wait of the host."""
    run(stub, """
    ctx = context(5000)
    h = ham(ctx, 5000)
    before = stub.stub_waits()
    names = launched(lambda: L.magnus_spectral_bounds(ctx, C.byref(h), None))
    assert stub.stub_waits() - before == 1
    assert sum("gershgorin" in n for n in names) == 2 and "code_build" in names[-1], names
    """)


@pytest.mark.parametrize("slow", ["coded", "arrays"])
def test_autotune_decides_between_the_coded_form_and_the_arrays(stub, slow):
    """Later calls use what was faster when the tuner timed it: one state, the commutator in two passes, a
    gradient, a batch (pairs against groups), a ragged batch."""
    run(stub, f"""
    N = 70000
    for name in (b"coded_iter", b"coded_pair"):
        stub.stub_cost(name, {50.0 if slow == "coded" else 0.01})
    ctx = context(2 * N, 8)
    h = ham(ctx, N, 10)
    fast = {slow == "arrays"}
    us = np.zeros(7)
    v, g = C.c_int32(), C.c_int32()
    def gradient():
        n = L.magnus_adjoint_workspace_bytes(N, 2, 2)
        f, df, loss, grad = np.full(4, 0.3), np.ones(4), C.c_double(), np.zeros(1)
        return L.magnus_propagate_adjoint(ctx, C.byref(h), 0.1, 2, B._dptr(f), B._dptr(df), 1, vector(N), vector(N), 2,
                                          vector(n // 16 + 1), n, C.byref(loss), B._dptr(grad), opts(), None, None)
    def ragged():
        f = np.full(4, 0.3); keep.append(f)
        P = (B.Problem * 2)(*[B.Problem(h, vector(4 * N), 4, 1, B._dptr(f)) for _ in range(2)])
        return L.magnus_propagate_ragged(ctx, P, 2, B.CF4, 0.1, 2, opts(), None, None)
    calls = dict(one=lambda: propagate(ctx, h), two_pass=lambda: propagate(ctx, h, B.M4), gradient=gradient,
                 batch=lambda: propagate(ctx, h, batch=4), ragged=ragged)
    def coded(names):
        return any("coded_iter" in n or "coded_pair_kernel" in n for n in names)
    assert all(coded(launched(f)) for f in calls.values())      # untuned: terms that fit the form are coded
    B._check(L.magnus_autotune(ctx, C.byref(h), 4, C.byref(v), C.byref(g), B._dptr(us), None, None))
    for name, f in calls.items():
        assert coded(launched(f)) == fast, name
    """)


@pytest.mark.parametrize("N,name", [(65535, "csr_rows_kernel"), (65536, "csr2_iter_kernel"), (131072, "csr2_iter_kernel")])
def test_variant_one_by_size(stub, N, name):
    run(stub, f"""
    ctx = context({N})
    h = ham(ctx, {N})
    names = [n for n in launched(lambda: propagate(ctx, h)) if "csr" in n]
    assert names and all("{name}" in n for n in names), names
    """, MAGNUS_CSR_VARIANT="1")


@pytest.mark.parametrize("N,batch", [(50021, 1), (50022, 1), (1, 1), (77, 3), (4133, 7)])
def test_complex_results_are_aligned(stub, N, batch):
    """The complex sums of dot products (Lanczos enclosures, gradients) lie at multiples of 16 bytes."""
    run(stub, f"""
    stub.stub_watch(b"cdot_final", 2)
    ctx = context({N}, {batch})
    h = ham(ctx, {N})
    names = launched(lambda: L.magnus_spectral_bounds_lanczos(ctx, C.byref(h), 4, 0.01, None))
    assert any("cdot_final" in n for n in names), names
    assert stub.stub_watched(0) == 0
    """)


def test_the_coded_form_takes_memory_when_csr_terms_come(stub):
    """Contexts of dense terms pay nothing for it; 153 bytes per row and a dictionary per block otherwise."""
    run(stub, """
    N = 70000
    ctx = context(N)
    at_create = stub.stub_live()
    assert at_create < 16 * 8 * N + 8 * 11 * N + (36 << 20)
    D = np.zeros(2 * 8 * 8); keep.append(D)
    d = lambda: B.Term(B.DENSE, 0, 8, 0, 8, None, None, D.ctypes.data, -1.0, 1.0)
    hd = B.Hamiltonian(d(), d(), 0.0, 0.0)
    B._check(L.magnus_spectral_bounds(ctx, C.byref(hd), None))
    B._check(propagate(ctx, hd))
    assert stub.stub_live() == at_create
    h = ham(ctx, N)
    rows = -(-N // 64) * 64
    blocks = min(1024, rows // 64)
    assert stub.stub_live() - at_create <= 154 * rows + blocks * (8192 + 4)
    assert any("coded_iter" in n for n in launched(lambda: propagate(ctx, h)))
    B._check(L.magnus_destroy(ctx))
    assert stub.stub_live() == 0
    """)


@pytest.mark.parametrize("room", [0, 3, 6, 9])
def test_without_memory_for_the_coded_form_calls_read_the_arrays(stub, room):
    """A context and calls that fit the memory without it work without it, whichever of its buffers is refused,
    and so do batches of dense terms without the scratch of split products."""
    run(stub, f"""
    N = 70000
    ctx = context(N, 2)
    stub.stub_limit(stub.stub_live() + ({room} << 20))
    h = ham(ctx, N)
    assert stub.stub_failures() > 0
    names = launched(lambda: propagate(ctx, h)) + launched(lambda: propagate(ctx, h, batch=2))
    assert any("csr" in n for n in names) and not any("coded" in n for n in names), names
    B._check(L.magnus_destroy(ctx))
    assert stub.stub_live() == 0
    stub.stub_limit(1 << 40)
    ctx = context(800, 150)
    need = stub.stub_live()
    B._check(L.magnus_destroy(ctx))
    stub.stub_limit(need - (8 << 20))
    ctx = context(800, 150)
    B._check(L.magnus_destroy(ctx))
    """)


@pytest.mark.parametrize("N,two", [(2000, True), (20000, False)])
def test_m6_keeps_its_commutators_only_where_iterations_read_them(stub, N, two):
    """Forty entries a row in K, P1 and P2: short against the other terms below 2^14 rows, not from there on.
    The preparation of another pair, and a second one of the same, run after it."""
    run(stub, f"""
    N = {N}
    stub.stub_fill(b"csr_commutator_kernelILb0", 3, 40, N)   # the rows' lengths
    ctx = context(N)
    h = ham(ctx, N)
    B._check(L.magnus_csr_commutator(ctx, C.byref(h), None))
    k = stub.stub_live()
    for _ in range(2):
        B._check(L.magnus_csr_m6_prepare(ctx, C.byref(h), None))
        kept = stub.stub_live() - k - 7 * 16 * N
        p = 2 * (40 * N * 20 + 4 * (N + 1))
        assert abs(kept - (p if {two} else 0)) < 1024, (kept, p)
        names = launched(lambda: propagate(ctx, h, B.M6))
        assert any("m6_two_kernel" in n for n in names) == {two}
        assert any("m6_kernel" in n for n in names) == (not {two})
    other = ham(ctx, N)
    B._check(L.magnus_csr_m6_prepare(ctx, C.byref(other), None))
    B._check(propagate(ctx, other, B.M6))
    B._check(L.magnus_destroy(ctx))
    assert stub.stub_live() == 0
    """, MAGNUS_CODED="0")


# either side of each line: rows, entries a row of each term, steps of two exponentials, coded
@pytest.mark.parametrize("N,per,steps,coded", [
    (16383, 20, 30, False), (16384, 9, 30, False), (16384, 10, 5, False), (16384, 10, 6, True), (16384, 14, 2, False),
    (16384, 14, 3, True), (28671, 10, 5, False), (28672, 5, 30, False), (28672, 6, 1, False), (28672, 6, 2, True),
    (49152, 6, 1, False), (49152, 6, 2, True), (49153, 1, 1, True), (65536, 1, 1, True)])
def test_when_one_state_is_coded(stub, N, per, steps, coded):
    run(stub, f"""
    ctx = context({N})
    h = ham(ctx, {N}, {per})
    names = launched(lambda: propagate(ctx, h, steps={steps}))
    assert any("coded_iter" in n for n in names) == {coded}, names
    """)


# rows, entries a row of each term, states, steps of two exponentials, as pairs
@pytest.mark.parametrize("N,per,batch,steps,pairs", [
    (3874, 3, 16, 1, True), (3875, 3, 16, 3, False), (3875, 3, 16, 4, True), (8191, 3, 16, 4, True), (8191, 2, 16, 4, False),
    (5000, 2, 12, 3, True), (8192, 3, 16, 4, False), (65536, 3, 16, 3, False), (65537, 3, 16, 3, True), (65537, 2, 16, 3, False),
    (8192, 3, 12, 3, True), (8192, 4, 16, 3, True), (8192, 4, 16, 1, False), (8191, 4, 16, 1, True),
    (21250, 5, 16, 1, False), (21251, 5, 16, 1, True), (21250, 5, 16, 2, True), (21250, 7, 16, 1, True), (80000, 4, 2, 1, True), (4096, 3, 48, 4, False), (70000, 3, 3, 3, True), (70000, 3, 2, 4, False),
    (155000, 3, 2, 3, False), (155001, 3, 2, 3, True), (160000, 2, 20, 3, True), (187500, 2, 16, 3, False),
    (187501, 2, 16, 3, True)])
def test_when_a_batch_runs_as_pairs(stub, N, per, batch, steps, pairs):
    run(stub, f"""
    ctx = context({N}, {batch})
    h = ham(ctx, {N}, {per})
    names = launched(lambda: propagate(ctx, h, steps={steps}, batch={batch}))
    assert any("coded_pair_kernel" in n for n in names) == {pairs}, names
    """, MAGNUS_PERSIST="0")


# five entries a row of both terms together, two and four states
@pytest.mark.parametrize("N,batch,steps,pairs", [
    (30999, 2, 1, True), (32000, 2, 6, False), (180000, 2, 3, False), (180001, 2, 1, True), (20000, 4, 6, False), (10000, 8, 4, True)])
def test_when_a_batch_of_short_rows_runs_as_pairs(stub, N, batch, steps, pairs):
    run(stub, f"""
    ctx = context({N}, {batch})
    h = B.Hamiltonian(term({N}, 2), term({N}, 3), -1.0, 1.0)
    B._check(L.magnus_spectral_bounds(ctx, C.byref(h), None))
    for t in (h.H1, h.H2):
        t.lam_min, t.lam_max = -1.0, 1.0
    names = launched(lambda: propagate(ctx, h, steps={steps}, batch={batch}))
    assert any("coded_pair_kernel" in n for n in names) == {pairs}, names
    """, MAGNUS_PERSIST="0")


def test_the_coded_form_takes_one_allocation(stub):
    run(stub, """
    ctx = context(70001)
    before, held = stub.stub_allocations(), stub.stub_live()
    ham(ctx, 5000)
    ham(ctx, 70001)
    assert stub.stub_allocations() == before + 1
    assert stub.stub_live() - held <= 153 * 70001 + (8 << 20) + 64 * 153 + 6 * 256
    B._check(L.magnus_destroy(ctx))
    assert stub.stub_live() == 0
    """)


# rows, entries a row of each term, states, workgroups of an iteration
@pytest.mark.parametrize("N,per,batch,blocks", [
    (65536, 4, 2, 512), (100003, 4, 2, 392), (131072, 4, 2, 1024), (150001, 4, 2, 592), (131072, 4, 3, 1024), (131072, 4, 4, 1024),
    (16384, 4, 16, 512), (131072, 8, 8, 1024), (131072, 7, 12, 768), (131072, 8, 12, 1536)])
def test_blocks_of_pairs(stub, N, per, batch, blocks):
    run(stub, f"""
    ctx = context({N}, {batch})
    h = ham(ctx, {N}, {per})
    launched(lambda: propagate(ctx, h, steps=3, batch={batch}))
    assert stub.stub_grid(b"coded_pair_kernel") == {blocks}, stub.stub_grid(b"coded_pair_kernel")
    """, MAGNUS_PERSIST="0")


def test_small_states_are_launched_before_a_ragged_call_waits(stub):
    """One problem of pairs, whose norms the call reports, beside one in the one-workgroup kernel: that one is
    on its way when the host waits for the pairs."""
    run(stub, """
    ctx = context(9000, 4)
    small, large = ham(ctx, 300), ham(ctx, 8000)
    f = np.full(4, 0.3)
    P = (B.Problem * 2)(*[B.Problem(h, vector(4 * h.H1.dim), 4, 1, B._dptr(f)) for h in (small, large)])
    before = stub.stub_waits()
    stub.stub_limit(stub.stub_live())  # without pinned memory: a wait of its own before them
    names = launched(lambda: L.magnus_propagate_ragged(ctx, P, 2, B.CF4, 0.1, 2, opts(), None, None))
    assert stub.stub_waits() == before + 1 and "event_wait" not in names
    stub.stub_limit(1 << 40)
    before = stub.stub_waits()
    names = launched(lambda: L.magnus_propagate_ragged(ctx, P, 2, B.CF4, 0.1, 2, opts(), None, None))
    at = lambda what: [k for k, n in enumerate(names) if what in n]
    assert at("coded_pair") and at("persist") and at("event_wait") == [len(names) - 1], names
    assert stub.stub_waits() == before
    B._check(L.magnus_destroy(ctx))
    """, MAGNUS_CODED="2")
