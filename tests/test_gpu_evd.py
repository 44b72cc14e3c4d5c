"""GPU parity of the EVD / ZCA whitening matrix (Sec. 2, Sec. 3.2) against the CPU oracle."""
import ctypes as C

import numpy as np
import pytest
import torch

import workloads as wl
from gpu_common import b, dev, ora, relF, workspace, DEV

pytestmark = pytest.mark.gpu


def run_evd(Phi32, Qs=None, **kw):
    M = Phi32.shape[0]
    T = torch.empty(M, M, device=DEV); Q = torch.empty(M, M, device=DEV); lam = torch.empty(M, device=DEV)
    ws = workspace(b.fw_workspace_bytes(b.FW_OP_WHITEN_EVD, M))
    b.fw_whiten_evd(dev(Phi32), M, b.evd_params(**kw), T, Q, Qs, lam, ws)
    torch.cuda.synchronize()
    return T.cpu().numpy(), Q.cpu().numpy(), lam.cpu().numpy()


@pytest.mark.parametrize("M,lo", [(2, -1), (7, -2), (64, -4), (65, -3), (130, -5), (256, -3), (1100, -4)])
def test_plain_gains(M, lo):
    Phi32 = wl.spd_matrix(M, M, np.logspace(0, lo, M)).astype(np.float32)
    T, Q, lam = run_evd(Phi32, eps=1e-5)
    To, Qo, lo_ = ora.whiten_evd(Phi32, eps=1e-5)
    assert relF(T, To) < 1e-4 and relF(Q, Qo) < 1e-4
    assert np.max(np.abs(lam - lo_)) <= 1e-6 * lo_[0] and np.all(np.diff(lam) <= 0)
    # whitening identity on the part of the spectrum that is not clamped (eq. (whitening))
    P = Phi32.astype(np.float64)
    if lo_[-1] > 1e-5:
        assert np.linalg.norm(T @ P @ T.T - np.eye(M)) / np.sqrt(M) < 1e-3
    assert np.array_equal(T, T.T) and np.array_equal(Q, Q.T)


def test_gain_variant_and_smoothing():
    M = 48
    Phi32 = wl.spd_matrix(8, M, np.logspace(1, -3, M)).astype(np.float32)
    Qs0 = np.eye(M, dtype=np.float32)
    Qs = dev(Qs0)
    T, Q, lam = run_evd(Phi32, Qs=Qs, gain_mode=1, g_max=10.0, beta=0.95)
    To, Qo, lo_ = ora.whiten_evd(Phi32, gain_mode=1, g_max=10.0)
    assert relF(T, To) < 1e-4 and relF(Q, Qo) < 1e-4
    assert relF(Qs.cpu().numpy(), ora.smooth_Q(Qs0, Qo, 0.95)) < 1e-5


def test_clamped_and_degenerate_spectrum():
    M = 40
    lam = np.r_[np.full(10, 2.0), np.full(10, 0.5), np.logspace(-4, -9, 20)]
    Phi32 = wl.spd_matrix(9, M, lam).astype(np.float32)
    T, Q, l = run_evd(Phi32, eps=1e-5)
    To, Qo, lo_ = ora.whiten_evd(Phi32, eps=1e-5)
    assert relF(T, To) < 1e-4 and relF(Q, Qo) < 1e-4


def test_config1_full_whitening():
    L = wl.config1()
    mu, Phi, phi, lbar = ora.block_moments(L.act, 0.0, True)
    Phi32 = Phi.astype(np.float32)
    T, Q, lam = run_evd(Phi32)
    To, Qo, lo_ = ora.whiten_evd(Phi32)
    assert relF(T, To) < 1e-4 and relF(Q, Qo) < 1e-4
    assert np.linalg.norm(T @ Phi32.astype(np.float64) @ T.T - np.eye(64)) / 8 < 1e-3


def reflected_diagonal(M, lam, seed):
    """Symmetric matrix with eigenvalues lam and eigenvectors H_1 H_2 (two reflections): closed forms for T and Q, built on the
    GPU in float64."""
    g = torch.Generator(device=DEV).manual_seed(seed)
    us = [torch.randn(M, generator=g, device=DEV, dtype=torch.float64) for _ in range(2)]
    us = [u / u.norm() for u in us]

    def form(d):
        X = torch.diag(d)
        for u in us:
            X = X - 2 * torch.outer(u, u @ X)
            X = X - 2 * torch.outer(X @ u, u)
        return X
    return form(torch.as_tensor(lam, device=DEV)), form


class EvdRun(C.Structure):
    _fields_ = [(n, C.c_int) for n in ("by_rows", "polls", "one_launch", "diagonal", "sweeps")]


def whiten_evd(Phi, M, T, Q, lam, ws, **how):
    """fw_whiten_evd with a look at the way it took (struct EvdRun of the sources); no Q_s."""
    f = b.lib._ZN2fw10whiten_evdEPKfiPK13fw_evd_paramsPfS5_S5_S5_PvmP12ihipStream_tPNS_6EvdRunE
    P = C.c_void_p
    f.argtypes = [P, C.c_int, C.POINTER(b.fw_evd_params), P, P, P, P, P, C.c_size_t, P, C.POINTER(EvdRun)]
    run = EvdRun(**how)
    rc = f(Phi.data_ptr(), M, C.byref(b.evd_params()), T.data_ptr(), Q.data_ptr(), None, lam.data_ptr(), ws.data_ptr(), ws.numel(),
           torch.cuda.current_stream().cuda_stream, C.byref(run))
    assert rc == 0
    return run


def decompose_known(M, **how):
    """Decomposition of a matrix whose T and Q are known, compared.  The matrix is stored as float32, so T and Q of a spectrum within
    [0.05, 1] carry about 2^-24 / 0.05; from 1536 features on their products run on operands of 16 significant bits (5e-6)."""
    lam = np.linspace(1.0, 0.05, M)
    Phi, form = reflected_diagonal(M, lam, M)
    T = torch.empty(M, M, device=DEV); Q = torch.empty(M, M, device=DEV); out = torch.empty(M, device=DEV)
    ws = workspace(b.fw_workspace_bytes(b.FW_OP_WHITEN_EVD, M))
    run = whiten_evd(Phi.float(), M, T, Q, out, ws, **how)
    d = torch.as_tensor(lam, device=DEV)
    rel = lambda x, y: float((x.double() - y).norm() / y.norm())
    bound = 2e-5 if M >= b.FW_REFRESH_SPLIT_MIN_M else 2e-6
    assert rel(T, form(d.rsqrt())) < bound and rel(Q, form(1 / d)) < bound
    assert float((out.double() - d).abs().max()) < 5e-7
    assert torch.equal(T, T.T) and torch.equal(Q, Q.T)
    return run


# Rows reduced one launch each before the launch for all others, which then starts from their last reflector: the direct decomposition is
# accepted every time (the start raced once: one call in twenty to a hundred was off and went through the sweeps, a tenth as fast).
@pytest.mark.parametrize("M", [2561, 2600, 3073])
def test_reduction_after_rows_of_their_own(M):
    for _ in range(12):
        run = decompose_known(M)
        assert run.one_launch and run.sweeps == 0


# One leaf, two leaves, the last 128 rows alone and with one row more, sizes where T and Q change form, and sizes whose first rows are
# reduced one launch each (beyond 2560: columns per thread change at 3072, 4096, 5120, 8192 rows).  The direct decomposition
# has to be the one that is accepted.
@pytest.mark.parametrize("M", [1, 16, 17, 127, 128, 129, 257, 513, 769, 1025, 1535, 1537, 2049, 2561, 3073, 4097, 5121, 8193])
def test_direct_decomposition_sizes(M):
    run = decompose_known(M)
    assert run.sweeps == 0 and run.one_launch == (M > 128) and run.diagonal == (M == 1)


# The reduction in one launch: workgroups of 8 rows (10 beyond 2048), the last one whole, with one row and with one row missing,
# the largest and smallest of its range.
@pytest.mark.parametrize("M", [135, 136, 137, 256, 512, 640, 641, 768, 1024, 1536, 2047, 2048, 2050, 2051, 2559, 2560])
def test_reduction_in_one_launch_sizes(M):
    run = decompose_known(M)
    assert run.sweeps == 0 and run.one_launch


# What runs where that launch is not possible: a launch per row, one size per range of its rule (columns per thread change at 256, 512,
# 768, 1024, 1536, 2048, 2560, 3072 rows).
@pytest.mark.parametrize("M", [129, 257, 513, 769, 1025, 1537, 2049, 2560, 2561, 3073])
def test_reduction_row_by_row_sizes(M):
    run = decompose_known(M, by_rows=1)
    assert run.sweeps == 0 and not run.one_launch


@pytest.mark.parametrize("M", [300, 1100, 2304])
def test_reduction_given_up(M):
    """Waits that end after one round: the decomposition is not accepted, and the sweeps give the result."""
    run = decompose_known(M, polls=1)
    assert run.one_launch and run.sweeps > 0


@pytest.mark.parametrize("sizes", [(300, 900), (2304, 2300), (2304, 600)])
def test_decompositions_on_two_streams(sizes):
    """Two threads with a stream each, whose workgroups the chip holds at a time or does not: every one gets what it gets alone, bit
    for bit, without sweeps."""
    import threading
    alone, got, errors = {}, {}, []

    def call(M, where, stream):
        try:
            with torch.cuda.stream(stream):
                T = torch.empty(M, M, device=DEV); Q = torch.empty(M, M, device=DEV); out = torch.empty(M, device=DEV)
                ws = workspace(b.fw_workspace_bytes(b.FW_OP_WHITEN_EVD, M))
                for _ in range(5):
                    run = whiten_evd(Phi[M], M, T, Q, out, ws)
                    assert run.one_launch and run.sweeps == 0
                stream.synchronize()
                where[M] = (T, Q, out)
        except BaseException as ex:  # noqa: BLE001
            errors.append(ex)

    Phi = {M: dev(wl.spd_matrix(M, M, np.logspace(0, -3, M)).astype(np.float32)) for M in sizes}
    torch.cuda.synchronize()
    for M in sizes:
        call(M, alone, torch.cuda.Stream())
    threads = [threading.Thread(target=call, args=(M, got, torch.cuda.Stream())) for M in sizes]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors
    for M in sizes:
        assert all(torch.equal(x, y) for x, y in zip(alone[M], got[M]))


@pytest.mark.parametrize("kind", ["dead", "duplicate", "identity", "zero", "graded", "tol"])
@pytest.mark.parametrize("M", [33, 200])
def test_special_matrices(kind, M):
    """Zero rows, rank deficiency, full deflation, a diagonal graded over 16 decades far above the clamp (ends in the Jacobi
    sweeps) and sweeps to a threshold of the caller's; T and Q against the oracle."""
    rng = np.random.default_rng(M)
    Phi = wl.spd_matrix(M, M, np.logspace(0, -3, M))
    kw = {}
    if kind == "dead":
        Phi[:, ::3] = 0; Phi[::3, :] = 0
    elif kind == "duplicate":
        Phi[:, 5] = Phi[:, 7]; Phi[5, :] = Phi[7, :]; Phi[5, 5] = Phi[7, 7]
    elif kind == "identity":
        Phi = np.eye(M)
    elif kind == "zero":
        Phi = np.zeros((M, M))
    elif kind == "graded":
        s = 10.0 ** np.linspace(8, 0, M)
        Phi = wl.spd_matrix(M, M, np.linspace(1, 0.3, M)) * s[:, None] * s[None, :]
    elif kind == "tol":
        kw = {"tol": 1e-12}
    Phi32 = Phi.astype(np.float32)
    T, Q, lam = run_evd(Phi32, eps=1e-5, **kw)
    if kind == "graded":
        # LAPACK has no relative accuracy here; D^-1/2 Phi D^-1/2 is well conditioned, so the whitening identity holds
        P = Phi32.astype(np.float64)
        assert np.all(lam > 0) and np.linalg.norm(T @ P @ T.T - np.eye(M)) / np.sqrt(M) < 0.05
        return
    To, Qo, lo_ = ora.whiten_evd(Phi32, eps=1e-5)
    assert relF(T, To) < 1e-5 and relF(Q, Qo) < 1e-5
    assert np.max(np.abs(lam - lo_)) <= 2e-7 * max(lo_[0], 1e-30)


@pytest.mark.parametrize("M", [600, 1100, 2300])
@pytest.mark.parametrize("kind", ["rows", "duplicates", "clusters"])
def test_deficient_and_clustered_spectra(kind, M):
    """Fewer rows than features, every feature there twice, three eigenvalues of high multiplicity, over more than four levels of
    merges: T, Q and the eigenvalues against the oracle, and the space that Phi_x takes to zero (gain 1/eps on all of it).
    Rounding Phi_x to float32 moves eigenvalues by up to 2^-24 |Phi_x|, the gain 1/sqrt(max(lambda, eps)) of one near eps by
    2^-25 |Phi_x| / eps of itself: eps is chosen so that this is 3e-6; 16-bit operands from 1536 features on add 5e-6."""
    rng = np.random.default_rng(M)
    if kind == "clusters":
        Phi, _ = reflected_diagonal(M, np.repeat([1.0, 0.25, 0.05], [M // 2, M // 3, M - M // 2 - M // 3]), M)
        Phi32, eps = Phi.float().cpu().numpy(), 1e-2
    else:
        X = rng.standard_normal((M // 4, M))
        if kind == "duplicates":
            X = rng.standard_normal((M, M // 2)).repeat(2, axis=1)
        Phi32, eps = (X.T @ X / len(X)).astype(np.float32), 0.2
    T, Q, lam = run_evd(Phi32, eps=eps)
    To, Qo, lo_ = ora.whiten_evd(Phi32, eps=eps)
    bound = 2e-5 if M >= b.FW_REFRESH_SPLIT_MIN_M else 1e-5
    assert relF(T, To) < bound and relF(Q, Qo) < bound
    assert np.max(np.abs(lam - lo_)) <= 2e-7 * lo_[0]
    if kind == "duplicates":       # (e_2k - e_2k+1) / sqrt 2 spans that space
        N = T[:, 0::2].astype(np.float64) - T[:, 1::2]
        want = np.zeros_like(N)
        want[0::2], want[1::2] = np.eye(M // 2), -np.eye(M // 2)
        assert relF(N, want / np.sqrt(eps)) < bound


@pytest.mark.parametrize("M", [40, 700, 1024, 1025, 1601])
def test_acceptance_sees_lost_orthogonality(M):
    """The check behind the direct decomposition, called by itself: exact eigenvectors pass; a null vector that is a copy of
    another, a zero one or a longer one fails by V V^T, entry by entry or (from 1025 rows on) against vectors (V Phi V^T does not see
    it), wherever it stands, and so does a row that leans on another by 1e-9; two rows turned towards each other fail
    by V Phi V^T alone."""
    lib = b.lib
    check = lib._ZN2fw13sym_eig_checkEPKfiPKdPdS4_S4_PvdddS4_PiP12ihipStream_t
    P = C.c_void_p
    check.argtypes = [P, C.c_int, P, P, P, P, P, C.c_double, C.c_double, C.c_double, P, P, P]
    ld, small, n = lib._ZN2fw10sym_eig_ldEi(M), lib._ZN2fw19sym_eig_small_bytesEi(M), lib._ZN2fw22sym_eig_matrix_doublesEi(M)
    r = M // 4
    Phi = torch.zeros(M, M, device=DEV)
    Phi[:r, :r] = torch.diag(torch.linspace(1, 0.5, r, device=DEV))
    q, _ = torch.linalg.qr(torch.as_tensor(np.random.default_rng(M).standard_normal((M - r, M - r))))
    good = torch.eye(M, dtype=torch.float64)
    good[r:, r:] = q               # any basis of the null space

    def verdict(V):
        Vd = torch.zeros(n, dtype=torch.float64, device=DEV)
        Vd[:M * ld].view(M, ld)[:, :M] = V.to(DEV)
        W, copy, scratch, lam = torch.zeros_like(Vd), torch.zeros_like(Vd), torch.zeros_like(Vd), torch.zeros(M, dtype=torch.float64, device=DEV)
        flag = torch.zeros(64, dtype=torch.int32, device=DEV)
        ws = workspace(small)
        rc = check(Phi.data_ptr(), M, Vd.data_ptr(), W.data_ptr(), copy.data_ptr(), scratch.data_ptr(), ws.data_ptr(), 2.0 ** -34, 2.0 ** -30 * 1e-5, 0.0,
                   lam.data_ptr(), flag.data_ptr(), torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        assert rc == 0
        return [int(f != 0) for f in flag[:2].tolist()]

    assert verdict(good) == [0, 0]
    for at in (r, (r + M) // 2, M - 1):
        other = good[r + 1]
        for row in (other, 0 * good[at], 1.001 * good[at], good[at] + 1e-9 * other):
            V = good.clone()
            V[at] = row
            assert verdict(V) == [0, 1]
    V = good.clone()
    c, s = np.cos(1e-6), np.sin(1e-6)
    V[0], V[r - 1] = c * good[0] + s * good[r - 1], c * good[r - 1] - s * good[0]
    assert verdict(V) == [1, 0]


@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
@pytest.mark.parametrize("M", [48, 200])
def test_one_feature_not_finite(M, bad):
    """A feature whose variance is not finite and that is correlated with no other: the direct decomposition leaves nothing, the sweeps
    that start over from the identity never rotate that feature, so V stays orthogonal and T and Q finite."""
    Phi32 = wl.spd_matrix(M, M, np.logspace(0, -3, M)).astype(np.float32)
    Phi32[7, :] = 0
    Phi32[:, 7] = 0
    Phi32[7, 7] = bad
    T, Q, _ = run_evd(Phi32)
    assert np.isfinite(T).all() and np.isfinite(Q).all()


@pytest.mark.parametrize("M", [1, 2, 63, 300, 1600])
@pytest.mark.parametrize("kw", [{}, {"gain_mode": 1}, {"tol": 1e-12}])
def test_diagonal_and_nearly_diagonal(M, kw):
    """Matrices that need no decomposition (diagonal; off-diagonal entries a tenth of what the acceptance allows), and one whose single
    off-diagonal entry, in either triangle, is just too large for that: T, Q, eigenvalues and Q_s against the oracle."""
    rng = np.random.default_rng(M)
    d = rng.permutation(np.logspace(1, -4, M))
    d[: M // 8] = 0
    kind = [np.diag(d)]
    noise = rng.uniform(-1, 1, (M, M)) * 0.1 * 2.0 ** -34 * np.sqrt(np.outer(d, d))
    kind.append(np.diag(d) + np.tril(noise, -1) + np.tril(noise, -1).T)
    if M > 10:
        i, j = int(np.argsort(d)[-1]), int(np.argsort(d)[-2])
        for at in ((i, j), (j, i)):
            P = np.diag(d)
            P[at] = 0.01 * np.sqrt(d[i] * d[j])
            kind.append(P)
    bound = 2e-5 if M >= b.FW_REFRESH_SPLIT_MIN_M else 1e-5
    for Phi in kind:
        Phi32 = Phi.astype(np.float32)
        Qs = dev(np.eye(M, dtype=np.float32))
        T, Q, lam = run_evd(Phi32, Qs=Qs, eps=1e-3, beta=0.5, **kw)
        To, Qo, lo_ = ora.whiten_evd(Phi32, eps=1e-3, gain_mode=kw.get("gain_mode", 0))
        assert relF(T, To) < bound and relF(Q, Qo) < bound
        assert np.max(np.abs(lam - lo_)) <= 2e-7 * max(lo_[0], 1e-30)
        assert relF(Qs.cpu().numpy(), ora.smooth_Q(np.eye(M), Qo, 0.5)) < bound
