"""SCF driver with the full-diagonalisation fallback on the GPU: the full
diagonalisation (a plan whose single submatrix is the whole matrix) against the
oracle's step with that layout and against LAPACK; a PFSM sequence that starts
with full steps; and a fall back when the previous eigenvectors no longer fit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

from oracle.pfsm_ref import eig_error, orthogonality, pfsm_ref, residual_norm  # noqa: E402
from pfsm_workloads import prescribed_problem, scf_sequence, uniform_layout  # noqa: E402


@pytest.fixture(scope="module")
def pf():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a visible MI355X")
    import paper_1502_07806_amd as pf
    pf.load_library()
    return pf


def _random_symmetric(n, seed):
    g = np.random.default_rng(seed)
    G = g.standard_normal((n, n))
    return 0.5 * (G + G.T)


def _random_orthogonal(n, seed):
    g = np.random.default_rng(seed)
    Q, R = np.linalg.qr(g.standard_normal((n, n)))
    return Q * np.sign(np.diag(R))[None, :]


@pytest.mark.parametrize("n,basis", [(300, "identity"), (640, "identity"), (640, "orthogonal")])
def test_full_diag_parity(pf, n, basis):
    dev = torch.device("cuda:0")
    A = _random_symmetric(n, n)
    V = np.eye(n) if basis == "identity" else _random_orthogonal(n, n + 1)
    fd = pf.FullDiag(n)
    lam, Vo = fd.solve(torch.from_numpy(A).to(dev), torch.from_numpy(V).to(dev))
    lam, Vo = lam.cpu().numpy(), Vo.cpu().numpy()
    lam_ref, V_ref, info = pfsm_ref(A, V, [0, n], halo=0, iterations=0)
    assert info == 0
    assert eig_error(lam, lam_ref) <= 1e-13
    assert eig_error(lam, np.linalg.eigvalsh(A)) <= 1e-13
    # the block Jacobi leaves off-diagonal entries below its noise floor of
    # 256 u ||B||, so residual and orthogonality scale like 256 u n
    floor = 256 * 2.0 ** -53 * n
    assert residual_norm(A, lam, Vo) <= floor
    assert orthogonality(Vo) <= floor
    # non-degenerate random spectrum: each eigenvector agrees with the oracle's (same signs)
    gaps = np.diff(lam_ref)
    tol = 1e-13 * np.abs(lam_ref).max() / np.minimum(np.r_[gaps, np.inf], np.r_[np.inf, gaps])
    assert np.all(np.abs(Vo - V_ref).max(axis=0) <= 100 * tol + 1e-12)


@pytest.mark.parametrize("n", [1, 2, 31, 33, 64, 65, 127, 129, 200])
def test_full_diag_equal_diagonal(pf, n):
    """Pair problems at the edges of their blocks (padding columns, partly
    filled last blocks) on the second-difference matrix: its equal diagonal
    entries give every first-round pair equal column norms (the tie rule of
    the rotation's sign), and its eigenvalues are 2 - 2 cos(k pi / (n + 1)).
    A few hundred rotations of norm-4 rows leave about n u 4 = 1e-13 in an
    eigenvalue and n u in an inner product; 1e-12 covers both at n = 200."""
    dev = torch.device("cuda:0")
    A = 2.0 * np.eye(n) - np.eye(n, k=1) - np.eye(n, k=-1)
    lam, V = pf.FullDiag(n).solve(torch.from_numpy(A).to(dev))
    lam, V = lam.cpu().numpy(), V.cpu().numpy()
    want = 2.0 - 2.0 * np.cos(np.arange(1, n + 1) * np.pi / (n + 1))
    assert np.max(np.abs(lam - want)) <= 1e-12
    assert np.max(np.abs(V.T @ V - np.eye(n))) <= 1e-12
    assert np.max(np.abs(A @ V - V * lam)) <= 1e-12


@pytest.mark.parametrize("n", [256, 500])
def test_late_sweeps_clustered(pf, n):
    """Eight levels of equal eigenvalues keep a single submatrix rotating past
    the sixteen sweeps with their own launches, so that the launch behind them
    spreads several sweeps over its workgroups.  Norm 7: an eigenvalue is off by
    at most about n u 7 (4e-13), entries of the residual and of V^T V - I by
    less; bound 1e-12 as above, times 7 where the norm enters."""
    dev = torch.device("cuda:0")
    g = np.random.default_rng(n)
    Q, _ = np.linalg.qr(g.standard_normal((n, n)))
    levels = np.sort(np.arange(n) % 8).astype(float)
    A = (Q * levels) @ Q.T
    A = (A + A.T) / 2
    full = pf.FullDiag(n)
    lam, V = full.solve(torch.from_numpy(A).to(dev))
    assert full.plan.debug_stats()["converged_sweep"][0] > 16
    lam, V = lam.cpu().numpy(), V.cpu().numpy()
    assert np.max(np.abs(lam - levels)) <= 7e-12
    assert np.max(np.abs(V.T @ V - np.eye(n))) <= 1e-12
    assert np.max(np.abs(A @ V - V * lam)) <= 7e-12


@pytest.mark.parametrize("max_sweeps", [12, 13, 40])
@pytest.mark.parametrize("n", [33, 64, 97, 300])
def test_full_diag_sweep_limits(pf, n, max_sweeps):
    """A limit of 12 solves every pair problem to the end, 13 the first sweep's
    and 40 nearly all in one sweep over the pairs between the blocks: the same
    eigenpairs, with the bounds of the equal-diagonal test (norm 2 here)."""
    dev = torch.device("cuda:0")
    A = _random_symmetric(n, n) / np.sqrt(n)
    lam, V = pf.FullDiag(n, max_sweeps).solve(torch.from_numpy(A).to(dev))
    lam, V = lam.cpu().numpy(), V.cpu().numpy()
    assert np.max(np.abs(lam - np.linalg.eigvalsh(A))) <= 1e-12
    assert np.max(np.abs(V.T @ V - np.eye(n))) <= 1e-12
    assert np.max(np.abs(A @ V - V * lam)) <= 1e-12


@pytest.mark.parametrize("n", [97, 300])
def test_sweep_limit_is_only_a_limit(pf, n):
    """Up to 39 the limit on the sweeps changes nothing but where they end: a
    matrix that needs fewer than twelve has the same bits under every limit, so
    that one whose count is close to its limit gets there too."""
    dev = torch.device("cuda:0")
    A = torch.from_numpy(_random_symmetric(n, 5 * n) / np.sqrt(n)).to(dev)
    runs = []
    for limit in (12, 13, 20, 39):
        full = pf.FullDiag(n, limit)
        runs.append([t.clone() for t in full.solve(A)])
        assert full.plan.debug_stats()["converged_sweep"][0] < 12
    for lam, V in runs[1:]:
        assert torch.equal(lam, runs[0][0]) and torch.equal(V, runs[0][1])


@pytest.mark.parametrize("n", [200, 512])
def test_full_diag_repeats_bitwise(pf, n):
    """No wave's rotation depends on how far another has come: repeated full
    diagonalisations, whose middle sweeps hand their columns over to Newton's
    iteration, give the same bits every time."""
    dev = torch.device("cuda:0")
    A = torch.from_numpy(_random_symmetric(n, 3 * n) / np.sqrt(n)).to(dev)
    full = pf.FullDiag(n)
    runs = [[t.clone() for t in full.solve(A)] for _ in range(4)]
    for lam, V in runs[1:]:
        assert torch.equal(lam, runs[0][0]) and torch.equal(V, runs[0][1])


@pytest.mark.parametrize("n,precision,tol", [(130, "fp64", 1e-12), (200, "fp64", 1e-12), (200, "mixed_bf16", 1e-8)])
def test_late_sweeps(pf, n, precision, tol):
    """Submatrices that need more sweeps than are enqueued round by round (two
    windows, each the whole of a dense random matrix in the identity basis):
    the single launch that finishes them gives the eigenpairs of the matrix.
    FP64 tolerance as above (norm about 2 sqrt(n)); mixed: its bar."""
    dev = torch.device("cuda:0")
    A = _random_symmetric(n, 7 * n) / np.sqrt(n)
    plan = pf.Plan(n, [0, n // 2, n], halo=n, iterations=0, precision=precision)
    lam, V = plan.solve(torch.from_numpy(A).to(dev), torch.eye(n, dtype=torch.float64, device=dev))
    spread = 4 if precision == "fp64" else 3
    assert min(plan.debug_stats()["converged_sweep"]) > spread  # past the sweeps with their own launches
    lam, V = lam.cpu().numpy(), V.cpu().numpy()
    assert np.max(np.abs(lam - np.linalg.eigvalsh(A))) <= tol
    if precision == "fp64":
        assert np.max(np.abs(V.T @ V - np.eye(n))) <= tol
        assert np.max(np.abs(A @ V - V * lam)) <= tol
    # the limit just below the last active sweep is reported
    conv = max(plan.debug_stats()["converged_sweep"])
    short = pf.Plan(n, [0, n // 2, n], halo=n, iterations=0, precision=precision, max_sweeps=conv - 1)
    short.solve(torch.from_numpy(A).to(dev), torch.eye(n, dtype=torch.float64, device=dev), check=False)
    assert int(short.info.item()) == -3


def test_scf_sequence_switches_to_pfsm(pf):
    dev = torch.device("cuda:0")
    n = 1024
    A0 = prescribed_problem(n, n // 2, 1e-2, 2500, clusters=True, device=dev)[0]
    seq = [A0] + scf_sequence(A0, 4, 2500)
    offs = uniform_layout(n, 128)
    drv = pf.SCFDriver(n, offs, halo=64, iterations=3, full_steps=2)
    V_prev = None
    for k, A in enumerate(seq):
        Ac = A.t().contiguous().t()
        lam, V = drv.step(Ac)
        An = A.cpu().numpy()
        lam_n = lam.cpu().numpy()
        # full steps are exact to rounding; PFSM steps carry the method's own
        # truncation (three folded-spectrum iterations), checked for parity below
        assert eig_error(lam_n, np.linalg.eigvalsh(An)) <= (1e-13 if k < 2 else 1e-7)
        if k >= 2:  # PFSM step: parity with the oracle from the same previous eigenvectors
            lam_ref, _, info = pfsm_ref(An, V_prev, offs, 64, 3, 2)
            assert info == 0 and eig_error(lam_n, lam_ref) <= 1e-10
        V_prev = V.cpu().numpy()
    assert [h.method for h in drv.history] == ["full", "full", "pfsm", "pfsm", "pfsm"]
    res = [h.residual for h in drv.history]
    assert all(r <= 256 * 2.0 ** -53 * n for r in res[:2]), res
    assert all(r <= drv.residual_tol for r in res[2:]), res


def test_scf_falls_back_when_basis_no_longer_fits(pf):
    dev = torch.device("cuda:0")
    n = 512
    A0 = prescribed_problem(n, n // 2, 1e-2, 2600, device=dev)[0]
    R = _random_symmetric(n, 2601)
    drv = pf.SCFDriver(n, uniform_layout(n, 128), halo=64, full_steps=1)
    drv.step(A0.t().contiguous().t())
    lam, V = drv.step(torch.from_numpy(R).to(dev))
    assert [(h.method, h.reason) for h in drv.history] == [("full", "start"), ("full", "dominance")]
    assert drv.history[1].dominance > 1e-2
    assert eig_error(lam.cpu().numpy(), np.linalg.eigvalsh(R)) <= 1e-13
    assert residual_norm(R, lam.cpu().numpy(), V.cpu().numpy()) <= 256 * 2.0 ** -53 * n
