"""The paper's root parameterisation on the GPU (QGBE_SAMPLER_ROOTS, and the
alternative elimination QGBE_SAMPLER_ROOTS_ALT) against the oracle's root
estimators, and the stability test of Sec. IV A at the paper's size."""
import numpy as np
import pytest

from paper_1912_04457_amd import qgbe
from paper_1912_04457_amd import workloads as W

pytestmark = pytest.mark.gpu

SEED = W.PHILOX_SEED
EST = {qgbe.SAMPLER_ROOTS: "root", qgbe.SAMPLER_ROOTS_ALT: "root_k3"}


def _case(name):
    print(f"\n[gpu case] {name}", flush=True)


def _grid(O, n_x, n_p, mask, p_half=(2.0, 2.0, 2.0)):
    return O.Grid(n_x=n_x, n_p=n_p, x_half=(3.0, 3.0, 3.0), p_half=p_half, species_mask=mask)


def _solver(g, precision, symmetric=True):
    return qgbe.Solver(n_x=g.n_x, n_p=g.n_p, x_half=g.x_half, p_half=g.p_half, species_mask=g.species_mask,
                       alpha_s=g.alpha_s, seed=SEED, precision=precision, symmetric=symmetric)


@pytest.mark.parametrize("sampler", [qgbe.SAMPLER_ROOTS, qgbe.SAMPLER_ROOTS_ALT])
@pytest.mark.parametrize("precision", [qgbe.FP64, qgbe.FP32])
def test_roots_parity_seven_species_ragged(O, sampler, precision):
    """Every channel of the 7 species on 2 cells and a ragged 5x6x4 grid:
    A, the gain+loss scale and the item sums element by element (the root
    samplers run in FP64 in either context precision)."""
    _case(f"roots parity sampler={sampler} precision={precision}")
    g = _grid(O, (2, 1, 1), (5, 6, 4), 0x7F, p_half=(2.0, 2.5, 1.5))
    f = W.random_f(31, g.cells, g.nodes) * 0.6
    with _solver(g, precision) as s:
        s.set_f(f)
        A, S, I, st = s.collision(50, sampler=sampler, scale=True, items=True)
        m = s.masses()      # the masses that collision term used
    A_ref, S_ref, I_ref = O.collision(g, f, m, SEED, 0, 50, estimator=EST[sampler], want_items=True)
    assert np.all(np.abs(S - S_ref) <= 1e-10 * S_ref + 1e-300)
    assert np.all(np.abs(A - A_ref) <= 1e-10 * S_ref + 1e-300)
    assert np.abs(I - I_ref).max() <= 1e-10 * np.abs(I_ref).max()
    assert S_ref.max() > 0 and st.n_accepted > 0
    for cell in range(g.cells):      # symmetric sampling conserves number per cell
        assert abs(A[:, cell].sum()) <= 1e-13 * S[:, cell].sum()


@pytest.mark.parametrize("sampler", [qgbe.SAMPLER_ROOTS, qgbe.SAMPLER_ROOTS_ALT])
def test_roots_direct_estimator(O, sampler):
    _case(f"roots direct sampler={sampler}")
    g = _grid(O, (1, 1, 1), (8, 8, 8), 1 << O.GLUON)
    f = W.random_f(32, g.cells, g.nodes, species_mask=1 << O.GLUON)
    with _solver(g, qgbe.FP64, symmetric=False) as s:
        s.set_f(f)
        A, S, _, _ = s.collision(64, sampler=sampler, scale=True)
        m = s.masses()
    A_ref, S_ref, _ = O.collision(g, f, m, SEED, 0, 64, estimator=EST[sampler], symmetric=False)
    assert np.all(np.abs(A - A_ref) <= 1e-10 * S_ref + 1e-300)
    assert abs(A.sum()) > 1e-6 * S.sum()     # the direct estimator does not conserve


def test_roots_at_the_stability_test_size(O):
    """40^3 nodes, f uniform in [0, 1], 100 samples per node (Sec. IV A): a
    seeded sample of 96 work items recomputed by the oracle for both
    eliminations, in the launch configuration of the stability test."""
    _case("roots 40^3 sampled items")
    g = _grid(O, (1, 1, 1), (40, 40, 40), 1 << O.GLUON)
    rng = np.random.Generator(np.random.PCG64(7))
    f = np.zeros((7, 1, g.nodes))
    f[O.GLUON, 0] = rng.uniform(0.0, 1.0, g.nodes)
    items = np.stack([np.zeros(96, int), np.zeros(96, int), rng.integers(0, g.nodes, 96)], 1)
    with _solver(g, qgbe.FP64, symmetric=False) as s:
        s.set_f(f)
        got = {}
        for sampler in EST:
            _, _, I, _ = s.collision(100, sampler=sampler, items=True)
            got[sampler] = I[items[:, 0], items[:, 1], items[:, 2]]
        m = s.masses()
    for sampler, est in EST.items():
        ref, scale = O.item_sums(g, f, m, SEED, 0, 100, items, symmetric=False, want_scale=True, estimator=est)
        assert np.all(np.abs(got[sampler] - ref) <= 1e-10 * scale + 1e-300), sampler
        assert np.count_nonzero(scale) > 80


def test_stability_spread_of_the_two_eliminations():
    """The experiment of Sec. IV A: the gluon number after one step of the
    direct estimator over 24 independent evaluations (seeds) from the same
    random f.  The alternative elimination spreads more than the paper's
    choice, and the CM-angle sampler less than both."""
    _case("stability experiment 40^3")
    n = 40
    P = W.node_momenta((n, n, n), (2.0, 2.0, 2.0))
    rng = np.random.Generator(np.random.PCG64(7))
    f = np.zeros((7, 1, len(P)))
    f[6, 0] = rng.uniform(0.0, 1.0, len(P))
    spread, mean = {}, {}
    with qgbe.Solver(n_x=(1, 1, 1), n_p=(n, n, n), x_half=(3.0, 3.0, 3.0), p_half=(2.0, 2.0, 2.0),
                     species_mask=1 << 6, alpha_s=0.3, seed=SEED, precision=qgbe.FP64, symmetric=False) as s:
        for sampler in (qgbe.SAMPLER_UNIFORM, qgbe.SAMPLER_ROOTS, qgbe.SAMPLER_ROOTS_ALT):
            N = []
            for r in range(24):
                s.set_f(f)                              # the same initial f (and E = |p| masses)
                qgbe.qgbe_set_step_index(s.ctx, 1000 + r)  # an independent Philox key
                N.append(s.step(0.01, 100, n_steps=1, sampler=sampler)[0]["N_total"])
            spread[sampler] = float(np.std(N, ddof=1))
            mean[sampler] = float(np.mean(N))
    print(f"[stability] N spread cm {spread[0]:.4g} roots {spread[2]:.4g} roots_alt {spread[3]:.4g}", flush=True)
    assert spread[qgbe.SAMPLER_ROOTS_ALT] > 1.2 * spread[qgbe.SAMPLER_ROOTS]
    assert spread[qgbe.SAMPLER_UNIFORM] < spread[qgbe.SAMPLER_ROOTS]
    # the three estimate the same step
    for k in (qgbe.SAMPLER_ROOTS, qgbe.SAMPLER_ROOTS_ALT):
        assert abs(mean[k] - mean[0]) < 5.0 * (spread[k] + spread[0]) / np.sqrt(24)


@pytest.mark.parametrize("sampler", [qgbe.SAMPLER_ROOTS, qgbe.SAMPLER_ROOTS_ALT])
@pytest.mark.parametrize("n_x,n_p,mask,N,precision", [((1, 1, 1), (24, 25, 24), 1 << 6, 70, qgbe.FP64),
                                                      ((2, 1, 1), (16, 17, 18), 0x49, 20, qgbe.FP32),
                                                      ((1, 1, 1), (9, 8, 7), 1 << 6, 600, qgbe.FP64)],
                         ids=["windows", "slots_f32_context", "shared_nodes"])
def test_roots_lds_plans(O, sampler, n_x, n_p, mask, N, precision):
    """Symmetric deposits in LDS accumulators: grids that take several launches
    (deposits recorded and replayed; with the scale output, the samples drawn
    again in every launch) and waves that share a node."""
    _case(f"roots plans sampler={sampler} {n_x} {n_p} mask={mask:#x} N={N}")
    g = _grid(O, n_x, n_p, mask)
    f = W.random_f(33, g.cells, g.nodes, species_mask=mask) * 0.6
    with _solver(g, precision) as s:
        s.set_f(f)
        A, _, I, st = s.collision(N, sampler=sampler, items=True)
        A2, _, I2, st2 = s.collision(N, sampler=sampler, scale=True, items=True)
        m = s.masses()
    A_ref, S_ref, I_ref = O.collision(g, f, m, SEED, 0, N, estimator=EST[sampler], want_items=True)
    for a in (A, A2):
        assert np.all(np.abs(a - A_ref) <= 1e-10 * S_ref + 1e-300)
    # the same samples by two routes: sums in another order
    assert np.abs(I - I2).max() <= 1e-12 * np.abs(I_ref).max()
    assert st.n_accepted == st2.n_accepted > 0
    for cell in range(g.cells):
        assert abs(A[:, cell].sum()) <= 1e-13 * S_ref[:, cell].sum()


def test_first_roots_call_beside_a_capture():
    """The first root-sampler call of a context allocates its record buffers; a
    capture that another stream is in meanwhile goes on, and a call without the
    buffers, captured first, gives the same term."""
    torch = pytest.importorskip("torch")
    _case("first roots call beside a capture")
    grid = dict(n_x=(1, 1, 1), n_p=(24, 25, 24), x_half=(3.0, 3.0, 3.0), p_half=(2.0, 2.5, 1.5), species_mask=1 << 6)
    f = torch.from_numpy(W.random_f(35, 1, 24 * 25 * 24, species_mask=1 << 6) * 0.6).cuda()
    x = torch.arange(8.0, device="cuda")
    A, B, C = (torch.full_like(f, float("nan")) for _ in range(3))
    own, other = torch.cuda.Stream(), torch.cuda.Stream()
    with qgbe.Solver(**grid, precision=qgbe.FP32, seed=SEED, stream=own.cuda_stream) as s:
        qgbe.qgbe_set_distribution(s.ctx, -1, f)
        torch.cuda.synchronize()
        before = qgbe.qgbe_workspace_bytes(s.ctx)
        captured = torch.cuda.CUDAGraph()
        with torch.cuda.graph(captured, stream=own):
            qgbe.qgbe_collision_term(s.ctx, 70, qgbe.SAMPLER_ROOTS, A)
        assert qgbe.qgbe_workspace_bytes(s.ctx) == before
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=other):
            y = x + 1.0
            qgbe.qgbe_collision_term(s.ctx, 70, qgbe.SAMPLER_ROOTS, B)
        assert qgbe.qgbe_workspace_bytes(s.ctx) > before
        for _ in range(2):
            captured.replay()
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(y, x + 1.0)
            qgbe.qgbe_collision_term(s.ctx, 70, qgbe.SAMPLER_ROOTS, C)
            torch.cuda.synchronize()
        _, S, _, _ = s.collision(70, sampler=qgbe.SAMPLER_ROOTS, scale=True)
    S = torch.from_numpy(S).cuda()
    for out in (A, B, C):
        assert bool(((out - A).abs() <= 1e-10 * S + 1e-300).all()) and float(A.abs().max()) > 0.0
