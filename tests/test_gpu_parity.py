"""GPU parity: the HIP path through the C ABI against the FP64 oracle.

Same seed, same step index, same f => the same Philox samples on both sides, so
the collision terms agree element by element:
  FP64 mode  |A_gpu - A_ref| <= 1e-10 * S(x,q)   and   ||dA||_2 <= 1e-10 ||A||_2
  FP32 mode  |A_gpu - A_ref| <= 1e-4  * S(x,q)   and   ||dA||_2 <= 1e-4  ||A||_2
S is the oracle's cell scale: the sum over all deposits at (x,q) of
|w V5 |M|^2 (gain + loss) ...|, the natural magnitude of the rounding error of a
gain-minus-loss difference (A itself vanishes where gain = loss).
"""
import numpy as np
import pytest

from paper_1912_04457_amd import qgbe
from paper_1912_04457_amd import workloads as W

pytestmark = pytest.mark.gpu

SEED = 0x5EED2019
TOL = {qgbe.FP64: 1e-10, qgbe.FP32: 1e-4}


def _case(name):
    print(f"\n[gpu case] {name}", flush=True)


def _grid_kw(wl):
    return dict(n_x=wl.n_x, n_p=wl.n_p, x_half=wl.x_half, p_half=wl.p_half,
                species_mask=wl.species_mask, alpha_s=wl.alpha_s)


def _compare(A, A_ref, S_ref, tol, what=""):
    err = np.abs(A - A_ref)
    bound = tol * S_ref
    bad = err > bound + 1e-300
    assert not bad.any(), (what, int(bad.sum()), float((err / np.maximum(S_ref, 1e-300)).max()))
    l2 = np.linalg.norm((A - A_ref).ravel()) / max(np.linalg.norm(A_ref.ravel()), 1e-300)
    assert l2 <= tol, (what, l2)


def _run_pair(O, wl, f, N, precision, step=0, symmetric=True):
    g = O.Grid(n_x=wl.n_x, n_p=wl.n_p, x_half=wl.x_half, p_half=wl.p_half,
               species_mask=wl.species_mask, alpha_s=wl.alpha_s)
    with qgbe.Solver(**_grid_kw(wl), precision=precision, symmetric=int(symmetric), seed=SEED) as s:
        s.set_f(f)
        qgbe.qgbe_set_step_index(s.ctx, step)
        A, _, I, st = s.collision(N, items=True)
        m_gpu = s.masses()
    m_ref = O.masses(g, f)
    A_ref, S_ref, I_ref = O.collision(g, f, m_ref, SEED, step, N, symmetric=symmetric, want_items=True)
    return dict(A=A, I=I, st=st, m=m_gpu, A_ref=A_ref, S_ref=S_ref, I_ref=I_ref, m_ref=m_ref, grid=g)


def test_device_info():
    torch = pytest.importorskip("torch")
    p = torch.cuda.get_device_properties(0)
    print(f"\n[device] {p.name} CUs={p.multi_processor_count} mem={p.total_memory / 2**30:.0f} GiB "
          f"arch={getattr(p, 'gcnArchName', '?')}", flush=True)
    assert p.multi_processor_count > 0


SMALL_7 = W.Workload("qg7_2cells_5x6x4", (2, 1, 1), (5, 6, 4), (3.0, 3.0, 3.0), (2.0, 2.5, 1.5),
                     0x7F, 100, "f64", 1, 0.01)


@pytest.mark.parametrize("precision", [qgbe.FP64, qgbe.FP32])
def test_gluon_config1(O, precision):
    """1 cell, 10^3 on [-2,2]^3, gg -> gg, f = 0.5 theta(1 - |p|), N = 1000."""
    _case(f"gluon C1 precision={precision}")
    wl = W.C1
    r = _run_pair(O, wl, W.initial_f(wl), 1000, precision)
    assert np.allclose(r["m"], r["m_ref"], rtol=1e-13, atol=0)
    _compare(r["A"], r["A_ref"], r["S_ref"], TOL[precision], "A")
    scale_items = np.abs(r["I_ref"]).max()
    assert np.allclose(r["I"], r["I_ref"], rtol=TOL[precision], atol=TOL[precision] * scale_items)
    assert r["st"].n_evals == 1000 * 1000
    assert r["st"].n_collide_launches >= 1


@pytest.mark.parametrize("precision", [qgbe.FP64, qgbe.FP32])
@pytest.mark.parametrize("symmetric", [True, False])
def test_seven_species_ragged(O, precision, symmetric):
    """70 channels, 2 cells, ragged 5x6x4 grid, N = 100 (not a multiple of 64)."""
    _case(f"7 species ragged precision={precision} symmetric={symmetric}")
    f = W.random_f(21, SMALL_7.cells, SMALL_7.nodes)
    r = _run_pair(O, SMALL_7, f, 100, precision, step=3, symmetric=symmetric)
    assert np.allclose(r["m"], r["m_ref"], rtol=1e-13, atol=0)
    _compare(r["A"], r["A_ref"], r["S_ref"], TOL[precision], "A")


@pytest.mark.parametrize("mask", [1 << 6, 0x7F], ids=["gluons", "qg7"])
def test_partial_node_block_fp32(O, mask):
    """105 momenta (3 x 5 x 7): the compacting variant (the gluon channel) and
    the plain ones, where chunks and the last node block end inside a block of
    4 consecutive nodes."""
    _case(f"3x5x7 nodes mask={mask:#x} fp32")
    wl = W.Workload("2cells_3x5x7", (2, 1, 1), (3, 5, 7), (3.0, 3.0, 3.0), (2.0, 2.5, 1.5),
                    mask, 100, "f32", 1, 0.01)
    f = W.random_f(24, wl.cells, wl.nodes, species_mask=mask)
    r = _run_pair(O, wl, f, 100, qgbe.FP32, step=6)
    # odd on every axis: the centre node at p = 0 (E = 0 for a massless lagged mass)
    assert np.allclose(r["m"], r["m_ref"], rtol=1e-13, atol=0)
    _compare(r["A"], r["A_ref"], r["S_ref"], TOL[qgbe.FP32], "A")
    scale_items = np.abs(r["I_ref"]).max()
    assert np.allclose(r["I"], r["I_ref"], rtol=TOL[qgbe.FP32], atol=TOL[qgbe.FP32] * scale_items)
    assert np.all(r["S_ref"][6, :, -1] > 0)   # the bar binds at the last node


@pytest.mark.parametrize("precision", [qgbe.FP64, qgbe.FP32])
def test_conservation(O, precision):
    _case(f"conservation precision={precision}")
    f = W.random_f(22, SMALL_7.cells, SMALL_7.nodes)
    r = _run_pair(O, SMALL_7, f, 64, precision)
    for cell in range(SMALL_7.cells):
        assert abs(r["A"][:, cell].sum()) <= 1e-13 * r["S_ref"][:, cell].sum()


def test_config3_lds_layout_fp32(O):
    """20^3, 7 species (three-slot channels with one f tile outside LDS), N = 8."""
    _case("C3 layout fp32 N=8")
    wl = W.C3
    f = W.initial_f(wl)
    r = _run_pair(O, wl, f, 8, qgbe.FP32)
    _compare(r["A"], r["A_ref"], r["S_ref"], 1e-4, "A")
    assert abs(r["A"].sum()) <= 1e-13 * r["S_ref"].sum()


@pytest.mark.parametrize("n_p,mask,N", [((32, 32, 32), 1 << 6, 4), ((24, 24, 24), 0x7F, 2),
                                         ((28, 28, 28), 0x7F, 1)],
                         ids=["g_32cube", "qg7_24cube", "qg7_28cube"])
def test_large_grid_lds_plans_fp32(O, n_p, mask, N):
    """Grids whose FP64 accumulators do not fit in LDS: 24^3 holds one slot
    per launch; at 32^3 and 28^3 not even one slot fits, and each slot runs
    as two node windows (launches whose accumulators cover half the nodes,
    corners outside left to the other), f from the global node quads."""
    _case(f"large grid {n_p} mask={mask:#x} N={N}")
    wl = W.C3.scaled(n_p=n_p, species_mask=mask)
    f = W.initial_f(wl)
    r = _run_pair(O, wl, f, N, qgbe.FP32)
    _compare(r["A"], r["A_ref"], r["S_ref"], 1e-4, "A")
    assert abs(r["A"].sum()) <= 1e-13 * r["S_ref"].sum()


def test_spatial_small_fp32(O):
    """4x4x1 cells of a Gaussian transverse profile, 8^3 momenta, N = 96."""
    _case("spatial small fp32")
    wl = W.C2.scaled(n_x=(4, 4, 1), n_p=(8, 8, 8), x_half=(6.0, 6.0, 0.375))
    r = _run_pair(O, wl, W.initial_f(wl), 96, qgbe.FP32)
    _compare(r["A"], r["A_ref"], r["S_ref"], 1e-4, "A")


def test_device_pointers_match_host(O):
    """Torch device tensors through the same ABI give the same result."""
    torch = pytest.importorskip("torch")
    _case("device pointers")
    wl = SMALL_7
    f = W.random_f(23, wl.cells, wl.nodes)
    with qgbe.Solver(**_grid_kw(wl), precision=qgbe.FP64, seed=SEED) as s:
        s.set_f(torch.from_numpy(f).cuda())
        A_dev = torch.zeros((7, wl.cells, wl.nodes), dtype=torch.float64, device="cuda")
        qgbe.qgbe_collision_term(s.ctx, 50, qgbe.SAMPLER_UNIFORM, A_dev)
        torch.cuda.synchronize()
        A_host, _, _, _ = s.collision(50)
    assert np.array_equal(A_dev.cpu().numpy(), A_host) or np.allclose(A_dev.cpu().numpy(), A_host, rtol=1e-12)


def test_step_parity_fp64(O):
    """Three upwind steps on a 2x2x1 spatial grid, dynamic masses, 7 species."""
    _case("step parity fp64")
    wl = W.Workload("qg7_2x2x1_6cube", (2, 2, 1), (6, 6, 6), (3.0, 3.0, 3.0), (2.0, 2.0, 2.0),
                    0x7F, 16, "f64", 3, 0.01)
    g = O.Grid(n_x=wl.n_x, n_p=wl.n_p, x_half=wl.x_half, p_half=wl.p_half, species_mask=wl.species_mask)
    f0 = W.smooth_f(wl.cells, wl.n_p, wl.p_half, amp_g=0.5)
    f0[:, 1:] *= 0.7
    st = O.State(f=f0.copy())
    ref = [O.step(g, st, wl.dt_fm, wl.n_samples, SEED) for _ in range(3)]
    with qgbe.Solver(**_grid_kw(wl), precision=qgbe.FP64, seed=SEED) as s:
        s.set_f(f0)
        stats = s.step(wl.dt_fm, wl.n_samples, n_steps=3)
        f_gpu = s.get_f()
    change = np.abs(st.f - f0).max()
    assert np.abs(f_gpu - st.f).max() <= 1e-10 * change
    for a, b in zip(stats, ref):
        assert a["N_total"] == pytest.approx(b["N_total"], rel=1e-13)
        assert a["E_total"] == pytest.approx(b["E_total"], rel=1e-12)
        assert np.allclose(a["mass2_avg"], b["mass2"].mean(axis=1), rtol=1e-12)
        # energy bookkeeping (Eq. current conservation; modified tensor of Sec. IV)
        assert abs(a["E_source"] - b["E_source"]) <= 1e-12 * b["E_total"]
        assert abs(a["E_collide"] - b["E_collide"]) <= 1e-12 * b["E_total"]
        assert a["E_total_mod"] == pytest.approx(b["E_total_mod"], rel=1e-12)
        assert a["entropy"] == pytest.approx(b["entropy"], rel=1e-12)
        assert np.allclose(a["T_ii"], b["T_ii"], rtol=1e-12)
    assert stats[0]["E_source"] == 0.0 and stats[1]["E_source"] != 0.0
    N0 = O.observables(g, f0, O.masses(g, f0))["N_total"]
    assert abs(stats[-1]["N_total"] - N0) <= 1e-13 * N0


def test_energy_source_accounts_for_kinetic_energy_change():
    """The energy test of Sec. IV with dynamic masses: in a homogeneous pure
    gluon system the kinetic energy changes by the mass source term plus the
    collision term's grid residue, step by step (FP32 integrand; the
    bookkeeping itself is FP64)."""
    _case("energy bookkeeping fp32")
    wl = W.Workload("g_1cell_10cube", (1, 1, 1), (10, 10, 10), (3.0, 3.0, 3.0), (2.0, 2.0, 2.0),
                    1 << 6, 128, "f32", 4, 0.01)
    P = W.node_momenta(wl.n_p, wl.p_half)
    f0 = np.zeros((7, 1, wl.nodes))
    f0[6, 0] = 0.5 * (np.linalg.norm(P, axis=1) < 1.5)
    with qgbe.Solver(**_grid_kw(wl), precision=qgbe.FP32, seed=SEED) as s:
        s.set_f(f0)
        stats = s.step(wl.dt_fm, wl.n_samples, n_steps=4)
    for k in range(1, 4):
        change = stats[k]["E_total"] - stats[k - 1]["E_total"]
        parts = stats[k]["E_source"] + stats[k]["E_collide"]
        assert abs(change - parts) <= 1e-12 * stats[k]["E_total"], k
        assert abs(stats[k]["E_collide"]) < 0.05 * abs(stats[k]["E_source"])
    assert all(st["E_total_mod"] < st["E_total"] for st in stats)


def test_step_parity_central_fp32(O):
    _case("step parity central fp32")
    wl = W.Workload("g_3x1x1_8cube", (3, 1, 1), (8, 8, 8), (3.0, 3.0, 3.0), (2.0, 2.0, 2.0),
                    1 << 6, 32, "f32", 2, 0.01, drift="central")
    g = O.Grid(n_x=wl.n_x, n_p=wl.n_p, x_half=wl.x_half, p_half=wl.p_half, species_mask=wl.species_mask)
    f0 = W.smooth_f(wl.cells, wl.n_p, wl.p_half, species_mask=wl.species_mask)
    f0[6, 0] *= 1.3
    st = O.State(f=f0.copy())
    for _ in range(2):
        O.step(g, st, wl.dt_fm, wl.n_samples, SEED, scheme="central")
    with qgbe.Solver(**_grid_kw(wl), precision=qgbe.FP32, drift=qgbe.DRIFT_CENTRAL, seed=SEED) as s:
        s.set_f(f0)
        stats = s.step(wl.dt_fm, wl.n_samples, n_steps=2)
        f_gpu = s.get_f()
    change = np.abs(st.f - f0).max()
    assert np.abs(f_gpu - st.f).max() <= 1e-4 * change
    N0 = O.observables(g, f0, O.masses(g, f0))["N_total"]
    assert abs(stats[-1]["N_total"] - N0) <= 1e-13 * N0


def test_constant_mass_and_flags(O):
    _case("constant mass + flags")
    wl = W.C1
    f = W.initial_f(wl)
    f[6, 0, 0] = -0.1           # a negative occupation must be flagged
    cm = [0.1] * 6 + [0.5]
    with qgbe.Solver(**_grid_kw(wl), precision=qgbe.FP64, mass_mode=qgbe.MASS_CONSTANT,
                     const_mass2=cm, seed=SEED) as s:
        s.set_f(f)
        st = qgbe.Stats()
        qgbe.qgbe_observables(s.ctx, st)
        assert np.allclose(s.masses()[:, 0], cm)
        assert st.flags & qgbe.FLAG_NEGATIVE_F
    g = O.Grid(n_p=wl.n_p, p_half=wl.p_half, species_mask=wl.species_mask)
    ref = O.observables(g, f, O.constant_masses(g, cm))
    assert st.N_total == pytest.approx(ref["N_total"], rel=1e-13)
    assert st.E_total == pytest.approx(ref["E_total"], rel=1e-13)


def test_empty_distribution_gives_zero(O):
    _case("empty f")
    with qgbe.Solver(**_grid_kw(SMALL_7), precision=qgbe.FP32, seed=SEED) as s:
        A, _, _, _ = s.collision(64)
    assert np.all(A == 0.0)


def test_errors_reported():
    _case("error paths")
    with qgbe.Solver(**_grid_kw(SMALL_7), precision=qgbe.FP32, seed=SEED) as s:
        with pytest.raises(qgbe.QgbeError) as e:
            qgbe.qgbe_collision_term(s.ctx, 0, qgbe.SAMPLER_UNIFORM, np.zeros((7, 2, 120)))
        assert e.value.status == qgbe.EINVAL
        with pytest.raises(qgbe.QgbeError):
            qgbe.qgbe_set_distribution(s.ctx, 9, np.zeros((2, 120)))
        with pytest.raises(qgbe.QgbeError):
            qgbe.qgbe_step(s.ctx, -1.0, 8, 0, 1)


@pytest.mark.parametrize("precision", [qgbe.FP64, qgbe.FP32])
def test_mc_error_estimate_matches_replicas(precision):
    """stats.mc_err_est (from each item's own samples) against the spread of
    the item sums over independent replicas (other step indices)."""
    _case(f"mc error estimate precision={precision}")
    wl = W.C3.scaled(n_p=(8, 8, 8))
    R, N = 16, 256
    with qgbe.Solver(**_grid_kw(wl), precision=precision, seed=SEED) as s:
        s.set_f(W.initial_f(wl))
        est, items = [], []
        for r in range(R):
            qgbe.qgbe_set_step_index(s.ctx, 100 + r)
            _, _, I, st = s.collision(N, items=True)
            est.append(st.mc_err_est)
            items.append(I)
    I = np.array(items)
    emp = np.sqrt(I.var(0, ddof=1).sum() / (I.mean(0) ** 2).sum())
    print(f"[mc error] estimate {np.mean(est):.4f} (spread {np.std(est):.4f}), replicas {emp:.4f}", flush=True)
    assert 0.8 < np.mean(est) / emp < 1.25


@pytest.mark.parametrize("n_x,n_p,mask,N", [((1, 1, 1), (2, 2, 2), 1 << 6, 1000), ((1, 1, 1), (9, 8, 7), 1 << 6, 130),
                                            ((1, 1, 1), (16, 16, 16), 0x41, 65), ((3, 1, 1), (5, 6, 7), 0x7F, 193),
                                            ((1, 1, 1), (16, 15, 17), 1 << 6, 1100)],
                         ids=["8nodes", "one_pair", "three_channels", "pairs_and_cus", "long_items"])
def test_waves_share_nodes_fp32(O, n_x, n_p, mask, N):
    """Fewer (cell, channel) pairs than compute units: several waves of a
    workgroup share a node, each a part of its samples (some waves with none,
    the last part short), and the item sums and the error estimate come from
    the parts; the scale output takes the same way."""
    _case(f"shared nodes {n_x} {n_p} mask={mask:#x} N={N}")
    wl = W.Workload("shared", n_x, n_p, (3.0, 3.0, 3.0), (2.0, 2.5, 1.5), mask, N, "f32", 1, 0.01)
    f = W.random_f(25, wl.cells, wl.nodes, species_mask=mask)
    r = _run_pair(O, wl, f, N, qgbe.FP32, step=2)
    _compare(r["A"], r["A_ref"], r["S_ref"], TOL[qgbe.FP32], "A")
    scale_items = np.abs(r["I_ref"]).max()
    assert np.allclose(r["I"], r["I_ref"], rtol=TOL[qgbe.FP32], atol=TOL[qgbe.FP32] * scale_items)
    with qgbe.Solver(**_grid_kw(wl), precision=qgbe.FP64, seed=SEED) as s:
        s.set_f(f)
        qgbe.qgbe_set_step_index(s.ctx, 2)
        _, S, _, st = s.collision(N, scale=True)
    with qgbe.Solver(**_grid_kw(wl), precision=qgbe.FP32, seed=SEED) as s:
        s.set_f(f)
        qgbe.qgbe_set_step_index(s.ctx, 2)
        A2, S2, _, st2 = s.collision(N, scale=True)
    _compare(A2, r["A_ref"], r["S_ref"], TOL[qgbe.FP32], "A with scale")
    assert np.all(np.abs(S2 - S) <= TOL[qgbe.FP32] * S + 1e-300)
    assert st2.n_accepted == st.n_accepted == r["st"].n_accepted
    if np.isfinite(st.mc_err_est):
        assert st2.mc_err_est == pytest.approx(st.mc_err_est, rel=1e-2)


@pytest.mark.parametrize("n_x,n_p,mask,N", [((1, 1, 1), (28, 29, 28), 1 << 6, 3), ((1, 1, 1), (20, 20, 20), 0x7F, 2),
                                            ((2, 1, 1), (15, 16, 14), 0x49, 40), ((1, 1, 1), (9, 8, 7), 1 << 6, 1025)],
                         ids=["windows", "slot_passes", "plain_and_queue", "shared_nodes"])
def test_lds_plans_fp64(O, n_x, n_p, mask, N):
    """The FP64 kernel's LDS plans: one slot over two node windows, three slots
    over two launches, groups with and without the compacting variant, and
    waves that share a node."""
    _case(f"fp64 plans {n_x} {n_p} mask={mask:#x} N={N}")
    wl = W.Workload("plans", n_x, n_p, (3.0, 3.0, 3.0), (2.0, 2.5, 1.5), mask, N, "f64", 1, 0.01)
    f = W.random_f(26, wl.cells, wl.nodes, species_mask=mask)
    r = _run_pair(O, wl, f, N, qgbe.FP64, step=2)
    _compare(r["A"], r["A_ref"], r["S_ref"], TOL[qgbe.FP64], "A")
    scale_items = np.abs(r["I_ref"]).max()
    assert np.allclose(r["I"], r["I_ref"], rtol=TOL[qgbe.FP64], atol=TOL[qgbe.FP64] * scale_items)
    for cell in range(wl.cells):
        assert abs(r["A"][:, cell].sum()) <= 1e-13 * r["S_ref"][:, cell].sum()


@pytest.mark.parametrize("n_x,n_p", [((1, 1, 1), (24, 25, 23)), ((511, 1, 1), (2, 2, 3)), ((600, 1, 1), (3, 2, 2)),
                                     ((3, 1, 1), (13, 14, 15))], ids=["one_cell", "511_cells", "600_cells", "parts"])
@pytest.mark.parametrize("precision", [qgbe.FP64, qgbe.FP32])
def test_masses_at_the_start_of_a_term(O, n_x, n_p, precision):
    """The masses that a collision term forms in its first pass over f: cells
    split over workgroups, and few and many cells (the sum over a cell's parts
    by its last workgroup or by a second kernel)."""
    _case(f"term start {n_x} {n_p} precision={precision}")
    wl = W.Workload("start", n_x, n_p, (3.0, 3.0, 3.0), (2.0, 2.5, 1.5), 0x7F, 1, "f64", 1, 0.01)
    f = W.random_f(29, wl.cells, wl.nodes)
    g = O.Grid(n_x=wl.n_x, n_p=wl.n_p, x_half=wl.x_half, p_half=wl.p_half, species_mask=0x7F)
    with qgbe.Solver(**_grid_kw(wl), precision=precision, seed=SEED) as s:
        for scale in (1.0, 0.5):  # the second time on other values
            s.set_f(scale * f)
            s.collision(1)
            assert np.allclose(s.masses(), O.masses(g, scale * f), rtol=1e-13, atol=0)


@pytest.mark.parametrize("N", [1, 64, 200, 1088], ids=["one", "one_batch", "short", "long"])
def test_small_queue_fp32(O, N):
    """Two slots whose accumulators leave room for the smaller of the sample
    queues only: batches that fill exactly, overflow and end partly filled, in
    the short and the long form of an item."""
    _case(f"small queue N={N}")
    wl = W.Workload("queue", (1, 1, 1), (17, 17, 17), (3.0, 3.0, 3.0), (2.0, 2.5, 1.5), 0x49, N, "f32", 1, 0.01)
    r = _run_pair(O, wl, W.random_f(27, 1, wl.nodes, species_mask=0x49), N, qgbe.FP32, step=2)
    _compare(r["A"], r["A_ref"], r["S_ref"], TOL[qgbe.FP32], "A")
    scale_items = np.abs(r["I_ref"]).max()
    assert np.allclose(r["I"], r["I_ref"], rtol=TOL[qgbe.FP32], atol=TOL[qgbe.FP32] * scale_items)
    assert abs(r["A"].sum()) <= 1e-13 * r["S_ref"].sum()


@pytest.mark.parametrize("n_x,n_p,mask,N,precision,learned",
                         [((1, 1, 1), (20, 20, 20), 0x7F, 80, qgbe.FP32, False),
                          ((2, 1, 1), (18, 19, 20), 0x49, 40, qgbe.FP64, False),
                          ((1, 1, 1), (40, 39, 41), 1 << 6, 5, qgbe.FP32, False),
                          ((2, 1, 1), (28, 27, 29), 1 << 6, 70, qgbe.FP32, True),
                          ((1, 1, 1), (19, 20, 21), 0x43, 30, qgbe.FP64, True),
                          ((1, 1, 1), (28, 28, 28), 1 << 6, 1500, qgbe.FP32, False)],
                         ids=["batches", "cells_f64", "four_windows", "learned_cells", "learned_f64", "long_items"])
def test_recorded_deposits(O, n_x, n_p, mask, N, precision, learned):
    """Grids whose deposit accumulators take more than one launch: the samples
    are drawn once and their deposits recorded and replayed, in one batch or
    several, over one node window or several, for every sampler and precision;
    with the scale output the same term draws its samples in every launch."""
    _case(f"recorded deposits {n_x} {n_p} mask={mask:#x} N={N} precision={precision} learned={learned}")
    wl = W.Workload("recorded", n_x, n_p, (3.0, 3.0, 3.0), (2.0, 2.5, 1.5), mask, N, "f32", 1, 0.01)
    f = W.random_f(27, wl.cells, wl.nodes, species_mask=mask)
    g = O.Grid(n_x=n_x, n_p=n_p, x_half=wl.x_half, p_half=wl.p_half, species_mask=mask, alpha_s=wl.alpha_s)
    with qgbe.Solver(**_grid_kw(wl), precision=precision, seed=SEED) as s:
        s.set_f(f)
        qgbe.qgbe_set_step_index(s.ctx, 4)
        if learned:
            table = W.random_mog_table(5, s.n_channels * wl.nodes)
            qgbe.qgbe_set_proposal_table(s.ctx, *table)
        sampler = qgbe.SAMPLER_LEARNED if learned else qgbe.SAMPLER_UNIFORM
        A, _, I, st = s.collision(N, sampler=sampler, items=True)
        A2, S2, I2, st2 = s.collision(N, sampler=sampler, scale=True, items=True)
        m = s.masses()
    if learned:
        A_ref, S_ref, I_ref = O.collision_learned(g, f, m, SEED, 4, N, *table, want_items=True)
    else:
        A_ref, S_ref, I_ref = O.collision(g, f, m, SEED, 4, N, want_items=True)
    for a, i in ((A, I), (A2, I2)):
        _compare(a, A_ref, S_ref, TOL[precision], "A")
        assert np.allclose(i, I_ref, rtol=TOL[precision], atol=TOL[precision] * np.abs(I_ref).max())
    for cell in range(wl.cells):
        assert abs(A[:, cell].sum()) <= 1e-13 * S_ref[:, cell].sum()
    assert st.n_accepted == st2.n_accepted
    assert st.mc_err_est == pytest.approx(st2.mc_err_est, rel=1e-9)


@pytest.mark.parametrize("n_x,n_p,mask,N,learned", [((1, 1, 1), (27, 27, 28), 1 << 6, 70, False),
                                                    ((2, 1, 1), (20, 20, 25), 0x49, 3, False),
                                                    ((1, 1, 1), (26, 27, 27), 1 << 6, 70, True),
                                                    ((2, 1, 1), (21, 20, 23), 0x49, 3, True)],
                         ids=["one_slot", "two_slots", "learned", "learned_two_slots"])
def test_long_form_of_short_items_fp32(O, n_x, n_p, mask, N, learned):
    """Grids whose accumulators fit in one launch beside the long-item form's own
    LDS only: that form runs for short items too."""
    _case(f"long form {n_x} {n_p} mask={mask:#x} N={N} learned={learned}")
    wl = W.Workload("long", n_x, n_p, (3.0, 3.0, 3.0), (2.0, 2.5, 1.5), mask, N, "f32", 1, 0.01)
    f = W.random_f(28, wl.cells, wl.nodes, species_mask=mask)
    g = O.Grid(n_x=n_x, n_p=n_p, x_half=wl.x_half, p_half=wl.p_half, species_mask=mask, alpha_s=wl.alpha_s)
    with qgbe.Solver(**_grid_kw(wl), precision=qgbe.FP32, seed=SEED) as s:
        s.set_f(f)
        qgbe.qgbe_set_step_index(s.ctx, 4)
        if learned:
            table = W.random_mog_table(5, s.n_channels * wl.nodes)
            qgbe.qgbe_set_proposal_table(s.ctx, *table)
        sampler = qgbe.SAMPLER_LEARNED if learned else qgbe.SAMPLER_UNIFORM
        A, _, I, _ = s.collision(N, sampler=sampler, items=True)
        A2, _, I2, _ = s.collision(N, sampler=sampler, scale=True, items=True)
        m = s.masses()
    if learned:
        A_ref, S_ref, I_ref = O.collision_learned(g, f, m, SEED, 4, N, *table, want_items=True)
    else:
        A_ref, S_ref, I_ref = O.collision(g, f, m, SEED, 4, N, want_items=True)
    for a, i in ((A, I), (A2, I2)):
        _compare(a, A_ref, S_ref, TOL[qgbe.FP32], "A")
        assert np.allclose(i, I_ref, rtol=TOL[qgbe.FP32], atol=TOL[qgbe.FP32] * np.abs(I_ref).max())


@pytest.mark.parametrize("n_p,sampler", [((66, 68, 70), qgbe.SAMPLER_UNIFORM), ((56, 57, 58), qgbe.SAMPLER_ROOTS),
                                         ((56, 57, 58), qgbe.SAMPLER_ROOTS_ALT), ((56, 57, 58), qgbe.SAMPLER_LEARNED)],
                         ids=["uniform", "roots", "roots_alt", "learned"])
def test_deposits_with_global_atomics(O, n_p, sampler):
    """FP64 grids of so many node windows that, with the scale output, one launch
    deposits with global atomics; against the oracle, and against the same term
    without that output, which records its deposits."""
    _case(f"global atomics {n_p} sampler={sampler}")
    wl = W.Workload("large", (1, 1, 1), n_p, (3.0, 3.0, 3.0), (2.0, 2.5, 1.5), 1 << 6, 4, "f64", 1, 0.01)
    f = W.random_f(28, 1, wl.nodes, species_mask=1 << 6) * 0.6
    g = O.Grid(n_x=(1, 1, 1), n_p=n_p, x_half=wl.x_half, p_half=wl.p_half, species_mask=1 << 6, alpha_s=wl.alpha_s)
    with qgbe.Solver(**_grid_kw(wl), precision=qgbe.FP64, seed=SEED) as s:
        s.set_f(f)
        if sampler == qgbe.SAMPLER_LEARNED:
            table = W.random_mog_table(5, s.n_channels * wl.nodes)
            qgbe.qgbe_set_proposal_table(s.ctx, *table)
        A, S, I, st = s.collision(4, sampler=sampler, scale=True, items=True)
        A2, _, I2, st2 = s.collision(4, sampler=sampler, items=True)
        m = s.masses()
    assert st.n_collide_launches == 1 and st2.n_collide_launches > 1
    if sampler == qgbe.SAMPLER_LEARNED:
        A_ref, S_ref, I_ref = O.collision_learned(g, f, m, SEED, 0, 4, *table, want_items=True)
    else:
        est = {qgbe.SAMPLER_UNIFORM: "cm", qgbe.SAMPLER_ROOTS: "root", qgbe.SAMPLER_ROOTS_ALT: "root_k3"}[sampler]
        A_ref, S_ref, I_ref = O.collision(g, f, m, SEED, 0, 4, estimator=est, want_items=True)
    # a node without a deposit may get the rounding of a stencil weight (a few
    # 2^-53 of the grid coordinate) from a sample on the face of its cell
    hit, most = S_ref > 0.0, S_ref.max()
    for a in (A, A2):
        assert np.all(np.abs(a - A_ref)[hit] <= 1e-10 * S_ref[hit])
        assert np.all(np.abs(a)[~hit] <= 8 * 2.0 ** -53 * max(n_p) * most)
        assert abs(a.sum()) <= 1e-13 * S_ref.sum()
    assert np.abs(I - I2).max() <= 1e-12 * np.abs(I_ref).max()
    assert st.n_accepted == st2.n_accepted > 0
