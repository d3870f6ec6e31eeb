"""Degenerate configurations through the C ABI against the FP64 oracle: species
subsets (channel tables without gluons, with one quark flavour, a single
species), the smallest grid the method allows (2 nodes per axis, where every
stencil spans the whole axis), a single sample per point (one lane of a
wavefront), massless particles on a grid with a node at p = 0, for the
CM-angle sampler in both precisions and the paper's root parameterisation
(FP64 in either context).  Bars as in the other parity
tests: FP64 1e-10 and FP32 1e-4 of the oracle's scale S, element by element,
and number conservation per cell."""
import numpy as np
import pytest

from paper_1912_04457_amd import qgbe
from paper_1912_04457_amd import workloads as W

pytestmark = pytest.mark.gpu

SEED = 0x5EED2019
TOL = {qgbe.FP64: 1e-10, qgbe.FP32: 1e-4}
EST = {qgbe.SAMPLER_UNIFORM: "cm", qgbe.SAMPLER_ROOTS: "root", qgbe.SAMPLER_ROOTS_ALT: "root_k3"}

MASKS = {"u": 1 << 0, "u_ubar": (1 << 0) | (1 << 3), "s_g": (1 << 2) | (1 << 6), "u_d_g": 0x43}


def _case(name):
    print(f"\n[gpu case] {name}", flush=True)


def _pair(O, n_x, n_p, mask, f, N, precision, sampler, p_half=(2.0, 2.5, 1.5)):
    g = O.Grid(n_x=n_x, n_p=n_p, x_half=(3.0, 3.0, 3.0), p_half=p_half, species_mask=mask)
    with qgbe.Solver(n_x=n_x, n_p=n_p, x_half=(3.0, 3.0, 3.0), p_half=p_half, species_mask=mask,
                     alpha_s=g.alpha_s, seed=SEED, precision=precision) as s:
        s.set_f(f)
        qgbe.qgbe_set_step_index(s.ctx, 5)
        A, S, _, st = s.collision(N, sampler=sampler, scale=True)
        m = s.masses()
    A_ref, S_ref, _ = O.collision(g, f, m, SEED, 5, N, estimator=EST[sampler])
    return g, A, S, st, A_ref, S_ref


def _check(g, A, A_ref, S_ref, tol):
    err = np.abs(A - A_ref)
    assert np.all(err <= tol * S_ref + 1e-300), float((err / np.maximum(S_ref, 1e-300)).max())
    for cell in range(g.cells):
        assert abs(A[:, cell].sum()) <= 1e-13 * S_ref[:, cell].sum() + 1e-300


@pytest.mark.parametrize("precision", [qgbe.FP64, qgbe.FP32])
@pytest.mark.parametrize("name", sorted(MASKS))
def test_species_subsets(O, name, precision):
    mask = MASKS[name]
    _case(f"species subset {name} precision={precision}")
    n_x, n_p = (2, 1, 1), (3, 4, 5)
    f = W.random_f(51, 2, int(np.prod(n_p)), species_mask=mask) * 0.7
    g, A, S, st, A_ref, S_ref = _pair(O, n_x, n_p, mask, f, 37, precision, qgbe.SAMPLER_UNIFORM)
    assert len(O.channels(g)) >= 1 and S_ref.max() > 0.0
    _check(g, A, A_ref, S_ref, TOL[precision])
    # species outside the mask never change
    out = [sp for sp in range(7) if not (mask >> sp) & 1]
    assert np.all(A[out] == 0.0)


@pytest.mark.parametrize("sampler", [qgbe.SAMPLER_UNIFORM, qgbe.SAMPLER_ROOTS, qgbe.SAMPLER_ROOTS_ALT])
@pytest.mark.parametrize("precision", [qgbe.FP64, qgbe.FP32])
def test_smallest_grid_single_sample(O, sampler, precision):
    _case(f"2^3 nodes, one sample, sampler={sampler} precision={precision}")
    n_x, n_p = (1, 1, 1), (2, 2, 2)
    f = W.random_f(52, 1, 8) * 0.5
    g, A, S, st, A_ref, S_ref = _pair(O, n_x, n_p, 0x7F, f, 1, precision, sampler)
    tol = TOL[precision] if sampler == qgbe.SAMPLER_UNIFORM else 1e-10
    _check(g, A, A_ref, S_ref, tol)


@pytest.mark.parametrize("precision", [qgbe.FP64, qgbe.FP32])
def test_frozen_species_stay_fixed_across_steps(precision):
    """A step updates only the evolving species; the others keep their values
    in both buffers of f, also after one of them is set anew between steps
    (an odd and an even number of steps after the setting)."""
    _case(f"frozen species across steps precision={precision}")
    n_x, n_p = (2, 1, 1), (4, 4, 4)
    mask = (1 << 0) | (1 << 6)                    # u and g evolve
    f = W.random_f(53, 2, 64) * 0.4               # every species occupied
    frozen = [sp for sp in range(7) if not (mask >> sp) & 1]
    with qgbe.Solver(n_x=n_x, n_p=n_p, x_half=(3.0, 3.0, 3.0), p_half=(2.0, 2.0, 2.0), species_mask=mask,
                     seed=SEED, precision=precision) as s:
        s.set_f(f)
        st = s.step(0.01, 32, n_steps=3)
        # every step launches at least one collision kernel, the same launches each step
        assert st[0]["n_collide_launches"] >= 1
        assert all(x["n_collide_launches"] == st[0]["n_collide_launches"] for x in st)
        g1 = s.get_f()
        assert np.array_equal(g1[frozen], f[frozen])
        assert not np.array_equal(g1[0], f[0]) and not np.array_equal(g1[6], f[6])
        f_d = np.full((1, 2, 64), 0.123)
        s.set_f(f_d, species=1)
        for n in (1, 2):
            s.step(0.01, 32, n_steps=n)
            g2 = s.get_f()
            assert np.all(g2[1] == 0.123)
            assert np.array_equal(np.delete(g2[frozen], frozen.index(1), axis=0),
                                  np.delete(f[frozen], frozen.index(1), axis=0))


@pytest.mark.parametrize("precision", [qgbe.FP64, qgbe.FP32])
@pytest.mark.parametrize("mask", [1 << 6, 0x43], ids=["g", "u_d_g"])
def test_massless_node_at_origin(O, mask, precision):
    """Constant zero masses on a grid odd on every axis (3 x 5 x 7): the node
    at p = 0 has E = 0, so as the observed particle it carries no weight; it
    still takes the deposits of other samples.  Unregulated poles make the
    scale S large; the bars are relative to it as everywhere."""
    _case(f"massless, node at p = 0, mask={mask:#x} precision={precision}")
    n_x, n_p, p_half = (2, 1, 1), (3, 5, 7), (2.0, 2.5, 1.5)
    f = W.random_f(57, 2, 105, species_mask=mask) * 0.5
    g = O.Grid(n_x=n_x, n_p=n_p, x_half=(3.0, 3.0, 3.0), p_half=p_half, species_mask=mask)
    centre = 52                                  # node (1, 2, 3)
    assert np.all(g.momenta()[centre] == 0.0)
    with qgbe.Solver(n_x=n_x, n_p=n_p, x_half=(3.0, 3.0, 3.0), p_half=p_half, species_mask=mask,
                     alpha_s=g.alpha_s, seed=SEED, precision=precision,
                     mass_mode=qgbe.MASS_CONSTANT, const_mass2=(0.0,) * 7) as s:
        s.set_f(f)
        qgbe.qgbe_set_step_index(s.ctx, 5)
        A, _, I, _ = s.collision(64, items=True)
        assert np.all(s.masses() == 0.0)
    A_ref, S_ref, I_ref = O.collision(g, f, np.zeros((7, 2)), SEED, 5, 64, want_items=True)
    _check(g, A, A_ref, S_ref, TOL[precision])
    assert np.all(np.isfinite(A)) and np.all(S_ref[6, :, centre] > 0)
    # the observed particle at p = 0: no direct sums
    assert np.all(I.reshape(2, -1, 105)[:, :, centre] == 0.0)
    assert np.all(I_ref.reshape(2, -1, 105)[:, :, centre] == 0.0)
