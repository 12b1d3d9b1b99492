"""GPU parity of the Symanzik gauge force and action (hisq_gauge_force,
hisq_gauge_action) against the FP64 oracle, link by link.

Bar: FP64, 1e-13 relative l2 over the force links and 1e-12 per link; the
action to 1e-13 relative.  Derived from the arithmetic: each force link is
a weighted sum of 48 loop products of at most five 3x3 factors of norm 1
(about 10^3 roundings at 2^-53 of O(1) terms), well inside 1e-13, while a
wrong or missing loop changes it by O(|coef|).

At 32^4 the input is an 8^4 field tiled four times per axis and rotated by a
random gauge transformation g: the force at x transforms as g(x) F g(x)^+ and
the action is invariant, so g (tiled oracle force) g^+ and 256 times the
8^4 action are exact answers for every link.
"""
import numpy as np
import pytest

import oracle
from _parity import check
from paper_1712_00143_amd import synth

pytestmark = pytest.mark.gpu

TOL = 1e-13
ONE_LOOP = (1.0, -0.0833, -0.0133)


def _hisq():
    from paper_1712_00143_amd import hisq
    return hisq


def _links(a):
    return np.asarray(a).reshape(-1, 9)


def _dag(m):
    return np.conj(np.swapaxes(m, -1, -2))


# (32, 8, 16, 4): the brick tile order (two whole x rows per tile, y and z
# multiples of 8) on a field that is not a tiled copy
@pytest.mark.parametrize("dims", [(4, 4, 6, 10), (6, 4, 4, 4), (8, 8, 8, 8), (32, 8, 16, 4)])
@pytest.mark.parametrize("coefs", [(1.0, 0.0, 0.0), (0.0, 1.0, 0.0), (0.0, 0.0, 1.0), ONE_LOOP])
def test_force_and_action_parity(dims, coefs):
    H = _hisq()
    lat = H.Lattice(dims)
    U = synth.thin_links(dims, 0.5, 120)
    F = lat.gauge_force(U, 5.8, coefs)
    check(_links(F), _links(oracle.gauge_force(dims, U, 5.8, coefs)), TOL, ("force", dims, coefs))
    s_ref = oracle.gauge_action(dims, U, 5.8, coefs)
    s = lat.gauge_action(U, 5.8, coefs)
    assert abs(s - s_ref) <= TOL * abs(s_ref), (s, s_ref)
    assert lat.gauge_action(U, 5.8, coefs) == s        # fixed-order reduction
    lat.close()


# 32^4: runs of 8 time slices per block; 24^3x48: runs of 5 with a last run of 3
@pytest.mark.parametrize("small,reps", [((8, 8, 8, 8), (4, 4, 4, 4)), ((12, 12, 12, 12), (2, 2, 2, 4))],
                         ids=["32x32x32x32", "24x24x24x48"])
def test_force_tiled_and_gauge_rotated(small, reps):
    import torch
    H = _hisq()
    dims = tuple(a * b for a, b in zip(small, reps))
    ncopy = reps[0] * reps[1] * reps[2] * reps[3]
    U8 = synth.thin_links(small, 0.5, 121)
    F8 = oracle.gauge_force(small, U8, 6.0, ONE_LOOP)
    s8 = oracle.gauge_action(small, U8, 6.0, ONE_LOOP)
    g = synth.random_su3(synth.volume(dims), 122)
    U = synth.gauge_transform(synth.tile_field(U8, small, reps), dims, g)
    Ft = synth.tile_field(F8, small, reps)
    ref = np.empty_like(Ft)
    for mu in range(4):
        ref[:, mu] = g @ Ft[:, mu] @ _dag(g)
    del Ft
    lat = H.Lattice(dims)
    t = torch.from_numpy(U.view(np.float64)).cuda()
    del U
    F = lat.gauge_force(t, 6.0, ONE_LOOP)
    check(_links(F.cpu().numpy().view(np.complex128)), _links(ref), TOL, ("force", dims))
    s = lat.gauge_action(t, 6.0, ONE_LOOP)
    assert abs(s - ncopy * s8) <= 1e-12 * abs(s), (s, ncopy * s8)
    lat.close()


def test_small_extents_are_refused():
    H = _hisq()
    dims = (2, 4, 4, 4)
    lat = H.Lattice(dims)
    U = synth.thin_links(dims, 0.4, 1)
    with pytest.raises(H.HisqError) as e:
        lat.gauge_force(U, 6.0, ONE_LOOP)
    assert e.value.status == H.HISQ_ERR_ARG
    with pytest.raises(H.HisqError):
        lat.gauge_action(U, 6.0, ONE_LOOP)
    lat.close()


@pytest.mark.parametrize("coefs", [(1.0, -0.08, -0.01), (0.0, 1.0, 0.0), (0.7, 0.0, 0.2)])
@pytest.mark.parametrize("dims", [(6, 14, 10, 12), (10, 6, 12, 14), (34, 4, 4, 16), (8, 8, 8, 16), (8, 8, 8, 18)])
def test_gauge_force_ragged_even_tiles(dims, coefs):
    """The kernel around even sites takes tiles of 64 even sites in groups of
    about four time slices; it serves lattices above 8192 sites.  The largest
    that it does not take and, of those it takes, whole tiles (72, 68) and ragged
    last ones (78.75), partial last groups, x extents that do not divide a tile, and the
    loop classes switched off."""
    H = _hisq()
    U = synth.thin_links(dims, 0.4, 71)
    lat = H.Lattice(dims)
    F = lat.gauge_force(U, 6.5, coefs)
    check(np.asarray(F).reshape(-1, 9), oracle.gauge_force(dims, U, 6.5, coefs).reshape(-1, 9), 1e-13, (dims, coefs))
    lat.close()


@pytest.mark.parametrize("coefs", [(1.0, -0.08, -0.01), (0.0, 1.0, 0.0), (1.0, -0.08, 0.0)])
@pytest.mark.parametrize("dims", [(8, 8, 16, 16), (6, 14, 14, 14), (34, 4, 4, 32), (10, 12, 12, 12), (20, 6, 10, 14)])
def test_gauge_force_either_side_of_the_rectangle_line(dims, coefs):
    """With rectangles the kernel around even sites starts above 16384 sites:
    the largest lattice that the direct sum takes and, of those above, ragged and
    whole last tiles of 64 even sites, x extents that do not divide a tile."""
    H = _hisq()
    U = synth.thin_links(dims, 0.4, 72)
    lat = H.Lattice(dims)
    F = lat.gauge_force(U, 6.5, coefs)
    check(np.asarray(F).reshape(-1, 9), oracle.gauge_force(dims, U, 6.5, coefs).reshape(-1, 9), 1e-13, (dims, coefs))
    lat.close()
