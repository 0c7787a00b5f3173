"""Routes of the step kernels at the sizes where they can go wrong, each against
the FP64 oracle within the bounds of test_gpu_parity: stencil boxes that wrap
around periodic axes."""
import numpy as np
import pytest

import oracle
from lbcase import CHAIN_BOND, Case
from paper_0809_4958_amd import inputs
from test_gpu_parity import STORE, check, compare, make_ctx, say

pytestmark = pytest.mark.gpu

lbm = pytest.importorskip("paper_0809_4958_amd.lbm")


class NearestImage:
    """The oracle's box with every chain moved, exactly, to the periodic image
    nearest the origin, its bead positions moved back.  The oracle integrates
    absolute coordinates: at 12 nodes their rounding (an ulp of 1.8e-15) alone
    moves a compact chain's bead velocities by 1.2e-12 of a fluid velocity of
    1e-3 in 14 steps (the oracle against itself on the other image)."""

    def __init__(self, case):
        self.shift, chains = [], []
        for c in case.chains:
            by = np.array([float(n) if case.pmask >> a & 1 and c["anchor"][a] > n / 2 else 0.0
                           for a, n in enumerate(case.dims)])
            chains.append(dict(c, pos=np.asarray(c["pos"]) - by, anchor=list(np.asarray(c["anchor"]) - by)))
            self.shift.append(np.tile(by, (len(c["pos"]), 1)))
        own = case.chains
        case.chains = chains
        self.box = case.oracle_box()
        case.chains = own

    def beads(self):
        p, v = self.box.beads()
        return p + np.concatenate(self.shift), v

    def __getattr__(self, name):
        return getattr(self.box, name)


def run_case(case, storage, steps, label, **kw):
    """One case on the oracle and the library; asserts the parity bounds."""
    say("case", label, storage)
    ob = NearestImage(case) if case.pmask and case.chains else case.oracle_box()
    assert ob.step(steps) == 0
    ctx = make_ctx(case, storage, **kw)
    ctx.step(steps)
    assert ctx.sync_status() == lbm.OK
    check(compare(ctx, ob, case, storage), storage, label)
    ctx.close()


@pytest.mark.parametrize("streaming", ["two_buffers", "in_place"])
@pytest.mark.parametrize("storage", ["f64", "f32", "f16"])
@pytest.mark.parametrize("dims,pmask", [((13, 11, 9), 7), ((9, 4, 12), 2), ((10, 12, 5), 5), ((5, 5, 5), 7)])
def test_chains_around_periodic_edges(dims, pmask, storage, streaming):
    """Chains whose stencils cross the periodic edges and corners: compact ones,
    two of them overlapping across an edge, and one of bond 0.8 that spans the
    shortest periodic axis."""
    rng = np.random.default_rng(31)
    steps = 14
    bc = None if pmask == 7 else (oracle.BC_AFFINE, inputs.ou_strain(steps + 1, rng, corr_steps=20.0, rms=1e-3),
                                  0, 1, 0)
    near = [n - 0.7 if pmask >> a & 1 else (n - 1) / 2.0 for a, n in enumerate(dims)]
    far = [0.2 if pmask >> a & 1 else (n - 1) / 2.0 for a, n in enumerate(dims)]
    chains = []
    for beads, anchor, bond, k in ((7, near, CHAIN_BOND, 1.0), (5, far, CHAIN_BOND, 1.0), (9, near, 0.8, 0.003)):
        pos, vel = inputs.chain_init(beads, anchor, rng, bond=bond)
        if bond > 0.5:  # along the periodic axes only: the stencils stay off the walls
            free = [a for a in range(3) if not pmask >> a & 1]
            pos[:, free] = np.asarray(anchor)[free] + 0.05 * (pos[:, free] - np.asarray(anchor)[free])
        chains.append(dict(pos=pos, vel=vel, fene_k=k, anchor=anchor))
    case = Case(dims, collision=oracle.MRT, tau=0.8, periodic_mask=pmask, bc=bc,
                u0=1e-3 * rng.standard_normal(dims[::-1] + (3,)), chains=chains, reduce_every=7)
    run_case(case, storage, steps, f"wrapped chains {dims} {pmask} {streaming}",
             streaming=lbm.STREAM_AA if streaming == "in_place" else lbm.STREAM_AB)


@pytest.mark.parametrize("storage,tol", [("f64", 1e-13), ("f32", 1e-6), ("f16", 1e-5)])
@pytest.mark.parametrize("dims", [(40, 80, 96), (41, 79, 83)])
def test_check_record_of_many_row_ranges(dims, storage, tol):
    """Mass and momentum summed over more row ranges than a wavefront has lanes
    (16-byte chunks and node by node).  The bounds are those of the check
    records in test_gpu_parity and test_gpu_aa, relative to the mass."""
    rng = np.random.default_rng(37)
    case = Case(dims, collision=oracle.MRT, tau=0.7,
                bc=(oracle.BC_AFFINE, inputs.ou_strain(4, rng, corr_steps=20.0, rms=1e-4), 0, 1, 0),
                u0=1e-3 * rng.standard_normal(dims[::-1] + (3,)), reduce_every=2)
    say("case check record", dims, storage)
    ob = case.oracle_box()
    assert ob.step(2) == 0
    ctx = make_ctx(case, storage)
    ctx.step(2)
    mm_o, mm_g = ob.mass_mom(), ctx.read(0, lbm.F_MASS_MOM)
    say(mm_o, mm_g - mm_o)
    assert mm_g[0] == mm_o[0] == 2
    assert np.abs(mm_g[1:] - mm_o[1:]).max() < tol * mm_o[1]
    ctx.close()
