"""Routes of the step kernels at the sizes where they can go wrong, each against
the FP64 oracle within the bounds of test_gpu_parity: stencil boxes that wrap
around periodic axes."""
import hashlib

import numpy as np
import pytest

import oracle
from lbcase import CHAIN_BOND, Case, ks_case
from paper_0809_4958_amd import inputs
from test_gpu_extensions import accel_history
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


def walk(beads, anchor, rng, bond):
    pos, vel = inputs.chain_init(beads, anchor, rng, bond=bond)
    return dict(pos=pos, vel=vel, fene_k=1.0 if bond < 0.5 else 0.003, anchor=anchor)


@pytest.mark.parametrize("streaming", ["two_buffers", "in_place"])
@pytest.mark.parametrize("storage", ["f64", "f16"])
@pytest.mark.parametrize("beads,bond", [(1, CHAIN_BOND), (2, CHAIN_BOND), (9, 0.8), (64, 1.2), (65, CHAIN_BOND),
                                        (65, 1.2), (129, CHAIN_BOND), (256, 0.9)])
def test_chain_lengths_and_stencil_box_sizes(beads, bond, storage, streaming):
    """One bead to 256, around the 64 of a wavefront and the eight lanes of a
    bead, compact and stretched: stencil boxes inside and beyond the 1,024
    nodes whose force the chain pass tabulates, two chains overlapping."""
    rng = np.random.default_rng(41)
    steps, dims = 9, (34, 31, 33)
    A = inputs.ou_strain(steps + 1, rng, corr_steps=20.0, rms=1e-3)
    xc = [16.4, 15.2, 15.9]
    case = Case(dims, collision=oracle.MRT, tau=0.8, bc=(oracle.BC_AFFINE, A, 0, 1, 0),
                chains=[walk(beads, xc, rng, bond), walk(5, [17.1, 15.0, 16.3], rng, CHAIN_BOND)], reduce_every=3)
    if beads == 1:  # a pinned single bead has no size to compare positions with
        case.chains[0]["fix_com"] = False
    run_case(case, storage, steps, f"{beads} beads of bond {bond} {streaming}",
             streaming=lbm.STREAM_AA if streaming == "in_place" else lbm.STREAM_AB)


@pytest.mark.parametrize("beads", [12, 100])
def test_thermal_chain_lengths(beads):
    """Langevin noise, whose centre-of-mass sums stay inside the substeps, in
    one wavefront and over several."""
    rng = np.random.default_rng(43)
    steps, dims = 6, (18, 17, 19)
    A = inputs.ou_strain(steps + 1, rng, corr_steps=20.0, rms=1e-3)
    case = Case(dims, collision=oracle.MRT, tau=0.8, bc=(oracle.BC_AFFINE, A, 0, 1, 0), kT=1e-6, seed=77,
                chains=[walk(beads, [8.4, 8.1, 9.2], rng, CHAIN_BOND)])
    say("case thermal chain", beads)
    ob = case.oracle_box()
    assert ob.step(steps) == 0
    ctx = make_ctx(case, "f64")
    ctx.set_thermal(case.kT, case.seed)
    ctx.step(steps)
    check(compare(ctx, ob, case, "f64"), "f64", f"thermal chain of {beads}")
    ctx.close()


@pytest.mark.parametrize("beads", [40, 150])
def test_overstretched_bond_latches_at_the_oracles_step(beads):
    """Beads thrown apart: the bond reaches its maximum extension in the middle
    of a step; the error, its step and the state before it are the oracle's."""
    rng = np.random.default_rng(47)
    dims = (20, 20, 20)
    A = inputs.ou_strain(12, rng, corr_steps=20.0, rms=1e-3)
    chain = walk(beads, [9.5, 9.5, 9.5], rng, CHAIN_BOND)
    chain.update(zeta=0.1 / beads, fene_k=1e-6, vel=np.zeros((beads, 3)))
    chain["vel"][beads // 2:, 0] = 0.8
    case = Case(dims, collision=oracle.MRT, tau=0.8, bc=(oracle.BC_AFFINE, A, 0, 1, 0), chains=[chain])
    say("case overstretched bond", beads)
    ob = case.oracle_box()
    code = ob.step(10)
    assert code == -4 and 0 < ob.step_index < 10
    ctx = make_ctx(case, "f64")
    ctx.step(10)
    assert ctx.sync_status() == lbm.ERR_FENE
    assert ctx.read(0, lbm.F_STEP, strict=False)[0] == ob.step_index
    check(compare(ctx, ob, case, "f64", strict=False), "f64", "overstretched")
    ctx.close()


@pytest.mark.parametrize("streaming", ["two_buffers", "in_place"])
@pytest.mark.parametrize("storage", ["f32", "f16"])
@pytest.mark.parametrize("dims", [(3, 3, 3), (4, 5, 3), (5, 4, 6), (7, 9, 5), (8, 6, 7), (13, 12, 11), (33, 10, 6),
                                  (48, 7, 5), (63, 6, 9), (64, 5, 6), (65, 8, 5), (121, 9, 7), (130, 6, 5),
                                  (254, 5, 4), (263, 4, 5), (1030, 4, 4)])
def test_rows_of_any_length(dims, storage, streaming):
    """Rows that lane vectors divide and rows padded to them, shorter than a
    wavefront, longer, and cut by its edges at every place; two buffers (read
    in place, then pulled) and in place (both parities); two boxes, the second
    with its axes turned, and where one fits a chain next to a wall."""
    rng = np.random.default_rng(53)
    cases = []
    for k, d in enumerate((dims, (dims[1], dims[2], dims[0]))):
        A = inputs.ou_strain(10, rng, corr_steps=20.0, rms=1e-3 * 8 / max(d))
        chains = [walk(6, [2.6, 2.4, (d[2] - 1) / 2.0], rng, CHAIN_BOND)] if min(d) >= 5 else []
        cases.append(Case(d, collision=oracle.MRT, tau=0.8, bc=(oracle.BC_AFFINE, A, 0, 1, 0),
                          u0=1e-3 * rng.standard_normal(d[::-1] + (3,)), chains=chains, reduce_every=2))
    say("case rows", dims, storage, streaming)
    ctx = lbm.Context([c.dims for c in cases], collision=oracle.MRT, tau=0.8, storage=STORE[storage], reduce_every=2,
                      streaming=lbm.STREAM_AA if streaming == "in_place" else lbm.STREAM_AB)
    for k, c in enumerate(cases):
        c.add_to(ctx, k)
    obs = [c.oracle_box() for c in cases]
    for n in (1, 1, 3, 4):
        ctx.step(n)
        assert ctx.sync_status() == lbm.OK
        for k, c in enumerate(cases):
            assert obs[k].step(n) == 0
            check(compare(ctx, obs[k], c, storage, box=k), storage, f"rows {c.dims} {streaming}")
            mm_o, mm_g = obs[k].mass_mom(), ctx.read(k, lbm.F_MASS_MOM)
            if mm_o[0] > 0:
                assert mm_g[0] == mm_o[0]
                assert np.abs(mm_g[1:] - mm_o[1:]).max() < {"f32": 1e-6, "f16": 1e-5}[storage] * mm_o[1]
    ctx.close()


def test_reads_follow_every_step_and_write():
    """The device state is fetched once per step or write: reads in between, on
    the host and on the device, never see an older one."""
    import ctypes

    import torch

    rng = np.random.default_rng(59)
    dims = (12, 11, 13)
    A = inputs.ou_strain(20, rng, corr_steps=20.0, rms=1e-3)
    case = Case(dims, collision=oracle.MRT, tau=0.8, bc=(oracle.BC_AFFINE, A, 0, 1, 0),
                chains=[walk(5, [5.4, 5.1, 6.2], rng, CHAIN_BOND)])
    ob, ctx = case.oracle_box(), make_ctx(case, "f64", stream=torch.cuda.current_stream().cuda_stream)
    u_dev = torch.zeros(dims[::-1] + (3,), dtype=torch.float64, device="cuda")
    p_dev = torch.zeros((5, 3), dtype=torch.float64, device="cuda")
    assert ctx.read(0, lbm.F_STEP) == 0
    ctx.write_state(0, lbm.F_STEP, 4)
    assert ctx.read(0, lbm.F_STEP) == 4
    ctx.write_state(0, lbm.F_STEP, 0)
    for n in range(1, 6):
        ctx.step(1)
        assert ob.step(1) == 0
        for _ in range(2):
            assert ctx.read(0, lbm.F_STEP) == n
            for field, to in ((lbm.F_U, u_dev), (lbm.F_BEAD_POS, p_dev)):
                st = lbm.load().lb_read_fields(ctx._h, 0, field, ctypes.c_void_p(to.data_ptr()), to.numel() * 8, 1)
                assert st == lbm.OK
            assert np.array_equal(u_dev.cpu().numpy(), ctx.read(0, lbm.F_U))
            assert np.array_equal(p_dev.cpu().numpy(), ctx.read(0, lbm.F_BEAD_POS, n_beads=5))
        check(compare(ctx, ob, case, "f64"), "f64", f"step {n}")
    ctx.close()


@pytest.mark.parametrize("streaming", ["two_buffers", "in_place"])
@pytest.mark.parametrize("storage", ["f64", "f32", "f16"])
@pytest.mark.parametrize("kT,body", [(2e-6, True), (2e-6, False), (0.0, True), (0.0, False)])
def test_noise_and_body_force_of_a_box_that_was_thermal(kT, body, storage, streaming):
    """The step kernel follows the last temperature set and the boxes' body
    force: each of the four combinations, in a context that was made thermal
    at another temperature first."""
    steps = 24
    case = ks_case(21, steps, dt=10, res=9, tau=0.6, n_beads=8, f32_samples=storage != "f64")
    case.kT, case.seed = kT, 77
    if body:
        case.body = accel_history(steps, np.random.default_rng(3))
    say("case noise", kT, "body", body, storage, streaming)
    ob = case.oracle_box()
    assert ob.step(steps) == 0
    ctx = make_ctx(case, storage, streaming=lbm.STREAM_AA if streaming == "in_place" else lbm.STREAM_AB)
    ctx.set_thermal(1e-4, 5)
    ctx.set_thermal(kT, 77)
    ctx.step(steps)
    check(compare(ctx, ob, case, storage), storage, f"noise {kT} body {body} {streaming}")
    ctx.close()


@pytest.mark.parametrize("streaming", ["two_buffers", "in_place"])
def test_reads_follow_the_replays_of_a_captured_step(streaming):
    """A step captured on the context's stream and replayed by the caller: every
    readout is the state behind the last replay, on the host and on the device."""
    import ctypes

    import torch

    rng = np.random.default_rng(61)
    dims = (12, 11, 13)
    case = Case(dims, collision=oracle.MRT, tau=0.8,
                bc=(oracle.BC_AFFINE, inputs.ou_strain(20, rng, corr_steps=20.0, rms=1e-3), 0, 1, 0),
                u0=1e-3 * rng.standard_normal(dims[::-1] + (3,)), chains=[walk(5, [5.4, 5.1, 6.2], rng, CHAIN_BOND)])
    say("case captured step", streaming)
    stream = torch.cuda.Stream()
    ob = case.oracle_box()
    ctx = make_ctx(case, "f64", stream=stream.cuda_stream,
                   streaming=lbm.STREAM_AA if streaming == "in_place" else lbm.STREAM_AB)
    ctx.step(1)
    assert ob.step(1) == 0 and ctx.read(0, lbm.F_STEP) == 1
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        ctx.step(1)
    u = torch.zeros(dims[::-1] + (3,), dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    for n in range(2, 8):
        with torch.cuda.stream(stream):
            graph.replay()
        assert ob.step(1) == 0
        for _ in range(2):
            assert ctx.read(0, lbm.F_STEP) == n
            st = lbm.load().lb_read_fields(ctx._h, 0, lbm.F_U, ctypes.c_void_p(u.data_ptr()), u.numel() * 8, 1)
            assert st == lbm.OK and np.array_equal(u.cpu().numpy(), ctx.read(0, lbm.F_U))
        assert ctx.sync_status() == lbm.OK
        check(compare(ctx, ob, case, "f64"), "f64", f"replay {n - 1}")
    ctx.close()


def arena_bytes(dims, storage):
    """The populations of one buffer without padding."""
    return 19 * int(np.prod(dims)) * {"f64": 8, "f32": 4, "f16": 2}[storage]


@pytest.fixture
def torch_allocs(monkeypatch):
    """Sizes the contexts made with torch_alloc ask for; with `most` set, larger
    ones are refused as PyTorch refuses what it has no memory for."""
    import torch

    class Log:
        def __init__(self):
            self.sizes, self.most = [], None

    log, give = Log(), torch.cuda.caching_allocator_alloc

    def alloc(n, *a):
        log.sizes.append(n)
        if log.most is not None and n > log.most:
            raise torch.cuda.OutOfMemoryError("refused by the test")
        return give(n, *a)

    monkeypatch.setattr(torch.cuda, "caching_allocator_alloc", alloc)
    return log


@pytest.mark.parametrize("streaming", ["two_buffers", "in_place"])
@pytest.mark.parametrize("storage,dims", [("f16", (73, 10, 12)), ("f16", (9, 9, 11)), ("f16", (100, 7, 9)),
                                          ("f32", (65, 9, 10)), ("f32", (40, 6, 9))])
def test_context_fits_where_its_own_nodes_do(storage, dims, streaming, torch_allocs):
    """With memory for the boxes' own nodes alone (no padded row, in place no
    x-face velocity) a context is made all the same, and steps right."""
    rng = np.random.default_rng(67)
    case = Case(dims, collision=oracle.MRT, tau=0.8,
                bc=(oracle.BC_AFFINE, inputs.ou_strain(8, rng, corr_steps=20.0, rms=1e-3 * 8 / max(dims)), 0, 1, 0),
                u0=1e-3 * rng.standard_normal(dims[::-1] + (3,)), reduce_every=2,
                chains=[walk(5, [4.1, 3.6, 4.4], rng, CHAIN_BOND)] if min(dims) > 6 else [])
    say("case least memory", dims, storage, streaming)
    torch_allocs.most = arena_bytes(dims, storage)
    ob = case.oracle_box()
    ctx = make_ctx(case, storage, torch_alloc=True, streaming=lbm.STREAM_AA if streaming == "in_place" else lbm.STREAM_AB)
    torch_allocs.most = None  # the readouts below stage FP64 fields
    for n in (1, 2, 3):
        ctx.step(n)
        assert ctx.sync_status() == lbm.OK and ob.step(n) == 0
        check(compare(ctx, ob, case, storage), storage, f"least memory {dims} {streaming}")
    ctx.close()


@pytest.mark.parametrize("streaming", ["two_buffers", "in_place"])
@pytest.mark.parametrize("storage,dims", [("f16", (33, 9, 40)), ("f16", (1030, 4, 6)), ("f16", (9, 17, 9)),
                                          ("f16", (73, 41, 20)), ("f32", (65, 65, 9)), ("f32", (5, 11, 7))])
def test_padding_stays_within_its_bound(storage, dims, streaming, torch_allocs):
    """Half as many nodes again in x (short rows: up to 16) and a quarter in y."""
    nx, ny, nz = dims
    ctx = lbm.Context([dims], storage=STORE[storage], torch_alloc=True,
                      streaming=lbm.STREAM_AA if streaming == "in_place" else lbm.STREAM_AB)
    ctx.close()
    most = arena_bytes((max(16, 3 * nx // 2 + 8), ny + ny // 4, nz), storage)
    say("case padding", dims, storage, torch_allocs.sizes[0], "of", most)
    assert torch_allocs.sizes[0] <= most


@pytest.mark.parametrize("streaming,dims", [("two_buffers", (73, 3000, 3000)), ("in_place", (97, 4001, 4001))])
def test_large_contexts_are_not_padded(streaming, dims, torch_allocs):
    """Padding that adds more than 1/32 of the device's memory is not asked for
    (the allocations are recorded and refused)."""
    torch_allocs.most = 0
    with pytest.raises(lbm.LBError) as e:
        lbm.Context([dims], storage=lbm.STORE_F16DEV, torch_alloc=True,
                    streaming=lbm.STREAM_AA if streaming == "in_place" else lbm.STREAM_AB)
    assert e.value.status == lbm.ERR_OOM
    say("case unpadded", dims, max(torch_allocs.sizes))
    assert max(torch_allocs.sizes) == arena_bytes(dims, "f16")


@pytest.mark.parametrize("streaming", ["two_buffers", "in_place"])
@pytest.mark.parametrize("storage,pmask", [("f64", 0), ("f16", 0), ("f32", 7)])
def test_chains_step_without_a_force_table(storage, pmask, streaming, torch_allocs):
    """The chains' force table (24 KiB each) is an allocation that can be done
    without: the force is gathered from the beads, k_chain writes no table."""
    rng = np.random.default_rng(71)
    dims, steps = (16, 15, 17), 6
    bc = None if pmask else (oracle.BC_AFFINE, inputs.ou_strain(steps + 1, rng, corr_steps=20.0, rms=1e-3), 0, 1, 0)
    case = Case(dims, collision=oracle.MRT, tau=0.8, periodic_mask=pmask, bc=bc,
                u0=1e-3 * rng.standard_normal(dims[::-1] + (3,)),
                chains=[walk(b, [7.4, 7.1, 8.2], rng, CHAIN_BOND) for b in (5, 9, 70)])
    say("case no force table", storage, pmask, streaming)
    ob = case.oracle_box()
    assert ob.step(steps) == 0
    ctx = make_ctx(case, storage, torch_alloc=True, streaming=lbm.STREAM_AA if streaming == "in_place" else lbm.STREAM_AB)
    torch_allocs.most = 3 * 24576 - 1
    ctx.step(steps)
    assert ctx.sync_status() == lbm.OK and max(torch_allocs.sizes[-12:]) >= 3 * 24576
    torch_allocs.most = None
    check(compare(ctx, ob, case, storage), storage, f"no force table {streaming}")
    ctx.close()


@pytest.mark.parametrize("target", ["device", "device, odd address", "pinned host"])
def test_bead_readouts_reach_every_target_a_copy_does(target):
    """Bead readouts into memory given as the device's: this device's (written by
    the kernel) and the rest (staged and copied; another device's is one of them)."""
    import ctypes

    import torch

    rng = np.random.default_rng(73)
    case = Case((12, 12, 12), bc=(oracle.BC_AFFINE, inputs.ou_strain(4, rng, corr_steps=20.0, rms=1e-3), 0, 1, 0),
                chains=[walk(7, [5.4, 5.1, 6.2], rng, CHAIN_BOND)])
    say("case bead target", target)
    ctx = make_ctx(case, "f64")
    ctx.step(2)
    n = 7 * 3 * 8
    buf = torch.zeros(n + 8, dtype=torch.uint8, device="cuda" if "device" in target else "cpu",
                      pin_memory=target.startswith("pinned"))
    off = 1 if "odd" in target else 0
    for field in (lbm.F_BEAD_POS, lbm.F_BEAD_VEL, lbm.F_BEAD_REL):
        st = lbm.load().lb_read_fields(ctx._h, 0, field, ctypes.c_void_p(buf.data_ptr() + off), n, 1)
        assert st == lbm.OK, ctx.last_error()
        assert buf[off:off + n].cpu().numpy().tobytes() == ctx.read(0, field, n_beads=7).tobytes()
    ctx.close()


# First 16 hex digits of the SHA-256 of the populations behind each step.
PLAIN_STEP_BITS = {
    ("f32", "mrt"): ["dac02b90f3528f46", "d41e2e064b3108dd", "f476958486f8cfe0"],
    ("f32", "bgk"): ["2e0bc38bb79ead1d", "eb74b4b2e3d732a8", "e5c62ad05582ef26"],
    ("f16", "mrt"): ["47a80750daeb32e6", "20d5697b8ee77a54", "164d81fa9889261f"],
    ("f16", "bgk"): ["53fd99d6c4679fd6", "2c6ad08155da820c", "6c54f521cb7cbe9e"],
}


def plain_step_bits(storage, collision):
    rng = np.random.default_rng(79)
    dims = (40, 36, 44)
    case = Case(dims, collision=collision, tau=0.6,
                bc=(oracle.BC_AFFINE, inputs.ou_strain(8, rng, corr_steps=20.0, rms=1e-4), 0, 1, 0),
                u0=1e-3 * rng.standard_normal(dims[::-1] + (3,)))
    ctx = make_ctx(case, storage)
    bits = []
    for _ in range(3):
        ctx.step(1)
        bits.append(hashlib.sha256(np.ascontiguousarray(ctx.read(0, lbm.F_POP_DEV)).tobytes()).hexdigest()[:16])
    ctx.close()
    return bits


@pytest.mark.parametrize("storage,collision", [("f32", "mrt"), ("f16", "mrt"), ("f32", "bgk"), ("f16", "bgk")])
def test_plain_step_rounds_as_before(storage, collision):
    """The plain step's rounding is part of its results: FP16 storage turns a last
    bit into another half-precision value now and then, and a long run into
    another, equally accurate one.  A change to the extended collisions (body
    force, noise) leaves it alone."""
    say("case plain step bits", storage, collision)
    assert plain_step_bits(storage, {"mrt": oracle.MRT, "bgk": oracle.BGK}[collision]) == PLAIN_STEP_BITS[storage, collision]


@pytest.mark.parametrize("storage", ["f64", "f16"])
@pytest.mark.parametrize("nch,pmask,dims", [(1, 7, (20, 18, 22)), (3, 7, (17, 19, 21)), (2, 5, (26, 13, 24)),
                                            (40, 7, (16, 15, 17))])
def test_chains_stretched_over_a_periodic_box(nch, pmask, dims, storage):
    """Stencil boxes of thousands of nodes, shared by several workgroups of the
    force pass: beads on a line along the periodic axes, beside compact chains that
    need one; steps with and without a check pass, graph replays."""
    rng = np.random.default_rng(83)
    steps = 11
    bc = None if pmask == 7 else (oracle.BC_AFFINE, inputs.ou_strain(steps + 1, rng, corr_steps=20.0, rms=1e-4),
                                  0, 1, 0)
    chains = []
    for k in range(nch):
        # a line over the periodic axes, or a compact walk somewhere in the box
        line, free = k % 8 == 0, [pmask >> a & 1 for a in range(3)]
        mid = np.array([rng.uniform(0, n) if f and k else (n - 1) / 2.0 for n, f in zip(dims, free)])
        beads = 40 if line else 6
        if line:
            span = np.array([n - 1.5 if f else 2.0 for n, f in zip(dims, free)])
            pos = ((np.arange(beads)[:, None] + 0.5) / beads - 0.5) * span + mid
        else:
            pos = walk(beads, mid, rng, CHAIN_BOND)["pos"]
        chains.append(dict(pos=pos, vel=np.zeros((beads, 3)), fene_k=1e-4, anchor=list(mid)))
    case = Case(dims, collision=oracle.MRT, tau=0.8, periodic_mask=pmask, bc=bc,
                u0=1e-3 * rng.standard_normal(dims[::-1] + (3,)), chains=chains, reduce_every=4)
    say("case stretched", nch, pmask, dims, storage)
    ob = NearestImage(case)
    ctx = make_ctx(case, storage, graph_steps=4)
    for n in (1, 2, 8):
        ctx.step(n)
        assert ob.step(n) == 0 and ctx.sync_status() == lbm.OK
        assert ctx.read(0, lbm.F_STEP) == ob.step_index
    check(compare(ctx, ob, case, storage), storage, f"stretched {nch} {dims}")
    ctx.close()


@pytest.mark.parametrize("storage", ["f32", "f16"])
def test_autotuning_keeps_the_shape_that_fills_the_chip(storage, tmp_path):
    """A 32^3 box starts with items of one workgroup iteration; two are 40 % slower
    (8 and 11 us), so tuning keeps what it began with, and so does the cache."""
    cache = str(tmp_path / "tune.jsonl")

    def make():
        ctx = lbm.Context([(32, 32, 32)], collision=oracle.MRT, tau=0.6, storage=STORE[storage], tune_cache=cache)
        ctx.set_boundary(0, lbm.BC_AFFINE, np.zeros((2, 9)), t0=0, dt=1000)
        ctx.step(1)
        ctx.sync()
        return ctx, ctx.describe()

    ctx, start = make()
    ctx.autotune(7)
    say("case autotune", storage, start, "->", ctx.describe())
    assert "->30x17x1" in start and ctx.describe() == start
    ctx.close()
    ctx, again = make()
    assert again == start
    ctx.close()


def tune_line(storage, dims, shape, periodic=0, vw=None):
    """A line of an autotuner cache: the item shape of an MRT box."""
    import json

    d = dict(key=f"S{STORE[storage]}C1_{dims[0]}x{dims[1]}x{dims[2]}p{periodic}", ex=shape[0], ey=shape[1], ez=shape[2])
    return json.dumps(d if vw is None else dict(d, vw=vw)) + "\n"


@pytest.mark.parametrize("vw,taken", [(0, False), (None, False), (2, True)])
def test_tile_shapes_of_older_caches_are_not_row_shapes(vw, taken, tmp_path):
    """An autotuner cache from when a 121-node row ran as tiles: its 16 planes per
    item do not become 16 iterations of a row item."""
    cache, dims = tmp_path / "tune.jsonl", (121, 24, 25)

    def shape(path):
        ctx = lbm.Context([dims], collision=oracle.MRT, tau=0.6, storage=lbm.STORE_F32, tune_cache=path)
        ctx.set_boundary(0, lbm.BC_AFFINE, np.zeros((2, 9)), t0=0, dt=1000)
        ctx.step(1)
        d = ctx.describe().split("->")[-1]
        ctx.close()
        return d

    cache.write_text(tune_line("f32", dims, (64, 4, 16), vw=vw))
    say("case old cache", vw, shape(None), shape(str(cache)))
    assert (shape(str(cache)) == "64x4x16") if taken else (shape(str(cache)) == shape(None))


SHAPES = [  # dims, periodic axes, items of one iteration each, items of several
    ("tiles", (34, 30, 25), 0, (16, 8, 1), (32, 20, 7)),
    ("tiles", (23, 37, 18), 0, (21, 1, 1), (21, 35, 16)),
    ("tiles", (48, 20, 19), 7, (16, 4, 1), (48, 20, 6)),
    ("tiles", (19, 33, 14), 5, (19, 1, 1), (19, 31, 14)),
    ("rows", (150, 21, 22), 0, (64, 8, 1), (64, 8, 2)),
    ("rows", (150, 21, 22), 0, (64, 8, 1), (64, 8, 4)),
    ("rows", (95, 25, 23), 0, (93, 5, 1), (93, 5, 3)),
    ("rows", (61, 40, 24), 0, (59, 8, 1), (59, 8, 3)),
    ("rows", (64, 33, 20), 0, (62, 8, 1), (62, 8, 4)),
]


@pytest.mark.parametrize("streaming", ["two_buffers", "in_place"])
@pytest.mark.parametrize("storage,kind,dims,pmask,small,large", [
    (st,) + s for s in SHAPES for st in ("f64", "f32", "f16") if s[0] == "tiles" or st != "f64"])  # FP64 has no rows
def test_item_shape_does_not_change_a_bit(storage, kind, dims, pmask, small, large, streaming, tmp_path, monkeypatch):
    """Items of several planes, positions per thread or workgroup iterations (the
    shapes of large contexts, fixed here through the autotuner cache) give the
    bits of items that take one pass through every loop, as the small boxes of the
    parity tests do; a chain meets some of the iterations of an item."""
    if kind == "tiles":
        monkeypatch.setenv("LBM_NO_VEC", "1")
    rng = np.random.default_rng(89)
    bc = None if pmask == 7 else (oracle.BC_AFFINE, inputs.ou_strain(8, rng, corr_steps=20.0, rms=1e-3 * 8 / max(dims)),
                                  0, 1, 0)
    case = Case(dims, collision=oracle.MRT, tau=0.8, periodic_mask=pmask, bc=bc,
                u0=1e-3 * rng.standard_normal(dims[::-1] + (3,)), reduce_every=3,
                chains=[walk(9, [(n - 1) / 2.0 for n in dims], rng, CHAIN_BOND),
                        walk(5, [4.3, 5.1, 3.7], rng, CHAIN_BOND)])
    mode = lbm.STREAM_AA if streaming == "in_place" else lbm.STREAM_AB
    say("case item shapes", kind, dims, pmask, small, large, storage, streaming)
    ctxs = []
    for k, shape in enumerate((small, large)):
        cache = tmp_path / f"tune{k}.jsonl"
        cache.write_text(tune_line(storage, dims, shape, periodic=pmask, vw=2 if kind == "rows" else 0))
        ctxs.append(make_ctx(case, storage, streaming=mode, tune_cache=str(cache)))
    for n in (1, 4, 1):
        out = []
        for ctx, shape in zip(ctxs, (small, large)):
            ctx.step(n)
            assert ctx.sync_status() == lbm.OK
            assert ctx.describe().endswith("->%dx%dx%d" % shape)
            out.append([ctx.read(0, lbm.F_POP_DEV), ctx.read(0, lbm.F_BEAD_POS, n_beads=14),
                        ctx.read(0, lbm.F_MASS_MOM)])
        assert all(np.array_equal(a, b) for a, b in zip(*out))
    for ctx in ctxs:
        ctx.close()


@pytest.mark.parametrize("streaming", ["two_buffers", "in_place"])
@pytest.mark.parametrize("storage,dims", [("f16", (41, 6, 7)), ("f16", (47, 9, 5)), ("f16", (73, 5, 9)), ("f16", (95, 7, 5)),
                                          ("f16", (161, 4, 5)), ("f16", (191, 5, 4)), ("f32", (37, 6, 7)),
                                          ("f32", (47, 5, 9)), ("f32", (81, 9, 5)), ("f32", (95, 5, 6)),
                                          ("f32", (177, 4, 5)), ("f32", (191, 5, 4))])
def test_padded_rows_of_three_word_vectors(dims, storage, streaming):
    """Row lengths padded to whole vectors of three words, the last node in each
    place of its vector."""
    test_rows_of_any_length(dims, storage, streaming)


@pytest.mark.parametrize("items", ["tiles", "rows"])
@pytest.mark.parametrize("storage", ["f32", "f16"])
def test_in_place_equals_two_buffers(storage, items, monkeypatch):
    """In-place tile and row items against the two-buffer tiles: FP16 bit for bit,
    FP32 to the 8 units in the last place of test_gpu_aa."""
    cases = [ks_case(n, 40, dt=20, res=9, n_beads=6, config_idx=2, box_idx=i) for i, n in enumerate([20, 27])]
    say("case in place", items, "vs two-buffer tiles", storage)
    ctxs = []
    for mode, tiles in ((lbm.STREAM_AA, items == "tiles"), (lbm.STREAM_AB, True)):
        monkeypatch.setenv("LBM_NO_VEC", "1") if tiles else monkeypatch.delenv("LBM_NO_VEC", raising=False)
        ctx = lbm.Context([c.dims for c in cases], collision=cases[0].collision, tau=cases[0].tau,
                          storage=STORE[storage], streaming=mode)
        for k, c in enumerate(cases):
            c.add_to(ctx, k)
        ctxs.append(ctx)
    for n in (13, 14):  # odd, then even step counts
        for ctx in ctxs:
            ctx.step(n)
        for k in range(len(cases)):
            pa, pb = (c.read(k, lbm.F_POP_DEV) for c in ctxs)
            if storage == "f16":
                assert np.array_equal(pa, pb), (n, k)
            else:
                assert np.abs(pa - pb).max() <= 8 * np.spacing(np.float32(np.abs(pb).max())), (n, k)
    for ctx in ctxs:
        ctx.close()


@pytest.mark.parametrize("boxes,iterations", [(1, 1), (16, 1), (32, 3), (64, 4)])
def test_iterations_of_half_precision_row_items(boxes, iterations):
    """Items of FP16 row boxes by the size of the context: 32 boxes of 64^3 in
    single iterations took 156 us a step, in threes 137, and 16 boxes do not gain."""
    ctx = lbm.Context([(64, 64, 64)] * boxes, collision=oracle.MRT, tau=0.6, storage=lbm.STORE_F16DEV)
    for b in range(boxes):
        ctx.set_boundary(b, lbm.BC_AFFINE, np.zeros((2, 9)), t0=0, dt=1000)
    ctx.step(1)
    ctx.sync()
    assert ctx.describe().endswith(f"->62x8x{iterations}")
    ctx.close()


@pytest.mark.parametrize("storage,nx,streaming,padded", [
    ("f16", 42, lbm.STREAM_AB, False), ("f16", 42, lbm.STREAM_AA, True), ("f32", 21, lbm.STREAM_AB, True),
    ("f32", 21, lbm.STREAM_AA, True), ("f16", 68, lbm.STREAM_AB, False), ("f16", 52, lbm.STREAM_AB, True),
    ("f16", 121, lbm.STREAM_AB, True), ("f32", 65, lbm.STREAM_AB, True)])
def test_rows_are_padded_where_that_is_faster(storage, nx, streaming, padded, torch_allocs):
    """Rows that a vector divides keep their length where the padded pitch stores
    more than its alignment saves (42 FP16 nodes on two buffers in 48: 7 % slower;
    in place 42 is a quarter slower)."""
    dims = (nx, 16, 9)
    ctx = lbm.Context([dims], storage=STORE[storage], streaming=streaming, torch_alloc=True)
    ctx.close()
    say("case pitch", storage, nx, streaming, torch_allocs.sizes[0], arena_bytes(dims, storage))
    assert (torch_allocs.sizes[0] > arena_bytes(dims, storage)) == padded


@pytest.mark.parametrize("storage,tol", [("f64", 1e-13), ("f32", 1e-6), ("f16", 1e-5)])
@pytest.mark.parametrize("dims", [(12, 31, 40), (44, 30, 26), (206, 70, 130), (42, 11, 13), (66, 9, 8), (68, 7, 9),
                                  (34, 8, 11), (21, 12, 10)])
def test_check_record_of_short_chunks_and_capped_ranges(dims, storage, tol):
    """Rows of whole four- and two-node chunks but not eight, single nodes, and a
    box whose row ranges are capped, against the sums of the oracle's populations in extended
    precision (its own running sum of 34 million terms is 1.2e-13 off them)."""
    rng = np.random.default_rng(37)
    case = Case(dims, collision=oracle.MRT, tau=0.7,
                bc=(oracle.BC_AFFINE, inputs.ou_strain(4, rng, corr_steps=20.0, rms=1e-4), 0, 1, 0),
                u0=1e-3 * rng.standard_normal(dims[::-1] + (3,)), reduce_every=2)
    say("case check record", dims, storage)
    ob = case.oracle_box()
    assert ob.step(2) == 0
    f = ob.pop()[:, 1:-1, 1:-1, 1:-1].astype(np.longdouble).sum(axis=(1, 2, 3))
    exact = np.array([f.sum()] + [f[1 + 2 * a] - f[2 + 2 * a] + sum(
        c[a] * f[7 + k] for k, c in enumerate(DIAGONALS)) for a in range(3)], dtype=float)
    ctx = make_ctx(case, storage)
    ctx.step(2)
    mm = ctx.read(0, lbm.F_MASS_MOM)
    say(exact, mm[1:] - exact)
    assert mm[0] == 2 and np.abs(mm[1:] - exact).max() < tol * exact[0]
    ctx.close()


DIAGONALS = [(1, 1, 0), (-1, -1, 0), (1, -1, 0), (-1, 1, 0), (1, 0, 1), (-1, 0, -1), (1, 0, -1), (-1, 0, 1), (0, 1, 1),
             (0, -1, -1), (0, 1, -1), (0, -1, 1)]  # directions 7 to 18
