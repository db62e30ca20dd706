"""GPU parity of the fast mobility product (ARB_PAIR_FMM).

Two oracles: the plain sum over cell pairs of the same interpolation
approximation (oracle/fastsum.py), which the GPU must reproduce to FP32
rounding (1e-5 of the largest entry), and the dense RPY sum (oracle/rpy.py),
which it must approach within the approximation's error, falling with the
order.  Inputs: loose blobs in slabs above the wall and in free space, ragged
leaves, explicit and automatic leaf levels, the degenerate trees (one cell,
coincident blobs, a single blob)."""
import numpy as np
import pytest

from oracle import bodies, fastsum, rpy, rpy_rot, single_blob, system
from paper_2107_10800_amd import arb
from paper_2107_10800_amd import workloads as W

pytestmark = pytest.mark.gpu


def blobs(N, box, seed, z0=1.5):
    rng = np.random.default_rng(seed)
    pos = rng.uniform(0, 1, (N, 3)) * np.array(box, float)
    pos[:, 2] += z0
    return pos, rng.standard_normal((N, 3))


def fmm(pos, lam, wall, n, L, a=1.0, eta=1.0, leaf=0, precision=arb.ARB_FP64):
    ctx = arb.arb_create(wall=wall, a=a, eta=eta, pair_kernel=arb.ARB_PAIR_FMM, fmm_order=n,
                         fmm_levels=L, fmm_leaf=leaf, precision=precision)
    try:
        return arb.arb_rpy_apply(ctx, pos, lam).reshape(-1, 3)
    finally:
        arb.arb_destroy(ctx)


# (N, box, wall, n, L): cells hold more blobs than proxies (n^3) on average, so
# that both interpolations are exercised next to the sparse-cell paths
CASES = [
    (2400, (48, 48, 10), False, 4, 2),
    (1501, (48, 48, 10), False, 3, 2),
    (2401, (48, 48, 10), False, 5, 2),
    (1100, (48, 48, 10), True, 4, 2),
    (700, (30, 60, 8), True, 3, 2),
]


@pytest.mark.parametrize("N,box,wall,n,L", CASES)
def test_matches_the_oracle_of_the_approximation(N, box, wall, n, L):
    pos, lam = blobs(N, box, 100 + N)
    a, eta = 0.9, 1.3
    pos *= a
    print(f"fmm vs oracle approximation: N={N} wall={wall} n={n} L={L}", flush=True)
    ref = fastsum.fmm_apply(pos, lam, a, eta, wall, n, L)
    dense = rpy.mobility_apply(pos, lam, a, eta, wall)
    approx = np.abs(ref - dense).max() / np.abs(dense).max()
    for prec in (arb.ARB_FP64, arb.ARB_FP32C):     # double and float sums
        u = fmm(pos, lam, wall, n, L, a, eta, precision=prec)
        err = np.abs(u - ref).max() / np.abs(ref).max()
        print(f"  precision {prec}: GPU vs approximation {err:.1e}; approximation vs dense "
              f"{approx:.1e}", flush=True)
        assert err <= 1e-5
        assert approx > 10 * err          # the comparison resolves the approximation


# (N, wall, n, L): M2L's batches at the edges of their tiles: one 16-proxy tile partly
# filled (n = 2: 8 proxies, n = 3: 27), full ones (n = 4: 64), a last tile of 8 (n = 6)
# and of 7 (n = 7) proxies; batches of 1 to 32 columns (16 with torques), and blobs
# crowded towards one side so that dense and sparse listed cells occur side by side
@pytest.mark.parametrize("N,wall,n,L", [(260, False, 2, 3), (300, True, 2, 3), (900, False, 3, 3),
                                        (1500, True, 4, 2), (6000, False, 6, 2),
                                        (3500, True, 6, 2), (5000, False, 7, 2)])
def test_m2l_batches_against_the_oracle(N, wall, n, L):
    rng = np.random.default_rng(N + n)
    pos = rng.uniform(0, 1, (N, 3))
    pos[:, 0] **= 2
    pos = pos * np.array([60.0, 60.0, 15.0]) + np.array([0, 0, 1.5])
    lam = rng.standard_normal((N, 3))
    ref = fastsum.fmm_apply(pos, lam, 1.0, 1.0, wall, n, L)
    for prec in (arb.ARB_FP64, arb.ARB_FP32C):
        err = np.abs(fmm(pos, lam, wall, n, L, precision=prec) - ref).max() / np.abs(ref).max()
        print(f"m2l batches N={N} wall={wall} n={n} L={L} precision {prec}: {err:.1e}", flush=True)
        assert err <= 1e-5
    if wall or n > 4:
        return
    F = rng.standard_normal((N, 6))
    wl = W.Workload("loose", 1.0, 1.0, False, np.zeros((N, 3)), np.arange(N + 1, dtype=np.int32),
                    pos, np.tile([1.0, 0, 0, 0], (N, 1)), F, extra=dict(single_blob=True))
    ref = fastsum.fmm_apply(pos, F, 1.0, 1.0, False, n, L, kernel=rot_kernel(1.0, 1.0))
    for prec in (arb.ARB_FP64, arb.ARB_FP32C):
        ctx = arb.context_for(wl, precision=prec, pair_kernel=arb.ARB_PAIR_FMM, fmm_order=n,
                              fmm_levels=L)
        try:
            uw = arb.arb_body_mobility_apply(ctx, F)
        finally:
            arb.arb_destroy(ctx)
        assert np.abs(uw - ref).max() <= 1e-5 * np.abs(ref).max()


def leaves_of(counts, rng):
    """counts[i] blobs in cell i of a row of 8 x 1 x 1 cells of side 10 (leaf level 3 of a
    cube of side 80); the corner blobs span the cube."""
    pos = [np.array([[0.0, 0.0, 2.0], [80.0, 80.0, 82.0]])]
    for i, m in enumerate(counts):
        pos.append(rng.uniform(0.2, 9.8, (m, 3)) + np.array([10.0 * i, 0.0, 2.0]))
    return np.vstack(pos)


# the near field's blocks at the edges of their tiles: leaves of 1 to 257 blobs side by
# side (targets and source tiles of 1, 63, 64, 65, 128, 129 and 257), every leaf level
# including the direct sum of a single leaf
@pytest.mark.parametrize("L", [0, 3])
@pytest.mark.parametrize("wall", [False, True])
def test_near_field_blocks_at_their_edges(wall, L):
    rng = np.random.default_rng(21 + L)
    pos = leaves_of([1, 63, 64, 65, 257, 128, 129, 2], rng)
    lam = rng.standard_normal((len(pos), 3))
    ref = fastsum.fmm_apply(pos, lam, 1.0, 1.0, wall, 2, L) if L else \
        rpy.mobility_apply(pos, lam, 1.0, 1.0, wall)
    for prec in (arb.ARB_FP64, arb.ARB_FP32C):
        u = [fmm(pos, lam, wall, 2, L or 1, precision=prec) for _ in range(2)]
        assert np.array_equal(u[0], u[1])
        assert np.abs(u[0] - ref).max() <= 1e-5 * np.abs(ref).max()


# leaves too small for a wavefront's 64 steps both ways are summed one way, fuller ones both
# ways, by the tree's steps in all (a row of nearly empty leaves, of leaves just below and
# just above half a tile, of full tiles, and mixed); orders 2 to 4 also join the sums of
# many groups of lanes in M2L's sparse part
@pytest.mark.parametrize("counts", [[1, 7, 30, 2, 5, 3, 64, 20], [39] * 8, [41] * 8, [64] * 8,
                                    [3, 3, 300, 300, 3, 3, 2, 1]])
@pytest.mark.parametrize("n,wall", [(2, True), (3, False), (4, True)])
def test_near_field_one_way_and_both_ways(counts, n, wall):
    rng = np.random.default_rng(33 + n)
    pos = leaves_of(counts, rng)
    lam = rng.standard_normal((len(pos), 3))
    ref = fastsum.fmm_apply(pos, lam, 1.0, 1.0, wall, n, 3)
    for prec in (arb.ARB_FP64, arb.ARB_FP32C):
        u = [fmm(pos, lam, wall, n, 3, precision=prec) for _ in range(2)]
        assert np.array_equal(u[0], u[1])
        assert np.abs(u[0] - ref).max() <= 1e-5 * np.abs(ref).max()


# order 2: every listed cell of M2L strung together, cells of at most 7 blobs with those,
# the others with their 8 proxies; lists of more than a wavefront's 64 entries (in space)
# and of a few (a row of cells), both channels
@pytest.mark.parametrize("N,box,wall,L", [(4000, (60, 60, 60), False, 3), (900, (40, 40, 40), True, 3),
                                          (700, (200, 6, 6), True, 4)])
def test_strung_lists_of_order_two(N, box, wall, L):
    rng = np.random.default_rng(N)
    pos = rng.uniform(0, 1, (N, 3))
    pos[:, 0] **= 2
    pos = pos * np.array(box, float) + np.array([0, 0, 1.5])
    F = rng.standard_normal((N, 6))
    ref = fastsum.fmm_apply(pos, F[:, :3], 1.0, 1.0, wall, 2, L)
    ref6 = fastsum.fmm_apply(pos, F, 1.0, 1.0, False, 2, L, kernel=rot_kernel(1.0, 1.0))
    wl = W.Workload("loose", 1.0, 1.0, False, np.zeros((N, 3)), np.arange(N + 1, dtype=np.int32),
                    pos, np.tile([1.0, 0, 0, 0], (N, 1)), F, extra=dict(single_blob=True))
    for prec in (arb.ARB_FP64, arb.ARB_FP32C):
        u = [fmm(pos, F[:, :3], wall, 2, L, precision=prec) for _ in range(2)]
        assert np.array_equal(u[0], u[1])
        assert np.abs(u[0] - ref).max() <= 1e-5 * np.abs(ref).max()
        ctx = arb.context_for(wl, precision=prec, pair_kernel=arb.ARB_PAIR_FMM, fmm_order=2,
                              fmm_levels=L)
        try:
            uw = arb.arb_body_mobility_apply(ctx, F)
        finally:
            arb.arb_destroy(ctx)
        assert np.abs(uw - ref6).max() <= 1e-5 * np.abs(ref6).max()


def test_near_field_without_room_for_its_slots():
    """The near field's slots are optional memory (2.9 GB here: 260,000 blobs in 64
    leaves): with less than that left on the device, everything else (under 0.1 GB)
    fitting, the product sums the near field one way.  The tensor's floats are the same
    for both directions and the sums double, over 64,000 near blobs per blob: rounding
    at most 64,000 x 2^-53 of the sum of the magnitudes, a few hundred times the
    largest velocity."""
    import torch

    rng = np.random.default_rng(8)
    N, left = 260000, 2 << 30
    pos, lam = rng.uniform(0, 200.0, (N, 3)), rng.standard_normal((N, 3))
    u = fmm(pos, lam, False, 4, 2)
    filler = []
    try:
        while True:
            torch.cuda.empty_cache()
            room = torch.cuda.mem_get_info()[0] - left
            if room < 64 << 20:
                break
            filler.append(torch.empty(min(room, 16 << 30), dtype=torch.uint8, device="cuda"))
        free = torch.cuda.mem_get_info()[0]
        print(f"free on the device: {free / 2 ** 30:.2f} GiB", flush=True)
        assert free < 5 * left // 4
        v = fmm(pos, lam, False, 4, 2)
    finally:
        filler.clear()
        torch.cuda.empty_cache()
    assert np.abs(u - v).max() <= 1e-9 * np.abs(u).max()


def test_products_share_a_tree_with_torques():
    """The translational product of single-blob bodies runs on the tree of the
    generalised one (no slots: the near field one way), before and after it."""
    rng = np.random.default_rng(5)
    pos = leaves_of([65, 40, 64, 3, 0, 70, 129, 20], rng)
    M = len(pos)
    F = rng.standard_normal((M, 6))
    wl = W.Workload("loose", 1.0, 1.0, False, np.zeros((M, 3)), np.arange(M + 1, dtype=np.int32),
                    pos, np.tile([1.0, 0, 0, 0], (M, 1)), F, extra=dict(single_blob=True))
    ref3 = fastsum.fmm_apply(pos, F[:, :3], 1.0, 1.0, False, 2, 3)
    ref6 = fastsum.fmm_apply(pos, F, 1.0, 1.0, False, 2, 3, kernel=rot_kernel(1.0, 1.0))
    for prec in (arb.ARB_FP64, arb.ARB_FP32C):
        ctx = arb.context_for(wl, precision=prec, pair_kernel=arb.ARB_PAIR_FMM, fmm_order=2,
                              fmm_levels=3)
        try:
            first = arb.arb_mobility_apply(ctx, F[:, :3]).reshape(-1, 3)
            uw = arb.arb_body_mobility_apply(ctx, F)
            after = arb.arb_mobility_apply(ctx, F[:, :3]).reshape(-1, 3)
        finally:
            arb.arb_destroy(ctx)
        for u in (first, after):
            assert np.abs(u - ref3).max() <= 1e-5 * np.abs(ref3).max()
        assert np.abs(uw - ref6).max() <= 1e-5 * np.abs(ref6).max()


@pytest.mark.parametrize("wall", [False, True])
def test_direct_sum_when_no_level_separates(wall):
    """fmm_levels = 1, a cluster narrower than 8a (no level with side >= 2a
    below the root), a single blob and coincident blobs: the direct sum."""
    pos, lam = blobs(300, (30, 30, 10), 7)
    for L in (1,):
        u = fmm(pos, lam, wall, 4, L)
        ref = rpy.mobility_apply(pos, lam, 1.0, 1.0, wall)
        assert np.abs(u - ref).max() <= 1e-5 * np.abs(ref).max()
    small, lam2 = blobs(50, (5, 5, 3), 8)
    small[1] = small[0]
    u = fmm(small, lam2, wall, 6, 0)
    ref = rpy.mobility_apply(small, lam2, 1.0, 1.0, wall)
    assert np.abs(u - ref).max() <= 1e-5 * np.abs(ref).max()
    one = np.array([[3.0, 4.0, 5.0]])
    u = fmm(one, lam2[:1], wall, 4, 0)
    ref = rpy.mobility_apply(one, lam2[:1], 1.0, 1.0, wall)
    assert np.abs(u - ref).max() <= 1e-6 * np.abs(ref).max()


@pytest.mark.parametrize("wall", [False, True])
def test_error_against_dense_falls_with_order(wall):
    """The slab of the headline product (16,384 blobs, 400a x 400a x
    [1.5a, 20a]), automatic leaf level: 48 sampled rows of the dense oracle."""
    sl = W.slab()
    pos, lam = sl["pos"], sl["lam"]
    rows = np.random.default_rng(4).choice(len(pos), 48, replace=False)
    ref = rpy.mobility_apply(pos, lam, 1.0, 1.0, wall, targets=rows)
    errs = []
    for n in (3, 4, 5, 6):
        u = fmm(pos, lam, wall, n, 0)
        errs.append(np.abs(u[rows] - ref).max() / np.abs(ref).max())
    print(f"slab wall={wall}: sampled max error by order 3..6:", ["%.1e" % e for e in errs],
          flush=True)
    assert all(b < a for a, b in zip(errs, errs[1:]))
    assert errs[-1] <= 2e-4


def test_every_order_at_four_levels():
    """Orders 2..8 on the slab above the wall with the leaf level fixed at 4,
    so that M2M (levels 3, 2) and L2L (levels 3, 4), which are specialised to
    the order, run at every order: sampled dense rows, the error falling with
    the order (3e-2 at order 2 to about 1e-6 at order 8)."""
    sl = W.slab()
    pos, lam = sl["pos"], sl["lam"]
    rows = np.random.default_rng(5).choice(len(pos), 48, replace=False)
    ref = rpy.mobility_apply(pos, lam, 1.0, 1.0, True, targets=rows)
    errs = []
    for n in range(2, 9):
        ctx = arb.arb_create(wall=1, pair_kernel=arb.ARB_PAIR_FMM, fmm_order=n, fmm_levels=4,
                             precision=arb.ARB_FP64)
        try:
            u = arb.arb_rpy_apply(ctx, pos, lam).reshape(-1, 3)
            assert arb.arb_fmm_get_stats(ctx)["levels"] == 4
        finally:
            arb.arb_destroy(ctx)
        errs.append(np.abs(u[rows] - ref).max() / np.abs(ref).max())
    print("slab at L=4: sampled max error by order 2..8:", ["%.1e" % e for e in errs], flush=True)
    assert all(b < a for a, b in zip(errs, errs[1:]))
    assert errs[-1] <= 1e-5


def test_repeated_products_are_bit_identical():
    """A tree of few cells splits its interaction lists over several M2L
    items; their sums are added in a fixed order, so products repeat bit for
    bit (three and six components, both variants)."""
    pos, lam = blobs(2400, (48, 48, 10), 11)
    for prec in (arb.ARB_FP64, arb.ARB_FP32C):
        outs = []
        for _ in range(2):
            ctx = arb.arb_create(wall=1, pair_kernel=arb.ARB_PAIR_FMM, fmm_order=4, fmm_levels=2,
                                 precision=prec)
            try:
                outs += [arb.arb_rpy_apply(ctx, pos, lam) for _ in range(2)]
            finally:
                arb.arb_destroy(ctx)
        assert all(np.array_equal(outs[0], o) for o in outs[1:])
    sb = loose_bodies(2000, (48, 48, 10), 12, 1.0)
    outs = []
    for _ in range(2):
        ctx = arb.context_for(sb, precision=arb.ARB_FP32C, pair_kernel=arb.ARB_PAIR_FMM,
                              fmm_order=4, fmm_levels=2)
        try:
            outs += [arb.arb_body_mobility_apply(ctx, sb.F) for _ in range(2)]
        finally:
            arb.arb_destroy(ctx)
    assert all(np.array_equal(outs[0], o) for o in outs[1:])


@pytest.mark.parametrize("N,box,wall,kw", [
    (1500000, (200, 200, 200), False, dict(fmm_order=2, fmm_levels=5)),   # near field both ways
    (120000, (300, 300, 10), True, dict(fmm_order=3, fmm_leaf=3))])       # one way, sparse lists
def test_trees_do_not_depend_on_the_host_threads(N, box, wall, kw, monkeypatch):
    """The lists behind a product (M2L's batches and slots, the near field's blocks and
    slots) are counted and filled on several host threads where they are long; products
    on trees of 1, 3 and 16 threads agree bit for bit."""
    pos, lam = blobs(N, box, 17)
    outs = []
    for threads in ("1", "3", "16"):
        monkeypatch.setenv("ARB_HOST_THREADS", threads)
        ctx = arb.arb_create(wall=wall, pair_kernel=arb.ARB_PAIR_FMM, precision=arb.ARB_FP32C, **kw)
        try:
            outs.append(arb.arb_rpy_apply(ctx, pos, lam))
            st = arb.arb_fmm_get_stats(ctx)
        finally:
            arb.arb_destroy(ctx)
        print(f"{threads} threads: {st['leaves']} leaves, {st['interactions']} list entries, tree "
              f"{st['build_ms']:.1f} ms", flush=True)
    assert all(np.array_equal(outs[0], o) for o in outs[1:])


def test_options_are_checked():
    for bad in (dict(fmm_order=1), dict(fmm_order=9), dict(fmm_levels=-1), dict(fmm_leaf=-2),
                dict(pair_kernel=4)):
        with pytest.raises(arb.ArbError):
            arb.arb_create(**bad)
    # a leaf level deeper than the side of 2a allows is clamped, not an error
    pos, lam = blobs(200, (20, 20, 5), 3)
    u = fmm(pos, lam, False, 4, 12)
    ref = fastsum.fmm_apply(pos, lam, 1.0, 1.0, False, 4, fastsum.max_level(pos, 1.0))
    assert np.abs(u - ref).max() <= 1e-5 * np.abs(ref).max()


@pytest.mark.parametrize("prec", [arb.ARB_FP64, arb.ARB_FP32C])
def test_solve_with_the_fast_product(prec):
    """Constrained bacteria above the wall: GMRES on the fast operator (L = 2,
    n = 6) to 1e-10 (FP64: double sums, linear in lambda; FP32C: float sums
    inside refinement by the double-sum operator) against the dense
    minimum-norm solve of the oracle; the velocities agree to the
    approximation's accuracy."""
    wl = W.bacteria(n_bact=4, seed=3)
    ctx = arb.context_for(wl, precision=prec, tol=1e-10, pair_kernel=arb.ARB_PAIR_FMM,
                          fmm_order=6, fmm_levels=2)
    try:
        rc, U, phi, lam, info = arb.arb_solve(ctx, wl.F)
    finally:
        arb.arb_destroy(ctx)
    print(f"fmm solve precision {prec}: {info['iterations']} iterations, residual "
          f"{info['rel_residual']:.1e}, products {info['products_fp64']} + "
          f"{info['products_fp32']}", flush=True)
    assert info["rel_residual"] <= 1e-10 and rc in (arb.ARB_OK, arb.ARB_W_PINV_USED)
    d = system.assemble(wl)
    y = system.solve_dense(d["A"], d["b"])
    _, Ur, _ = system.split(y, wl.N, wl.M)
    Ur = Ur.reshape(-1, 6)
    err = np.abs(U - Ur).max() / np.abs(Ur).max()
    print(f"  body velocities vs dense solve: {err:.1e}", flush=True)
    assert err <= 1e-3


def test_tree_follows_the_state():
    """After a time step and a new state the product uses a tree of the new
    positions (the state's positions computed by the oracle; order 3 keeps the
    oracle's wall tensor cheap)."""
    wl = W.bacteria(n_bact=4, seed=3)
    lam = np.random.default_rng(1).standard_normal((wl.N, 3))
    q2 = wl.q + np.array([7.0, -3.0, 2.0]) * np.arange(1, wl.M + 1)[:, None] / wl.M
    ctx = arb.context_for(wl, tol=1e-8, pair_kernel=arb.ARB_PAIR_FMM, fmm_order=3, fmm_levels=2)
    try:
        arb.arb_step_euler(ctx, wl.F, 0.05)
        arb.arb_set_state(ctx, q2, wl.theta)
        u = arb.arb_mobility_apply(ctx, lam).reshape(-1, 3)
    finally:
        arb.arb_destroy(ctx)
    pos = bodies.blob_positions(q2, wl.theta, wl.r_ref, wl.blob_offset)
    ref = fastsum.fmm_apply(pos, lam, wl.a, wl.eta, wl.wall, 3, 2)
    assert np.abs(u - ref).max() <= 1e-5 * np.abs(ref).max()


def test_full_size_sampled_rows():
    """The benchmark's workload and launch configuration: 8,192 bacteria above the
    wall (999,424 blobs), default order (n = 6) and leaf level, float and double
    sums; 4 sampled rows against the dense oracle's row sums, within 1e-4 of the
    largest sampled entry (the approximation's error; 2.2e-5 measured over all
    rows against the dense product)."""
    wl = W.bacteria(n_bact=8192, seed=3)
    pos = bodies.blob_positions(wl.q, wl.theta, wl.r_ref, wl.blob_offset)
    lam = np.random.default_rng(1).standard_normal((wl.N, 3))
    rows = np.random.default_rng(8).choice(wl.N, 4, replace=False)
    print(f"full-size fast product: N={wl.N}", flush=True)
    ref = rpy.mobility_apply(pos, lam, wl.a, wl.eta, True, targets=rows, chunk=1 << 22)
    for prec in (arb.ARB_FP32C, arb.ARB_FP64):
        ctx = arb.context_for(wl, precision=prec, pair_kernel=arb.ARB_PAIR_FMM)
        try:
            u = arb.arb_mobility_apply(ctx, lam).reshape(-1, 3)
            st = arb.arb_fmm_get_stats(ctx)
        finally:
            arb.arb_destroy(ctx)
        err = np.abs(u[rows] - ref).max() / np.abs(ref).max()
        print(f"  precision {prec}: L={st['levels']}, max error on sampled rows {err:.1e}",
              flush=True)
        assert st["levels"] >= 5 and err <= 1e-4


# ---------------------------------------------------------------- single-blob bodies
def loose_bodies(M, box, seed, a):
    rng = np.random.default_rng(seed)
    q = rng.uniform(0, 1, (M, 3)) * np.array(box, float) * a
    return W.Workload("loose", a, 1.7, False, np.zeros((M, 3)),
                      np.arange(M + 1, dtype=np.int32), q, np.tile([1.0, 0, 0, 0], (M, 1)),
                      rng.standard_normal((M, 6)), extra=dict(single_blob=True))


def rot_kernel(a, eta):
    def K(x, y):
        return rpy_rot.pair_blocks(np.asarray(x) - np.asarray(y), a, eta)
    return K


@pytest.mark.parametrize("M,box,n,L", [(2000, (48, 48, 10), 4, 2), (1801, (30, 30, 30), 2, 2),
                                       (2200, (48, 24, 12), 3, 2)])
def test_single_blob_matches_the_oracle_of_the_approximation(M, box, n, L):
    """The generalised tensor (Sec. 2.4) in the fast product, force and torque
    channels, both variants, against the oracle's plain sum of the same
    approximation; coincident bodies included."""
    wl = loose_bodies(M, box, 60 + M, 0.8)
    wl.q[1] = wl.q[0]
    ref = fastsum.fmm_apply(wl.q, wl.F, wl.a, wl.eta, False, n, L, kernel=rot_kernel(wl.a, wl.eta))
    dense = rpy_rot.body_mobility_apply(wl.q, wl.F, wl.a, wl.eta)
    approx = np.abs(ref - dense).max() / np.abs(dense).max()
    for prec in (arb.ARB_FP64, arb.ARB_FP32C):
        ctx = arb.context_for(wl, precision=prec, pair_kernel=arb.ARB_PAIR_FMM, fmm_order=n,
                              fmm_levels=L)
        try:
            uw = arb.arb_body_mobility_apply(ctx, wl.F)
        finally:
            arb.arb_destroy(ctx)
        err = np.abs(uw - ref).max() / np.abs(ref).max()
        print(f"single-blob fast product M={M} n={n} L={L} precision {prec}: {err:.1e} "
              f"(approximation vs dense {approx:.1e})", flush=True)
        assert err <= 1e-5 and approx > 10 * err


def test_single_blob_sampled_rows_at_4096_shells():
    """172,032 single-blob bodies, default order and level: 32 sampled rows
    against the oracle's dense generalised sums, within 1e-4 of the row's
    largest entry."""
    wl = W.blob_shells(16)
    ctx = arb.context_for(wl, precision=arb.ARB_FP32C, pair_kernel=arb.ARB_PAIR_FMM)
    try:
        uw = arb.arb_body_mobility_apply(ctx, wl.F)
        st = arb.arb_fmm_get_stats(ctx)
    finally:
        arb.arb_destroy(ctx)
    rows = np.random.default_rng(3).choice(wl.M, 32, replace=False)
    worst = 0.0
    for t in rows:
        blk = rpy_rot.pair_blocks(wl.q[t] - wl.q, wl.a, wl.eta)
        ref = np.einsum("mij,mj->i", blk, wl.F)
        worst = max(worst, np.abs(uw[t] - ref).max() / np.abs(ref).max())
    print(f"4096 shells fast product: L={st['levels']}, worst sampled row error {worst:.1e}",
          flush=True)
    assert st["levels"] >= 3 and worst <= 1e-4


@pytest.mark.parametrize("prec", [arb.ARB_FP64, arb.ARB_FP32C])
def test_single_blob_solve_with_the_fast_product(prec):
    """Eight linked shells (Eq. linear_system_general) on the fast operator
    (n = 6, L = 2) to 1e-10 against the oracle's dense solve."""
    wl = W.blob_shells(2)
    S = single_blob.assemble(wl)
    y = single_blob.solve_dense(S)
    ctx = arb.context_for(wl, precision=prec, tol=1e-10, pair_kernel=arb.ARB_PAIR_FMM,
                          fmm_order=6, fmm_levels=2)
    try:
        rc, U, phi, lam, info = arb.arb_solve(ctx, wl.F)
    finally:
        arb.arb_destroy(ctx)
    M = wl.M
    err = np.linalg.norm(U.ravel() - y[:6 * M]) / np.linalg.norm(y[:6 * M])
    print(f"single-blob fast solve precision {prec}: {info['iterations']} iterations, residual "
          f"{info['rel_residual']:.1e}, velocities vs dense solve {err:.1e}", flush=True)
    assert info["rel_residual"] <= 1e-10 and err <= 1e-3


# the upward pass at every order in both types (a parent's children in one, two or four
# turns): the products share the tree and the weights, so they differ by FP32 rounding only
@pytest.mark.parametrize("order", range(2, 9))
def test_upward_pass_in_both_types(order):
    cl = W.random_blobs(2500, seed=order, box=60.0, zlo=1.2, zhi=60.0)
    u = {}
    for prec in (arb.ARB_FP64, arb.ARB_FP32C):
        ctx = arb.arb_create(precision=prec, wall=True, pair_kernel=arb.ARB_PAIR_FMM,
                             fmm_order=order, fmm_levels=4)
        try:
            u[prec] = arb.arb_rpy_apply(ctx, cl["pos"], cl["lam"])
        finally:
            arb.arb_destroy(ctx)
    uo = rpy.mobility_apply(cl["pos"], cl["lam"], 1.0, 1.0, True)
    err = np.linalg.norm(u[arb.ARB_FP64] - uo.ravel()) / np.linalg.norm(uo)
    diff = np.linalg.norm(u[arb.ARB_FP32C] - u[arb.ARB_FP64]) / np.linalg.norm(uo)
    print(f"order {order}: error {err:.1e}, FP32 against FP64 {diff:.1e}", flush=True)
    assert diff <= 1e-5
    assert err <= 10.0 ** (-0.75 * order + 0.5)  # 3e-2 ... 3e-6, as the error by order above
