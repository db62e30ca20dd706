"""GPU parity of the blob mobility product u = M lambda (Sec. 2.3) against the oracle.

Tolerances: relative L2 <= 1e-12 for the FP64 pair sum, <= 1e-5 for FP32C.
"""
import numpy as np
import pytest

from oracle import rpy
from paper_2107_10800_amd import arb
from paper_2107_10800_amd import workloads as W

pytestmark = pytest.mark.gpu

TOL = {arb.ARB_FP64: 1e-12, arb.ARB_FP32C: 1e-5}


def rel(a, b):
    return np.linalg.norm(np.ravel(a) - np.ravel(b)) / np.linalg.norm(np.ravel(b))


@pytest.fixture(scope="module")
def ctxs():
    out = {}
    for prec in (arb.ARB_FP64, arb.ARB_FP32C):
        for wall in (False, True):
            out[(prec, wall)] = arb.arb_create(precision=prec, wall=wall)
    yield out
    for c in out.values():
        arb.arb_destroy(c)


@pytest.mark.parametrize("n", [1, 7, 256, 300, 1000])
@pytest.mark.parametrize("wall", [False, True])
@pytest.mark.parametrize("prec", [arb.ARB_FP64, arb.ARB_FP32C])
def test_small_clouds(ctxs, n, wall, prec):
    # overlapping random clouds: near and far branches, several tiles, ragged tail
    cl = W.random_blobs(n, seed=100 + n)
    print(f"pair n={n} wall={wall} prec={prec}", flush=True)
    u = arb.arb_rpy_apply(ctxs[(prec, wall)], cl["pos"], cl["lam"])
    uo = rpy.mobility_apply(cl["pos"], cl["lam"], 1.0, 1.0, wall)
    assert rel(u, uo) <= TOL[prec]


def test_self_mobility_single_blob(ctxs):
    pos = np.array([[0.3, -1.0, 2.5]])
    lam = np.array([1.0, -2.0, 0.5])
    u = arb.arb_rpy_apply(ctxs[(arb.ARB_FP64, False)], pos, lam)
    assert np.allclose(u, lam / (6 * np.pi), rtol=1e-15, atol=0)


@pytest.mark.parametrize("slices", [1, 3, 16])
def test_slices_do_not_change_result(slices):
    cl = W.random_blobs(2000, seed=9, box=30.0)
    outs = []
    for sl in (slices, 0):
        c = arb.arb_create(precision=arb.ARB_FP64, wall=True, slices=sl)
        try:
            outs.append(arb.arb_rpy_apply(c, cl["pos"], cl["lam"]))
            again = arb.arb_rpy_apply(c, cl["pos"], cl["lam"])
            assert np.array_equal(outs[-1], again)  # deterministic reduction order
        finally:
            arb.arb_destroy(c)
    assert rel(outs[0], outs[1]) <= 1e-14


@pytest.mark.parametrize("prec", [arb.ARB_FP64, arb.ARB_FP32C])
def test_slab_full_size_sampled(ctxs, prec):
    # the 16,384-blob wall slab at full size, launch shape as in the benchmark;
    # the oracle evaluates sampled rows exactly against every source
    sl = W.slab()
    N = len(sl["pos"])
    print(f"pair slab N={N} prec={prec}", flush=True)
    u = arb.arb_rpy_apply(ctxs[(prec, True)], sl["pos"], sl["lam"]).reshape(N, 3)
    rng = np.random.default_rng(0)
    tg = np.unique(np.concatenate([[0, 255, 256, N - 1], rng.integers(0, N, 28)]))
    uo = rpy.mobility_apply(sl["pos"], sl["lam"], 1.0, 1.0, True, targets=tg)
    assert rel(u[tg], uo) <= TOL[prec]


@pytest.mark.parametrize("wall", [True, False])
def test_far_tiles_on_ordered_blobs(wall):
    # blobs stored in spatial order (the slab sorted along x; bacteria, whose
    # blobs are contiguous per body): most 64-blob tiles are compact and far
    # apart, so the symmetric FP32 kernel evaluates those tile pairs from the hi
    # parts of the positions alone; sampled rows against the oracle's compiled
    # route over every source, at the FP32 product's bar
    from oracle import rpy_c

    sl = W.slab()
    order = np.argsort(sl["pos"][:, 0], kind="stable")
    pos, lam = sl["pos"][order], sl["lam"][order]
    if not wall:
        pos = pos + np.array([0.0, 0.0, 30.0])
    N = len(pos)
    bact = W.bacteria(n_bact=256, seed=3)
    import oracle.bodies as ob
    bpos = ob.blob_positions(bact.q, bact.theta, bact.r_ref, bact.blob_offset)
    blam = np.random.default_rng(5).standard_normal(bpos.shape)
    for name, P, L in (("sorted slab", pos, lam), ("256 bacteria", bpos, blam)):
        c = arb.arb_create(precision=arb.ARB_FP32C, wall=wall, pair_kernel=arb.ARB_PAIR_SYMMETRIC)
        try:
            u = arb.arb_rpy_apply(c, P, L).reshape(-1, 3)
        finally:
            arb.arb_destroy(c)
        rng = np.random.default_rng(1)
        tg = np.unique(np.concatenate([[0, 63, 64, len(P) - 1], rng.integers(0, len(P), 124)]))
        uo = rpy_c.mobility_apply(P, L, 1.0, 1.0, wall, targets=tg)
        e = rel(u[tg], uo)
        print(f"  far tiles, {name}, wall={wall}: sampled-row error {e:.2e}", flush=True)
        assert e <= TOL[arb.ARB_FP32C]


@pytest.mark.parametrize("prec", [arb.ARB_FP64, arb.ARB_FP32C])
def test_context_product_in_library_order(prec):
    # the 16,384-blob slab as a context's state (one-blob bodies in the
    # generator's random order): the library runs its products on a copy sorted
    # along a Morton curve and reads lambda / writes u through the permutation.
    # u = M lambda and the saddle operator's first rows M lambda - K U on sampled
    # rows against the oracle's compiled route
    from oracle import rpy_c

    sl = W.slab()
    N = len(sl["pos"])
    wl = W.loose_blobs(sl["pos"])
    rng = np.random.default_rng(2)
    lam = sl["lam"]
    U = rng.standard_normal((N, 6))
    c = arb.context_for(wl, precision=prec)
    try:
        u = arb.arb_mobility_apply(c, lam).reshape(N, 3)
        Ay = arb.arb_system_apply(c, np.concatenate([lam.ravel(), U.ravel()]))
    finally:
        arb.arb_destroy(c)
    tg = np.unique(np.concatenate([[0, 63, 64, N - 1], rng.integers(0, N, 124)]))
    uo = rpy_c.mobility_apply(sl["pos"], lam, 1.0, 1.0, True, targets=tg)
    e1 = rel(u[tg], uo)
    # one-blob bodies at their tracking points: (K U)_i = u_i
    e2 = rel(Ay[:3 * N].reshape(N, 3)[tg], uo - U[tg, :3])
    print(f"  context product prec={prec}: {e1:.2e}, system rows {e2:.2e}", flush=True)
    assert e1 <= TOL[prec] and e2 <= TOL[prec]


def test_device_pointer_entry_point_matches_host(ctxs):
    import torch

    cl = W.random_blobs(777, seed=3)
    c = ctxs[(arb.ARB_FP32C, True)]
    u_host = arb.arb_rpy_apply(c, cl["pos"], cl["lam"])
    pos = torch.tensor(cl["pos"], dtype=torch.float64, device="cuda")
    lam = torch.tensor(cl["lam"], dtype=torch.float64, device="cuda")
    u = torch.zeros_like(lam)
    stream = torch.cuda.current_stream()
    arb.arb_rpy_apply_dev(c, 777, pos, lam, u, stream=stream.cuda_stream)
    torch.cuda.synchronize()
    assert np.array_equal(u.cpu().numpy().ravel(), u_host)


def test_below_wall_rejected(ctxs):
    pos = np.array([[0.0, 0.0, 3.0], [1.0, 1.0, 0.9]])
    with pytest.raises(arb.ArbError) as e:
        arb.arb_rpy_apply(ctxs[(arb.ARB_FP64, True)], pos, np.ones(6))
    assert e.value.code == arb.ARB_E_BELOW_WALL
    with pytest.raises(arb.ArbError) as e:
        arb.arb_rpy_apply(ctxs[(arb.ARB_FP64, False)], pos, np.array([1, np.nan, 0, 0, 0, 0.0]))
    assert e.value.code == arb.ARB_E_NAN


@pytest.mark.parametrize("n", [1, 65, 300, 1000, 5000])
@pytest.mark.parametrize("wall", [False, True])
@pytest.mark.parametrize("prec", [arb.ARB_FP64, arb.ARB_FP32C])
def test_symmetric_kernel_small(n, wall, prec):
    # symmetric kernel (each unordered pair once): ragged tiles and blocks,
    # coincident-free random clouds with overlapping pairs
    cl = W.random_blobs(n, seed=200 + n, box=8.0 + n ** (1 / 3))
    c = arb.arb_create(precision=prec, wall=wall, pair_kernel=arb.ARB_PAIR_SYMMETRIC)
    try:
        print(f"symmetric pair n={n} wall={wall} prec={prec}", flush=True)
        u = arb.arb_rpy_apply(c, cl["pos"], cl["lam"])
        assert arb.arb_get_slices(c, n) < 0
    finally:
        arb.arb_destroy(c)
    uo = rpy.mobility_apply(cl["pos"], cl["lam"], 1.0, 1.0, wall)
    assert rel(u, uo) <= TOL[prec]


@pytest.mark.parametrize("prec", [arb.ARB_FP64, arb.ARB_FP32C])
def test_symmetric_kernel_slab_sampled(prec):
    sl = W.slab()
    N = len(sl["pos"])
    c = arb.arb_create(precision=prec, wall=True, pair_kernel=arb.ARB_PAIR_SYMMETRIC)
    try:
        print(f"symmetric pair slab N={N} prec={prec}", flush=True)
        u = arb.arb_rpy_apply(c, sl["pos"], sl["lam"]).reshape(N, 3)
        shape = arb.arb_get_slices(c, N)
    finally:
        arb.arb_destroy(c)
    assert shape < 0
    rng = np.random.default_rng(1)
    tg = np.unique(np.concatenate([[0, 63, 64, 255, 256, N - 1], rng.integers(0, N, 26)]))
    uo = rpy.mobility_apply(sl["pos"], sl["lam"], 1.0, 1.0, True, targets=tg)
    assert rel(u[tg], uo) <= TOL[prec]


def test_symmetric_matches_target_parallel_fp64():
    # the two FP64 kernels agree to rounding on a ragged size above the autotune threshold
    cl = W.random_blobs(9000, seed=31, box=60.0, zlo=1.5, zhi=12.0)
    outs = []
    for kind in (arb.ARB_PAIR_TARGET, arb.ARB_PAIR_SYMMETRIC):
        c = arb.arb_create(precision=arb.ARB_FP64, wall=True, pair_kernel=kind)
        try:
            outs.append(arb.arb_rpy_apply(c, cl["pos"], cl["lam"]))
        finally:
            arb.arb_destroy(c)
    assert rel(outs[1], outs[0]) <= 1e-13


@pytest.mark.parametrize("kind", [arb.ARB_PAIR_TARGET, arb.ARB_PAIR_SYMMETRIC])
@pytest.mark.parametrize("prec", [arb.ARB_FP64, arb.ARB_FP32C])
def test_blob_radius_and_viscosity(kind, prec):
    # a != 1 and eta != 1: the FP32 kernels work in units of a and rescale
    a, eta = 0.7, 1.9
    cl = W.random_blobs(600, seed=77, box=10.0, zlo=1.05 * a, zhi=5.0)
    c = arb.arb_create(precision=prec, wall=True, a=a, eta=eta, pair_kernel=kind)
    try:
        u = arb.arb_rpy_apply(c, cl["pos"], cl["lam"])
    finally:
        arb.arb_destroy(c)
    uo = rpy.mobility_apply(cl["pos"], cl["lam"], a, eta, True)
    assert rel(u, uo) <= TOL[prec]


@pytest.mark.parametrize("kind", [arb.ARB_PAIR_TARGET, arb.ARB_PAIR_SYMMETRIC])
@pytest.mark.parametrize("prec", [arb.ARB_FP64, arb.ARB_FP32C])
def test_coincident_blobs_and_empty_input(kind, prec):
    # two distinct blobs at one position (r = 0 off the diagonal: the self-mobility
    # block) in the same and in different tiles; and N = 0
    cl = W.random_blobs(300, seed=41, box=9.0)
    pos = cl["pos"].copy()
    pos[7] = pos[3]          # same 64-blob tile
    pos[250] = pos[10]       # different tiles and I-blocks
    c = arb.arb_create(precision=prec, wall=True, pair_kernel=kind)
    try:
        u = arb.arb_rpy_apply(c, pos, cl["lam"])
        assert arb.arb_rpy_apply(c, np.zeros((0, 3)), np.zeros(0)).size == 0
    finally:
        arb.arb_destroy(c)
    uo = rpy.mobility_apply(pos, cl["lam"], 1.0, 1.0, True)
    assert np.all(np.isfinite(u))
    assert rel(u, uo) <= TOL[prec]


# products without atomics or slices of the caller's choice: one launch up to 1,024 blobs
# (one wavefront per target: 64 lanes, part of them, several turns), the ring of 64-blob
# tiles from 1,025 to 8,191 (odd and even numbers of tiles, where the opposite tile counts
# once; 4, 2 and 1 wavefronts per tile; a last tile of 1 blob and a full one)
@pytest.mark.parametrize("n", [2, 63, 64, 65, 1024, 1025, 1088, 2048, 2049, 4096, 4161, 5824, 8191])
@pytest.mark.parametrize("wall", [False, True])
@pytest.mark.parametrize("prec", [arb.ARB_FP64, arb.ARB_FP32C])
def test_small_and_mid_sizes(n, wall, prec):
    a, eta = 0.8, 1.3
    cl = W.random_blobs(n, seed=300 + n, box=8.0 + n ** 0.5, zlo=1.0, zhi=9.0)
    rng = np.random.default_rng(n)
    tg = np.unique(np.concatenate([[0, n - 1, n // 2, min(63, n - 1)], rng.integers(0, n, 40)]))
    uo = rpy.mobility_apply(cl["pos"], cl["lam"], a, eta, wall, targets=tg)
    loose = arb.arb_create(precision=prec, wall=wall, a=a, eta=eta)
    state = arb.context_for(W.loose_blobs(cl["pos"], a=a, eta=eta, wall=wall), precision=prec)
    try:
        print(f"pair n={n} wall={wall} prec={prec}", flush=True)
        for f in (lambda: arb.arb_rpy_apply(loose, cl["pos"], cl["lam"]),
                  lambda: arb.arb_mobility_apply(state, cl["lam"])):
            u = f()
            assert np.array_equal(u, f())
            assert rel(u.reshape(n, 3)[tg], uo) <= TOL[prec]
    finally:
        arb.arb_destroy(loose)
        arb.arb_destroy(state)


# the symmetric product leaves the buffer of its sums zero for the next one: products of
# two sizes in turn, the larger first and last
@pytest.mark.parametrize("prec", [arb.ARB_FP64, arb.ARB_FP32C])
def test_symmetric_products_in_turn(prec):
    ctx = arb.arb_create(precision=prec, wall=True, a=0.8, eta=1.3,
                         pair_kernel=arb.ARB_PAIR_SYMMETRIC)
    try:
        for n in (300, 70, 70, 300, 520, 300):
            cl = W.random_blobs(n, seed=n, box=8.0 + n ** 0.5, zlo=1.0, zhi=9.0)
            uo = rpy.mobility_apply(cl["pos"], cl["lam"], 0.8, 1.3, True)
            assert rel(arb.arb_rpy_apply(ctx, cl["pos"], cl["lam"]), uo.ravel()) <= TOL[prec]
    finally:
        arb.arb_destroy(ctx)


# the result in the place of an input: a product whose kernels write no result before they
# have read every input (or go through scratch) gives the bits of one with an array of its
# own; one launch at 300 blobs, the ring at 2,000, the tuned kernels at 8,192; whole
# overlap, and with the result a few blobs further on
@pytest.mark.parametrize("n", [300, 1024, 2000, 8192])
@pytest.mark.parametrize("prec", [arb.ARB_FP64, arb.ARB_FP32C])
def test_products_in_place(n, prec):
    import torch

    cl = W.random_blobs(n, seed=500 + n, box=8.0 + n ** 0.5, zlo=1.0, zhi=9.0)
    c = arb.arb_create(precision=prec, wall=True, pair_kernel=arb.ARB_PAIR_TARGET if n > 8191 else
                       arb.ARB_PAIR_AUTO)
    state = arb.context_for(W.loose_blobs(cl["pos"]), precision=prec,
                            pair_kernel=arb.ARB_PAIR_TARGET if n > 8191 else arb.ARB_PAIR_AUTO)
    st = torch.cuda.Stream()  # one stream for the copies and the products
    s = st.cuda_stream

    def room(x, shift):
        """x in the middle of a larger array, and the result's place beside it."""
        buf = torch.zeros(3 * n + 60, dtype=torch.float64, device="cuda")
        v = buf[30:30 + 3 * n]
        v.copy_(x)
        return v, buf[30 + shift:30 + shift + 3 * n]

    try:
        print(f"in place n={n} prec={prec}", flush=True)
        torch.cuda.set_stream(st)
        pos, lam = (torch.tensor(np.ravel(cl[k]), dtype=torch.float64, device="cuda")
                    for k in ("pos", "lam"))
        want, held = torch.zeros_like(lam), torch.zeros_like(lam)
        arb.arb_rpy_apply_dev(c, n, pos, lam, want, stream=s)
        arb.arb_mobility_apply_dev(state, lam, held, stream=s)
        for shift in (0, 30, -6):
            x, u = room(lam, shift)
            arb.arb_rpy_apply_dev(c, n, pos, x, u, stream=s)
            assert torch.equal(u, want), shift
            x, u = room(pos, shift)
            arb.arb_rpy_apply_dev(c, n, x, lam, u, stream=s)
            assert torch.equal(u, want), shift
            x, u = room(lam, shift)
            arb.arb_mobility_apply_dev(state, x, u, stream=s)
            assert torch.equal(u, held), shift
    finally:
        torch.cuda.synchronize()
        torch.cuda.set_stream(torch.cuda.default_stream())
        arb.arb_destroy(c)
        arb.arb_destroy(state)


# FP32 products below 8,192 blobs keep both parts of every position: one source at about
# (1000, 1000, 1000) and 1,984 targets about 255 away, in compact tiles, every coordinate
# just short of half a float step off its rounded value, the source down and the targets
# up.  The rounded positions alone are 1.7 x 0.98 x 2^-14 off in distance, 4.1e-7 of every
# velocity; the tensor in float adds errors of about random sign, at most 1 ulp of the
# reciprocal root (2^-23) and half of three roundings of r^2 (3 x 2^-25) if all of one sign
def test_mid_size_fp32_keeps_both_parts_of_the_positions():
    rng = np.random.default_rng(12)
    step = 2.0 ** -14                    # of floats in [512, 1024)
    n = 2048
    pos = 840.0 + np.floor(rng.uniform(0, 20.0, (n, 3)) / step) * step + 0.49 * step
    pos[:64] = 990.0 + np.floor(rng.uniform(0, 10.0, (64, 3)) / step) * step
    pos[5] = 1000.0 - 0.49 * step
    lam = np.zeros((n, 3))
    lam[5] = (0.7, -1.1, 0.4)
    uo = rpy.mobility_apply(pos, lam, 1.0, 1.0, False)[64:]
    err = {}
    for kind in (arb.ARB_PAIR_AUTO, arb.ARB_PAIR_TARGET):
        c = arb.arb_create(precision=arb.ARB_FP32C, pair_kernel=kind)
        try:
            u = arb.arb_rpy_apply(c, pos, lam).reshape(n, 3)[64:]
        finally:
            arb.arb_destroy(c)
        err[kind] = np.mean(np.sum(u * uo, 1) / np.sum(uo * uo, 1) - 1.0)
    print(f"mean error {err[arb.ARB_PAIR_AUTO]:.1e}, target-parallel kernel "
          f"{err[arb.ARB_PAIR_TARGET]:.1e}", flush=True)
    assert abs(err[arb.ARB_PAIR_AUTO]) <= 2.0 ** -22
    assert abs(err[arb.ARB_PAIR_TARGET]) <= 2.0 ** -22


# the reported launch shape tells ordered sums (>= 0) from atomic ones (< 0), and the
# slices of the target-parallel kernel from a product without any
@pytest.mark.parametrize("n,kind,slices,want", [
    (300, arb.ARB_PAIR_AUTO, 0, lambda k: k > 0), (300, arb.ARB_PAIR_TARGET, 0, lambda k: k > 0),
    (300, arb.ARB_PAIR_SYMMETRIC, 0, lambda k: k < 0), (2000, arb.ARB_PAIR_AUTO, 0, lambda k: k == 0),
    (2000, arb.ARB_PAIR_AUTO, 3, lambda k: k == 3), (2000, arb.ARB_PAIR_TARGET, 0, lambda k: k > 0),
    (2000, arb.ARB_PAIR_SYMMETRIC, 0, lambda k: k < 0),
    (8191, arb.ARB_PAIR_AUTO, 0, lambda k: k == 0), (8192, arb.ARB_PAIR_AUTO, 0, lambda k: k != 0)])
def test_reported_launch_shape(n, kind, slices, want):
    cl = W.random_blobs(n, seed=n, box=8.0 + n ** 0.5)
    c = arb.arb_create(precision=arb.ARB_FP32C, pair_kernel=kind, slices=slices)
    try:
        assert arb.arb_get_slices(c, n) > 0          # before any product: the heuristic
        u = [arb.arb_rpy_apply(c, cl["pos"], cl["lam"]) for _ in range(3)]
        k = arb.arb_get_slices(c, n)
    finally:
        arb.arb_destroy(c)
    assert want(k), k
    if k >= 0:
        assert np.array_equal(u[1], u[2])
