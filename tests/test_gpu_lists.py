"""GPU: candidate lists where their rounding slack is what keeps a winner, and
calls at the limits of the lists' room and of a launch, against every seed."""
import numpy as np
import pytest

import apd_synth as S

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_2403_03571_amd as apd
    return apd.Context(0)


def _prob(inst):
    import paper_2403_03571_amd as apd
    return apd.Problem.from_instance(inst, "cuda:0")


def _instance(grid, x, A):
    dim, n = x.shape[1], len(x)
    v = np.full(n, 1.0 / n)
    v[0] += 1.0 - v.sum()
    return S.Instance(dim, grid, np.zeros(dim), np.ones(dim), x, A, v)


def _every_seed(ctx, prob, w):
    ctx.apd_set_culling(False)
    try:
        return ctx.apd_assign(prob, w, prec="fp64")
    finally:
        ctx.apd_set_culling(True)


@pytest.mark.parametrize("grid,rows", [((65536, 225), 32), ((225, 65536), 32), ((65537, 1, 9), 32)])
def test_near_ties_beside_clipped_tiles(ctx, grid, rows):
    """Pairs of seeds beside the grid's last tiles, which hold one column (row,
    layer) of very uneven pixels: the costs of a pair differ by 10^-9 to 10^-4 of
    themselves, far above the double rounding and far below that of an offset
    taken from the super-tile's centre in FP32."""
    import torch
    rng = np.random.default_rng(5)
    dim = len(grid)
    long = int(np.argmax(grid))
    thin = dim - 1 if long == 0 else 0
    side = 1.0 / grid[long]
    m = grid[long] // (2 * rows)
    x = np.full((m, 2, dim), 0.5)
    x[:, :, long] = ((2 * rows * np.arange(m) + rows / 2 + rng.uniform(-rows / 4, rows / 4, m)) * side)[:, None]
    mid = 1.0 - 0.5 / grid[thin]
    x[:, :, thin] = mid + rng.choice([-1, 1], (m, 2)) * rng.uniform(0.15, 1.0, (m, 2)) * rows * side
    r2 = (x[:, :, thin] - mid) ** 2
    w = np.zeros((m, 2))
    w[:, 1] = r2[:, 1] - r2[:, 0] + np.exp(rng.uniform(np.log(1e-9), np.log(1e-4), m)) * r2.max(1) * \
        rng.choice([-1.0, 1.0], m)
    n = 2 * m
    assert n > 256
    inst = _instance(grid, x.reshape(n, dim), np.tile(np.eye(dim), (n, 1, 1)))
    prob, wd = _prob(inst), torch.as_tensor(w.reshape(n), device="cuda:0")
    ref = _every_seed(ctx, prob, wd)
    try:
        for ppl in (0, 4, 8):
            ctx.apd_set_pixels_per_lane(ppl)
            for prec in ("fp32", "bf16", "fp64"):
                bad = int((ctx.apd_assign(prob, wd, prec=prec) != ref).sum())
                assert bad == 0, (ppl, prec, bad)
                out = ctx.apd_dual_objective_grad(prob, wd, prec=prec, counts=True)
                assert torch.equal(out["counts"].cpu(), torch.bincount(ref.reshape(-1).cpu().long(), minlength=n))
    finally:
        ctx.apd_set_pixels_per_lane(0)


@pytest.mark.parametrize("dim,grid", [(2, (64, 70)), (3, (17, 20, 33))])
@pytest.mark.parametrize("n", [2, 6])
def test_ill_conditioned_seeds_far_away(ctx, dim, grid, n):
    """Pairs of seeds 10^6 box sides away on either side along the least
    eigenvalue's direction of matrices of condition number 10^12: their costs tie
    up to the rounding of the double evaluation, which decides the labels."""
    import torch
    rng = np.random.default_rng(n)
    R = np.linalg.qr(rng.normal(size=(n // 2, dim, dim)))[0]
    ev = np.array([1e-12] + [1.0] * (dim - 1))
    A = (R * ev) @ np.swapaxes(R, -1, -2)
    A = np.repeat(0.5 * (A + np.swapaxes(A, -1, -2)), 2, axis=0)
    x = 0.5 + 1e6 * np.array([1.0, -1.0])[None, :, None] * R[:, None, :, 0]
    inst = _instance(grid, x.reshape(n, dim), A)
    prob, wd = _prob(inst), torch.zeros(n, dtype=torch.float64, device="cuda:0")
    ref = _every_seed(ctx, prob, wd)
    assert len(ref.unique()) > 1
    try:
        for ppl in (0, 4, 8):
            ctx.apd_set_pixels_per_lane(ppl)
            for prec in ("fp32", "bf16", "fp64"):
                assert torch.equal(ctx.apd_assign(prob, wd, prec=prec), ref), (ppl, prec)
    finally:
        ctx.apd_set_pixels_per_lane(0)


def _seconds(f, reps=5):
    import time

    import torch
    f()
    best = float("inf")
    for _ in range(reps):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        f()
        torch.cuda.synchronize()
        best = min(best, time.perf_counter() - t0)
    return best


def test_regions_whichever_way_the_power_is_given(ctx):
    """power = 0 (the header's name of the squared norm, what a zeroed struct
    holds) takes the same way as power = 2: the super-tiles' lists by way of
    regions, without which this call takes three times as long."""
    import torch
    inst = S.custom(2, 53333, (4000, 4000), seed=1, sigma=0.2)
    prob, wd = _prob(inst), torch.zeros(inst.n, dtype=torch.float64, device="cuda:0")
    took, labels = [], []
    for power in (2, 0):
        prob.power = power
        took.append(_seconds(lambda: ctx.apd_assign(prob, wd)))
        labels.append(ctx.apd_assign(prob, wd))
    assert torch.equal(*labels) and took[1] < 1.5 * took[0], took


def test_first_moments_of_a_very_long_axis(ctx):
    """An axis of more than 2^30 pixels: counts and centroids of the two halves
    of a row (their second moments leave 64 bits there)."""
    import torch
    M = 1200000000
    x = np.array([[0.85, 0.5], [0.97, 0.5]])
    prob = _prob(_instance((M, 1), x, np.tile(np.eye(2), (2, 1, 1))))
    cut = int(round(0.91 * M))
    for prec in ("fp32", "fp64"):
        out = ctx.apd_dual_objective_grad(prob, torch.zeros(2, dtype=torch.float64, device="cuda:0"), prec=prec,
                                          counts=True, centroids=True)
        k = out["counts"].cpu().numpy()
        assert abs(int(k[0]) - cut) <= 1 and k.sum() == M
        want = np.array([0.5 * k[0], k[0] + 0.5 * k[1]]) / M
        np.testing.assert_allclose(out["centroids"].cpu().numpy()[:, 0], want, rtol=1e-12, atol=0)


def _spread(dim, grid, n, seed):
    """Many seeds, made quickly."""
    rng = np.random.default_rng(seed)
    R = np.linalg.qr(rng.normal(size=(n, dim, dim)))[0]
    ev = np.exp(0.3 * rng.standard_normal((n, dim)))
    A = (R * ev[:, None, :]) @ np.swapaxes(R, -1, -2)
    return _instance(grid, rng.random((n, dim)), 0.5 * (A + np.swapaxes(A, -1, -2)))


@pytest.mark.parametrize("dim,grid,n", [
    (3, (128, 120, 126), 90000),   # 21 voxels per cell: two tiles per super-tile
    (3, (100, 128, 97), 31000),    # 40: four
    (3, (8, 8, 40960), 40000),     # tiles along one axis only
    (2, (1000, 1100), 30000),      # 36 pixels per cell: a list per tile
    (2, (1000, 1100), 4000),       # too few pairs: every seed
    (3, (96, 100, 90), 14000)])    # 62 per cell, numbers in the fixed scratch
def test_lists_of_dense_seeds(ctx, dim, grid, n):
    """Super-tiles of a few tiles or of one, lists of records or of numbers, in the
    context's room and in the fixed scratch: labels, gaps and counts against the
    pass over every seed."""
    import torch
    prob = _prob(_spread(dim, grid, n, n))
    w = torch.as_tensor(np.random.default_rng(n).uniform(-0.1, 0.1, n) * n ** (-2.0 / dim), device="cuda:0")
    ref = _every_seed(ctx, prob, w)
    want = torch.bincount(ref.reshape(-1).cpu().long(), minlength=n)
    for prec in ("fp32", "fp64"):
        assert torch.equal(ctx.apd_assign(prob, w, prec=prec), ref)
        for noalloc in (False, True):
            out = ctx.apd_dual_objective_grad(prob, w, prec=prec, counts=True, noalloc=noalloc)
            assert torch.equal(out["counts"].cpu(), want)
    lab, gap = ctx.apd_assign(prob, w, rel_gap=True)
    assert torch.equal(lab, ref) and bool(((gap >= 0) & (gap <= 1)).all())


def test_dense_seeds_and_fixed_scratch_keep_their_lists(ctx):
    """Seeds just too dense for super-tiles of three cell diameters, and lists too
    long for records in the fixed scratch, are not left to scans of every seed by
    every tile (four and eight times the time)."""
    import torch

    def took(side, n, **kw):
        prob = _prob(_spread(3, (side,) * 3, n, 1))
        w = torch.zeros(n, dtype=torch.float64, device="cuda:0")
        return _seconds(lambda: ctx.apd_dual_objective_grad(prob, w, **kw))

    assert took(128, 34952) < 3.0 * took(128, 26214)
    assert took(230, 30000, noalloc=True) < 4.0 * took(230, 30000)


def test_room_of_lists_that_are_not_used(ctx):
    """Dense seeds in a context of their own (the runtime's own room taken before):
    4225 super-tiles' records and at most as many regions' half as large, 415 and
    288 MB, and some 60 for the seeds, not 1.5 GB for each of 15625 tiles."""
    import torch
    import paper_2403_03571_amd as apd
    n = 200000
    prob = _prob(_spread(3, (200, 200, 200), n, 2))
    w = torch.zeros(n, dtype=torch.float64, device="cuda:0")
    small = _prob(_spread(3, (100, 100, 100), 25000, 2))
    ctx.apd_dual_objective_grad(small, w[:25000])
    c = apd.Context(0)
    try:
        free = torch.cuda.mem_get_info()[0]
        c.apd_dual_objective_grad(prob, w)
        assert free - torch.cuda.mem_get_info()[0] < 1 << 30
    finally:
        c.close()


def test_numbers_instead_of_records_in_little_memory(ctx):
    """Records of 8.4 GiB with 14 GiB free: the lists hold the seeds' numbers, in an
    evaluation and in a fit's captured ones, and the results stay the same."""
    import torch
    import paper_2403_03571_amd as apd
    side, per = 22912, 280
    n = side * side // per
    rng = np.random.default_rng(9)
    a, t = rng.uniform(1.0, 3.0, n), rng.uniform(0.0, np.pi, n)
    prob = _prob(_instance((side, side), rng.random((n, 2)), S.aniso2d(a, t)))
    w = torch.zeros(n, dtype=torch.float64, device="cuda:0")

    def work():
        c = apd.Context(0)
        try:
            free = torch.cuda.mem_get_info()[0]
            out = c.apd_dual_objective_grad(prob, w, counts=True)
            fit, _ = c.apd_fit_weights(prob, eps=1e-6, max_evals=3)
            return out["counts"], out["g"], fit, free - torch.cuda.mem_get_info()[0]
        finally:
            c.close()

    want = work()
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    held = []
    while torch.cuda.mem_get_info()[0] > 15 << 30:
        held.append(torch.empty(1 << 30, dtype=torch.uint8, device="cuda:0"))
    try:
        got = work()
    finally:
        held.clear()
        torch.cuda.empty_cache()
    assert want[3] > 8 << 30 and got[3] < 3 << 30
    assert torch.equal(got[0], want[0]) and got[1] == want[1] and torch.equal(got[2], want[2])


@pytest.mark.parametrize("grid,n,rows,gap_rows", [
    ((100, 101, 102), 2700, 2, 4), ((79, 80, 82), 2000, 2, 2), ((100, 101, 102), 2200, 4, 4),
    ((600000, 1, 1), 2000, 4, 4), ((20000, 3, 2), 900, 4, 4), ((9, 7, 3), 40, 2, 2)])
def test_rows_of_passes_with_gaps_and_of_thin_grids(ctx, grid, n, rows, gap_rows):
    """Two rows per lane on dense 3D grids, but not for the relative gaps and not
    where the tiles stick out of the grid; labels and gaps against every seed."""
    import torch
    prob = _prob(_spread(3, grid, n, n))
    w = torch.zeros(n, dtype=torch.float64, device="cuda:0")
    ref = _every_seed(ctx, prob, w)
    assert torch.equal(ctx.apd_assign(prob, w), ref)
    assert ctx.apd_last_pass_stats()["pixels_per_lane"] == rows
    lab, gap = ctx.apd_assign(prob, w, rel_gap=True)
    assert ctx.apd_last_pass_stats()["pixels_per_lane"] == gap_rows
    exact = ctx.apd_assign(prob, w, prec="fp64", rel_gap=True)[1]
    assert torch.equal(lab, ref) and bool((gap <= exact * (1 + 1e-6) + 1e-12).all())


def test_regions_have_room_for_their_seeds(ctx):
    """Regions no longer than their lists have room for: four times the pixels at
    the same density take about four times as long, not sixteen."""
    import torch
    took = []
    for side in (2000, 4000):
        n = side * side // 100
        prob = _prob(S.custom(2, n, (side, side), seed=1, sigma=0.0))
        w = torch.zeros(n, dtype=torch.float64, device="cuda:0")
        took.append(_seconds(lambda: ctx.apd_dual_objective_grad(prob, w)))
    assert took[1] < 10.0 * took[0], took


def test_autotune_knows_the_default(ctx):
    """Where the default's two rows per lane, which cannot be set, are the fastest
    (36 us, 44 with four), the tuned context keeps the rule that takes them."""
    import torch
    n = 213
    prob = _prob(_spread(3, (40, 40, 40), n, 3))
    w = torch.zeros(n, dtype=torch.float64, device="cuda:0")
    labels = ctx.apd_assign(prob, w)
    assert ctx.apd_last_pass_stats()["pixels_per_lane"] == 2
    try:
        choice = ctx.apd_autotune(prob, w, reps=20)
        assert len(choice["pass_ms"]) == 6 and min(choice["pass_ms"]) > 0.0
        assert (choice["variant"], choice["culling"], choice["pixels_per_lane"]) == (1, 1, 0)
        assert torch.equal(ctx.apd_assign(prob, w), labels)
        assert ctx.apd_last_pass_stats()["pixels_per_lane"] == 2
    finally:
        ctx.apd_set_variant(2)
        ctx.apd_set_culling(True)
        ctx.apd_set_pixels_per_lane(0)


def test_autotune_after_the_seeds_grew():
    """The autotuner's passes write their gradient into the context's own buffer, which
    more seeds than it holds (1024 at first) replace: the new one is written, and nothing
    beside it."""
    import torch

    import paper_2403_03571_amd as apd
    ctx = apd.Context(0)
    small = _prob(_spread(3, (40, 40, 40), 213, 3))
    ctx.apd_autotune(small, torch.zeros(213, dtype=torch.float64, device="cuda:0"), reps=1)
    for n in (1025, 3971, 5000):
        prob = _prob(_spread(3, (64, 64, 64), n, 3))
        w = torch.zeros(n, dtype=torch.float64, device="cuda:0")
        beside = [torch.full((1 << 14,), 7, dtype=torch.uint8, device="cuda:0") for _ in range(8)]
        choice = ctx.apd_autotune(prob, w, reps=1)
        assert len(choice["pass_ms"]) == 6 and min(choice["pass_ms"]) > 0.0
        assert all(bool((b == 7).all()) for b in beside)
        a, b = ctx.apd_dual_objective_grad(prob, w), apd.Context(0).apd_dual_objective_grad(prob, w)
        assert a["g"] == b["g"] and torch.equal(a["grad"], b["grad"])


def test_batched_autotune_times_a_kernel_once(ctx):
    """The two tiers' lists run one kernel: one time for both, and the FP32 name if
    it is the fastest."""
    probs = [_prob(S.custom(2, 40 + b, (128, 96), seed=b, sigma=0.0)) for b in range(6)]
    try:
        r = ctx.apd_autotune_batched(probs, evals=4)
        assert r["fit_ms"][4] == r["fit_ms"][1] > 0.0 and r["kernel"] != "bf16-lists"
    finally:
        ctx.apd_set_batch_kernel(None)


@pytest.mark.parametrize("dim,grid", [(2, (400, 390)), (3, (60, 61, 59))])
@pytest.mark.parametrize("n", [1024, 1025, 10240, 10241])
def test_edges_of_the_blocks_over_seeds(ctx, dim, grid, n):
    """One or several blocks in the first and last kernel of an evaluation, and the
    most seeds whose super-tile bounds a thread of 512 keeps in registers: labels and
    counts against every seed, the scalars of all tiers the same to the last bit."""
    import torch
    prob = _prob(_spread(dim, grid, n, n))
    w = torch.as_tensor(np.random.default_rng(n).uniform(-0.1, 0.1, n) * n ** (-2.0 / dim), device="cuda:0")
    ref = _every_seed(ctx, prob, w)
    want = torch.bincount(ref.reshape(-1).cpu().long(), minlength=n)
    outs = []
    for prec in ("fp32", "bf16", "fp64"):
        assert torch.equal(ctx.apd_assign(prob, w, prec=prec), ref)
        outs += [ctx.apd_dual_objective_grad(prob, w, prec=prec, counts=True, noalloc=na) for na in (False, True)]
    for out in outs:
        assert torch.equal(out["counts"].cpu(), want) and torch.equal(out["grad"], outs[0]["grad"])
        assert out["g"] == outs[0]["g"] and out["maxrel"] == outs[0]["maxrel"]
