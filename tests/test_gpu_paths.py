"""GPU: the edges of the launch and dispatch rules (work splits, list
lengths, remainders), each against the CPU oracle or against the same
problem on another path."""
import numpy as np
import pytest

import apd_synth as S
import oracle as O

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_2403_03571_amd as apd
    return apd.Context(0)


def _prob(inst):
    import paper_2403_03571_amd as apd
    return apd.Problem.from_instance(inst, "cuda:0")


@pytest.mark.parametrize("count", [1, 255, 257, 600])
def test_batch_work_list(ctx, count):
    """The list of active work over fewer, as many and more instances than a
    block has threads, instances leaving at different evaluations: each fit
    certified by the oracle's recount, and bit-identical to a batch of one."""
    insts = [S.custom(2, 2 + b % 7, (33 + 8 * (b % 5), 70), seed=b, sigma=0.3) for b in range(count)]
    probs = [_prob(i) for i in insts]
    ws, reps, status = ctx.apd_fit_weights_batched(probs, eps=0.05)
    assert status == "APD_OK" and len({r.evals for r in reps}) > (1 if count > 1 else 0)
    for b in {0, count // 2, count - 1}:
        one, rep, _ = ctx.apd_fit_weights_batched([probs[b]], eps=0.05)
        assert rep[0].evals == reps[b].evals
        np.testing.assert_array_equal(one[0].cpu().numpy(), ws[b].cpu().numpy())
        assert O.evaluate(insts[b], ws[b].cpu().numpy()).maxrel < 0.05


@pytest.mark.parametrize("dim,grid", [(2, (70, 45)), (3, (19, 13, 21))])
@pytest.mark.parametrize("prec", ["fp32", "bf16"])
@pytest.mark.parametrize("ppl", [4, 8])
def test_recheck_in_the_tile(ctx, dim, grid, prec, ppl):
    """Every pixel of the tiles re-checked (each seed twice: exact ties), half
    of them, or none: labels, counts (pixel weights among them) and gaps
    against the oracle."""
    import torch
    for twice in (11, 5, 0):
        inst = S.custom(dim, 11, grid, seed=twice + dim, sigma=0.3)
        x = np.concatenate([inst.x, inst.x[:twice]])
        A = np.concatenate([inst.A, inst.A[:twice]])
        n = len(x)
        w = np.random.default_rng(3).uniform(-0.01, 0.01, 11)
        w = np.concatenate([w, w[:twice]])
        inst = S.Instance(dim, grid, inst.lo, inst.hi, x, A, np.full(n, 1.0 / n))
        inst.v[0] += 1.0 - inst.v.sum()
        ctx.apd_set_pixels_per_lane(ppl)
        try:
            for case in (inst, S.masked(inst, S.disk_weights(grid, inst.lo, inst.hi, (0.5,) * dim, 0.45))):
                prob = _prob(case)
                wd = torch.as_tensor(w, device="cuda:0")
                ref, best, second = O.assign(case, w)
                lab, gap = ctx.apd_assign(prob, wd, prec=prec, rel_gap=True)
                np.testing.assert_array_equal(lab.cpu().numpy(), ref)
                np.testing.assert_array_equal(ctx.apd_assign(prob, wd, prec=prec).cpu().numpy(), ref)
                rel = (second - best) / (second + w.max())
                assert np.all(gap.cpu().numpy() <= rel * (1 + 1e-6) + 1e-12)
                out = ctx.apd_dual_objective_grad(prob, wd, prec=prec, counts=True)
                q = np.ones(case.J, np.int64) if case.mass is None else case.mass.astype(np.int64)
                np.testing.assert_array_equal(out["counts"].cpu().numpy(), np.bincount(ref, q, n).astype(np.int64))
                if twice == 11:
                    assert ctx.apd_last_pass_stats()["rechecked"] == case.J
        finally:
            ctx.apd_set_pixels_per_lane(0)


@pytest.mark.parametrize("dim,grid", [(2, (200, 130)), (3, (40, 33, 50))])
@pytest.mark.parametrize("n", [255, 256, 257, 2048, 2049, 3073, 12289])
def test_candidate_lists_by_the_number_of_seeds(ctx, dim, grid, n):
    """Lists from every seed in one round of a block or from super-tiles, with
    256 or 1024 threads, a thread's bounds in registers or read again: labels
    of both tiers and the static-scratch evaluation against the oracle, the
    weights offset by far more than their spread."""
    import torch
    inst = S.custom(dim, n, grid, seed=n, sigma=0.3, amax=4.0)
    w = np.random.default_rng(n).uniform(-0.3, 0.3, n) * n ** (-2.0 / dim) + 1e3
    prob, wd = _prob(inst), torch.as_tensor(w, device="cuda:0")
    ref, _, _ = O.assign(inst, w)
    for prec in ("fp32", "bf16"):
        np.testing.assert_array_equal(ctx.apd_assign(prob, wd, prec=prec).cpu().numpy(), ref)
        assert ctx.apd_last_pass_stats()["kernel"] == prec + "-lists"
    for noalloc in (False, True):
        out = ctx.apd_dual_objective_grad(prob, wd, counts=True, noalloc=noalloc)
        np.testing.assert_array_equal(out["counts"].cpu().numpy(), np.bincount(ref, minlength=n))


@pytest.mark.parametrize("dim,grid,n,rows", [
    (3, (79, 80, 82), 3, 2), (3, (81, 80, 82), 1300, 2), (3, (81, 80, 82), 1100, 4), (3, (129, 128, 128), 2100, 8),
    (3, (9, 7, 3), 40, 2), (2, (2048, 2049), 4100, 8), (2, (2048, 2047), 4100, 4), (2, (17, 5), 300, 4)])
def test_rows_per_lane_by_grid_and_seeds(ctx, dim, grid, n, rows):
    """Either side of each line of the rule for the rows per lane of the
    listed tile: the rows taken, labels and counts against every seed."""
    import torch
    inst = S.custom(dim, n, grid, seed=n, sigma=0.2)
    w = np.random.default_rng(n).uniform(-0.2, 0.2, n) * n ** (-2.0 / dim)
    prob, wd = _prob(inst), torch.as_tensor(w, device="cuda:0")
    try:
        ctx.apd_set_culling(False)
        ref = ctx.apd_assign(prob, wd, prec="fp64")
    finally:
        ctx.apd_set_culling(True)
    assert torch.equal(ctx.apd_assign(prob, wd, prec="fp32"), ref)
    assert ctx.apd_last_pass_stats()["pixels_per_lane"] == rows
    for noalloc in (False, True):
        out = ctx.apd_dual_objective_grad(prob, wd, counts=True, noalloc=noalloc)
        assert torch.equal(out["counts"].cpu(), torch.bincount(ref.cpu().long(), minlength=n))


@pytest.mark.parametrize("dim,grid,n", [(2, (2100, 1999), 15000), (3, (130, 121, 129), 29000)])
@pytest.mark.parametrize("spread", [1.0, 0.04])
def test_regions_of_super_tiles(ctx, dim, grid, n, spread):
    """Many super-tiles and seeds: lists by way of regions, the seeds spread
    evenly or so close together that the regions' lists overflow; labels, gaps
    and counts against the passes over every seed."""
    import torch
    inst = S.custom(dim, n, grid, seed=n, sigma=0.2)
    inst.x[:] = np.asarray(inst.lo) + spread * (inst.x - np.asarray(inst.lo))
    w = np.random.default_rng(n).uniform(-0.2, 0.2, n) * n ** (-2.0 / dim) * spread ** 2
    prob, wd = _prob(inst), torch.as_tensor(w, device="cuda:0")
    try:
        ctx.apd_set_culling(False)
        ref, exact = ctx.apd_assign(prob, wd, prec="fp64", rel_gap=True)
    finally:
        ctx.apd_set_culling(True)
    for prec in ("fp32", "bf16", "fp64"):
        assert torch.equal(ctx.apd_assign(prob, wd, prec=prec), ref)
    lab, gap = ctx.apd_assign(prob, wd, prec="fp32", rel_gap=True)
    assert torch.equal(lab, ref) and bool((gap <= exact * (1 + 1e-6) + 1e-12).all())
    out = ctx.apd_dual_objective_grad(prob, wd, counts=True)
    assert torch.equal(out["counts"].cpu(), torch.bincount(ref.cpu().long(), minlength=n))


@pytest.mark.parametrize("dim,grid", [(2, (64, 33)), (3, (32, 9, 17))])
@pytest.mark.parametrize("n", [2, 15, 16, 17, 33, 60, 64, 65, 90])
def test_moments_by_the_cells_of_a_tile(ctx, dim, grid, n):
    """Few to many cells in a tile (groups of 16 on the matrix cores, up to 64
    cells per tile there): counts, gradient and centroids of both tiers and
    tile shapes against the oracle."""
    import torch
    inst = S.custom(dim, n, grid, seed=n, sigma=0.2)
    w = np.random.default_rng(n).uniform(-0.2, 0.2, n) * n ** (-2.0 / dim)
    prob, wd = _prob(inst), torch.as_tensor(w, device="cuda:0")
    ev = O.evaluate(inst, w)
    try:
        for prec, ppl in (("fp32", 4), ("fp32", 8), ("bf16", 4), ("bf16", 8)):
            ctx.apd_set_pixels_per_lane(ppl)
            out = ctx.apd_dual_objective_grad(prob, wd, prec=prec, counts=True, centroids=True)
            np.testing.assert_array_equal(out["counts"].cpu().numpy(), ev.counts)
            np.testing.assert_array_equal(out["grad"].cpu().numpy(), ev.grad)
            np.testing.assert_allclose(out["centroids"].cpu().numpy(), ev.centroids, rtol=0, atol=1e-13)
            assert out["g"] == pytest.approx(ev.g, rel=1e-12, abs=1e-15)
    finally:
        ctx.apd_set_pixels_per_lane(0)


@pytest.mark.parametrize("dim,grid", [(2, (64, 33)), (3, (17, 9, 33))])
@pytest.mark.parametrize("n", [1, 3, 95, 96, 97, 255, 258, 700, 3000])
def test_tile_scans_by_the_number_of_candidates(ctx, dim, grid, n):
    """One candidate, one staged chunk of a tile, several, and every seed for
    want of room in the list, short and long scans over every seed: labels,
    counts and the certified gaps of both tile shapes against the oracle."""
    import torch
    inst = S.custom(dim, n, grid, seed=n, sigma=0.2)
    w = np.random.default_rng(n).uniform(-0.2, 0.2, n) * n ** (-2.0 / dim)
    prob, wd = _prob(inst), torch.as_tensor(w, device="cuda:0")
    ref, best, second = O.assign(inst, w)
    ctx.apd_set_variant(1)  # over every seed, the vector tile at any number
    try:
        for ppl in (4, 8):
            ctx.apd_set_pixels_per_lane(ppl)
            for lists in (True, False):
                ctx.apd_set_culling(lists)
                np.testing.assert_array_equal(ctx.apd_assign(prob, wd, prec="fp32").cpu().numpy(), ref)
                if n > 1:
                    lab, gap = ctx.apd_assign(prob, wd, prec="fp32", rel_gap=True)
                    np.testing.assert_array_equal(lab.cpu().numpy(), ref)
                    rel = (second - best) / (second + w.max())
                    assert np.all(gap.cpu().numpy() <= rel * (1 + 1e-6) + 1e-12)
                out = ctx.apd_dual_objective_grad(prob, wd, counts=True)
                np.testing.assert_array_equal(out["counts"].cpu().numpy(), np.bincount(ref, minlength=n))
    finally:
        ctx.apd_set_pixels_per_lane(0)
        ctx.apd_set_culling(True)
        ctx.apd_set_variant(2)


@pytest.mark.parametrize("dim,grid", [(2, (64, 33)), (3, (32, 9, 17))])
@pytest.mark.parametrize("n", [2, 17, 64, 65, 300])
def test_weighted_moments_by_the_cells_of_a_tile(ctx, dim, grid, n):
    """Pixel weights over the whole range of a byte, few to many cells in a
    tile: counts exactly, gradient, objective and centroids, both tile shapes
    and the static-scratch evaluation, against the oracle."""
    import torch
    q = np.random.default_rng(n).integers(0, 256, grid).astype(np.uint8)
    q.reshape(-1)[:70] = 255
    inst = S.masked(S.custom(dim, n, grid, seed=n, sigma=0.2), q)
    w = np.random.default_rng(n).uniform(-0.2, 0.2, n) * n ** (-2.0 / dim)
    prob, wd = _prob(inst), torch.as_tensor(w, device="cuda:0")
    ev = O.evaluate(inst, w)
    try:
        for ppl, noalloc in ((0, False), (4, False), (8, False), (0, True)):
            ctx.apd_set_pixels_per_lane(ppl)
            out = ctx.apd_dual_objective_grad(prob, wd, counts=True, centroids=True, noalloc=noalloc)
            np.testing.assert_array_equal(out["counts"].cpu().numpy(), ev.counts)
            np.testing.assert_allclose(out["grad"].cpu().numpy(), ev.grad, rtol=0, atol=1e-15)
            np.testing.assert_allclose(out["centroids"].cpu().numpy(), ev.centroids, rtol=0, atol=1e-13)
            assert out["g"] == pytest.approx(ev.g, rel=1e-12, abs=1e-15)
    finally:
        ctx.apd_set_pixels_per_lane(0)


@pytest.mark.parametrize("S_", [1, 15, 16, 17, 127, 129, 513, 4095, 4097])
def test_network_by_the_number_of_samples(ctx, S_):
    """Blocks of 16 samples, slices of the samples and chunks of 128, the
    features at an address that is a multiple of 4 bytes only: output, loss,
    gradient and one Adam step against the FP64 reference.  Every value passes
    through at most four sums of 128 terms or of a slice of the samples, each
    rounding 2^-24 of the sum of magnitudes: 2e-4 of the largest value."""
    import torch
    import paper_2403_03571_amd as apd
    from oracle import mlp
    rng = np.random.default_rng(S_)
    p0 = (mlp.init_params(5) + 0.01 * rng.standard_normal(mlp.n_params())).astype(np.float32)
    X = rng.standard_normal((S_, mlp.N_FEAT)).astype(np.float32)
    t = rng.standard_normal(S_).astype(np.float32)
    raw = torch.zeros(1 + X.size, dtype=torch.float32, device="cuda:0")
    raw[1:] = torch.as_tensor(X.reshape(-1), device="cuda:0")
    Xd, td = raw[1:].view(S_, mlp.N_FEAT), torch.as_tensor(t, device="cuda:0")
    net = apd.WarmStart(ctx, p0)
    P = p0.astype(np.float64)
    yr, _ = mlp.forward(P, X.astype(np.float64))
    assert np.abs(net.forward(Xd).cpu().numpy() - yr).max() <= 2e-4 * np.abs(yr).max()
    loss, g = net.loss_grad(Xd, td)
    lr_, gr = mlp.loss_and_grad(P, X.astype(np.float64), t.astype(np.float64))
    assert loss == pytest.approx(lr_, rel=2e-4)
    assert np.abs(g.cpu().numpy() - gr).max() <= 2e-4 * np.abs(gr).max()
    # Adam's first step moves a parameter by lr g / (|g| + 1e-8 sqrt(1 - 0.999))
    assert net.train_step(Xd, td, 1e-3) == loss
    gd = g.cpu().numpy().astype(np.float64)
    want = P - 1e-3 * gd / (np.abs(gd) + 1e-8)
    assert np.abs(net.params() - want).max() <= 1e-6


@pytest.mark.parametrize("dim,grid", [(2, (90, 70)), (3, (21, 18, 25))])
@pytest.mark.parametrize("power", [1, 2, 3, 4])
@pytest.mark.parametrize("n", [5, 70, 300, 3000])
def test_fp64_lists(ctx, dim, grid, power, n):
    """The double tier over candidate lists against the oracle and against
    itself over every seed: all powers, pixel weights, exact ties, and a box whose
    scale is outside single precision's range (lists off there)."""
    import torch
    for scale in (1.0, 1e-20):
        inst = S.custom(dim, n, grid, seed=n + power, sigma=0.3, lo=(0.0,) * dim, hi=(scale,) * dim)
        inst.power = power
        inst.x[1], inst.A[1] = inst.x[0], inst.A[0]
        r = 0.5 * scale * n ** (-1.0 / dim)
        w = np.random.default_rng(n).uniform(-0.3, 0.3, n) * r ** power
        w[1] = w[0]
        masked = S.masked(inst, S.disk_weights(grid, inst.lo, inst.hi, (0.5 * scale,) * dim, 0.45 * scale))
        masked.power = power
        wd = torch.as_tensor(w, device="cuda:0")
        for case in (inst, masked):
            prob = _prob(case)
            ref, _, _ = O.assign(case, w)
            outs = []
            for culling in (True, False):
                ctx.apd_set_culling(culling)
                try:
                    np.testing.assert_array_equal(ctx.apd_assign(prob, wd, prec="fp64").cpu().numpy(), ref)
                    outs.append(ctx.apd_dual_objective_grad(prob, wd, prec="fp64", counts=True, centroids=True))
                finally:
                    ctx.apd_set_culling(True)
            outs.append(ctx.apd_dual_objective_grad(prob, wd, prec="fp64", counts=True, centroids=True, noalloc=True))
            ev = O.evaluate(case, w)
            for out in outs:
                assert out["g"] == outs[0]["g"] and out["maxrel"] == outs[0]["maxrel"]
                assert out["g"] == pytest.approx(ev.g, rel=1e-12, abs=1e-15 * scale ** (power + dim))
                np.testing.assert_array_equal(out["counts"].cpu().numpy(), ev.counts)
                np.testing.assert_array_equal(out["grad"].cpu().numpy(), ev.grad)


@pytest.mark.parametrize("n", [1, 2, 5, 16, 17, 18, 65, 1280, 4096, 4097])
def test_features_by_the_number_of_seeds(ctx, n):
    """Fewer seeds than neighbours, a lane holding many of the nearest (seeds
    64 apart in number in one tight cluster), equal distances, and the pooled
    deficits by one block or a launch per hop: against the reference, to the
    FP32 rounding of the features (2^-24) and of sums of 16 doubles."""
    import paper_2403_03571_amd as apd
    from oracle import mlp
    inst = S.custom(2, n, 48, seed=n, sigma=0.3)
    if n == 1280:
        inst.x[::64] = 0.5 + 1e-3 * np.random.default_rng(0).random((20, 2))
    if n == 65:
        inst.x[:] = np.stack(np.meshgrid(np.arange(13) / 16 + 0.125, np.arange(5) / 8 + 0.25), -1).reshape(-1, 2)
    net = apd.WarmStart(ctx, mlp.init_params(0))
    F = net.features(_prob(inst)).cpu().numpy()
    d = mlp.deficit(inst.n, O.evaluate(inst, np.zeros(inst.n)).grad)
    ref = mlp.features(inst.x, inst.A, inst.v, inst.lo, inst.hi, d=d)
    np.testing.assert_allclose(F, ref, rtol=2e-6, atol=1e-6)
