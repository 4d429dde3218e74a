"""The stage calls over several views (sampler, forward, loss, error maps,
backward) against the single-view calls: views of different sizes and sample
counts (so different workgroup kinds), dense views, tile subsets, more views
than one launch takes; and whole training steps, stage by stage together
against view by view."""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu

SIZES = [(150, 107), (256, 256), (97, 33), (64, 160), (256, 80)]


@pytest.fixture(scope="module")
def B():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_15924_amd import binding
    binding.lib()
    return binding


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


def same(a, b):
    return torch.equal(a.view(torch.uint8), b.view(torch.uint8))


def camera(k, size):
    W, H = size
    return synth.look_at((2.7 * np.cos(k), 2.7 * np.sin(k), 0.4), fx=1.15 * max(size), fy=1.15 * max(size), width=W,
                         height=H)


# rates: permille of the pixels per view (None: dense); tiles: permille drawn (-1: all)
@pytest.mark.parametrize("rates,tiles,density,structure", [
    ([250] * 3, -1, False, 0), ([250] * 5, 400, True, 0), ([250, 250, 400, 700, 250], 400, False, 1),
    ([None] * 3, -1, False, 0), ([None, 250, 250, None, 60], -1, False, 0)])
def test_stages_equal_single_views(B, rates, tiles, density, structure):
    from paper_2606_15924_amd.pipeline import StepConfig, ViewBuffers
    n = 3000
    params = dev(synth.gaussians(n, 5, logscale_mean=-3.0))
    rp, lp = B.raster_params(), B.loss_params(structure=structure)
    n_sel = -1 if tiles < 0 else 12
    cfg = StepConfig(n_tiles_sel=n_sel)
    totals = [torch.zeros(2, dtype=torch.int64, device="cuda") for _ in range(2)]
    stats = [torch.zeros((n, 4), device="cuda") for _ in range(2)]
    touched = [torch.zeros(n, dtype=torch.uint8, device="cuda") for _ in range(2)]
    counters = [torch.zeros((2, B.COUNTER_SLOTS), dtype=torch.int64, device="cuda") for _ in range(2)]
    sets = [[], []]   # single calls, calls over the views
    for k, rate in enumerate(rates):
        W, H = SIZES[k]
        gt = dev(synth.image(H, W, k).astype(np.float32))
        for s in sets:
            vb = ViewBuffers(n, W, H, None if rate is None else max(1, 256 * rate // 1000), n_sel, "cuda")
            E, A = dev(synth.error_map(H, W, 40 + k).view(np.int16)), dev(synth.age_map(H, W, 50 + k).view(np.int16))
            for t in (vb.out, vb.dL, vb.err, vb.lam, vb.tile_loss, vb.state):
                t.fill_(-1.0)
            s.append((vb, gt, E, A, k + 3))
    def sparse(recs):
        return B.views_array([r for r, (vb, *_) in zip(recs, sets[1]) if not vb.dense])
    recs = [vb.record(v, gt, E, A) for vb, gt, E, A, v in sets[1]]
    for vb, gt, E, A, v in sets[0]:
        if not vb.dense:
            vb.sample(E, A, cfg, 2, v, totals[0])
    # one sample count per call: the views share their parameters
    for n_pix in sorted({vb.n_pix for vb, *_ in sets[1] if not vb.dense}):
        part = [r for r, (vb, *_) in zip(recs, sets[1]) if not vb.dense and vb.n_pix == n_pix]
        sp = next(vb for vb, *_ in sets[1] if not vb.dense and vb.n_pix == n_pix).sample_params(cfg, 2, 0)
        B.tgs_sample_views(B.views_array(part), sp, totals[1])
    for (a, *_), (b, *_) in zip(*sets):
        if not a.dense:
            m = int(a.tile_off[-1])
            assert same(a.valid_tiles, b.valid_tiles) and same(a.tile_off, b.tile_off)
            assert same(a.tile_slot, b.tile_slot) and same(a.pix[:m], b.pix[:m])
    assert torch.equal(*totals)
    totals[0] += 7   # dense views only: any count
    totals[1] += 7
    for s in sets:
        for k, (vb, *_) in enumerate(s):
            vb.project(params, B.camera(camera(k, SIZES[k])), rp)
            vb.bin_sort(alpha_min=rp.alpha_min)
    # the lists may have been reallocated
    recs = [vb.record(v, gt, E, A) for vb, gt, E, A, v in sets[1]]
    both = B.views_array(recs)
    for vb, *_ in sets[0]:
        vb.render_fwd(rp, counters[0])
    B.tgs_render_fwd_views(both, rp, counters[1])
    assert torch.equal(counters[0].sum(1), counters[1].sum(1))
    for vb, gt, *_ in sets[0]:
        vb.loss(gt, totals[0], lp)
    B.tgs_loss_views(both, totals[1], lp)
    for vb, gt, E, A, v in sets[0]:
        if not vb.dense:
            vb.ema_age(E, A, 0.4)
    B.tgs_ema_age_update_views(sparse(recs), 0.4)
    for vb, *_ in sets[0]:
        vb.render_bwd(rp, zero=False, stats=stats[0] if density else None, touched=touched[0])
    B.tgs_render_bwd_views(both, rp, touched[1], n, stats[1] if density else None)
    for k, ((a, _, Ea, Aa, _), (b, _, Eb, Ab, _)) in enumerate(zip(*sets)):
        for name in ("out", "ncontrib", "dL", "err", "lam", "tile_loss"):
            x, y = getattr(a, name), getattr(b, name)
            if not a.dense and name in ("out", "ncontrib", "dL", "err"):
                m = int(a.tile_off[-1])
                x, y = x[:m], y[:m]
            assert same(x, y), (k, name)
        assert same(Ea, Eb) and same(Aa, Ab), k
        # the same partial sums, at most 112 tiles x 4 batches here, added by
        # atomics in any order: each addition rounds to 2^-24 of a sum that
        # the field's largest value bounds up to a small factor
        tol = 448 * 2.0 ** -24 * 4 * a.g2d.abs().amax(0)
        assert bool(((a.g2d - b.g2d).abs() <= tol).all()), k
    assert torch.equal(*touched) and int(touched[0].sum()) > 0
    if density:
        tol = 448 * len(rates) * 2.0 ** -24 * 4 * stats[0].abs().amax(0)
        assert bool(((stats[0] - stats[1]).abs() <= tol).all())


def test_maps_shared_by_two_views_are_refused(B):
    from paper_2606_15924_amd.pipeline import ViewBuffers
    vb = [ViewBuffers(10, 64, 48, 64, -1, "cuda") for _ in range(2)]
    E, A = (torch.zeros((48, 64), dtype=torch.int16, device="cuda") for _ in range(2))
    with pytest.raises(RuntimeError):
        B.tgs_ema_age_update_views(B.views_array([v.record(0, E, E, A) for v in vb]), 0.4)


@pytest.mark.parametrize("views,kw", [([0, 1, 2], {}), ([0, 1, 0], {}), ([2, 1], {"density_stats": True}),
                                      ([0, 1, 2, 3, 4], {"n_tiles_sel": 20}), ([0, 2, 1], {"rate_permille": None}),
                                      ([1, 0], {"deterministic": True}),
                                      ([0, 1, 2], {"prefix_fraction": 0.2}),
                                      ([2, 0, 1, 2], {"prefix_fraction": 0.05, "n_tiles_sel": 11}),
                                      ([1, 2, 0], {"fuse_optimizer": False, "density_stats": True}),
                                      ([0, 3, 0], {"n_tiles_sel": 9, "learned_tiles": True})])
def test_second_step_equals_views_in_turn(B, views, kw):
    """The second step of a slot runs its views together on one stream; with
    view streams they run view by view.  The first step's images come from
    equal parameters, so the second step's samples and ages are equal bit for
    bit; its images hang on float atomics in the first update: 1e-3 of the
    value range, where one update moves a colour by about 1e-2."""
    from paper_2606_15924_amd.pipeline import StepConfig, Trainer
    n = 2000
    p = synth.gaussians(n, 8, logscale_mean=-3.0)
    sizes = [SIZES[0]] * 5 if kw.get("learned_tiles") else SIZES
    cams = [camera(k, s) for k, s in enumerate(sizes)]
    got = []
    for streams in (1, 2):
        gts = [dev(synth.image(h, w, k).astype(np.float32)) for k, (w, h) in enumerate(sizes)]
        E = [dev(synth.error_map(h, w, 60 + k).view(np.int16)) for k, (w, h) in enumerate(sizes)]
        A = [dev(synth.age_map(h, w, 70 + k).view(np.int16)) for k, (w, h) in enumerate(sizes)]
        tr = Trainer(dev(p.copy()), cams, gts, StepConfig(**{"rate_permille": 250, "view_streams": streams,
                                                             "fuse_views": streams == 1 and kw.get("fuse_optimizer", True), **kw}), E=E, A=A)
        for _ in range(2):
            used = tr.step(views)
        torch.cuda.synchronize()
        tr.check_counts(wait_all=True)
        got.append((tr, used, A))
    (ta, ua, Aa), (tb, ub, Ab) = got
    for k, (a, b) in enumerate(zip(ua, ub)):
        m = a.P_cap
        if not a.dense:
            m = int(a.tile_off[-1])
            assert same(a.valid_tiles, b.valid_tiles) and same(a.tile_off, b.tile_off) and same(a.pix[:m], b.pix[:m])
        assert float((a.out[:m] - b.out[:m]).abs().max()) < 1e-3, k
    for x, y in zip(Aa, Ab):
        assert same(x, y)
    assert torch.equal(ta.totals, tb.totals)
    assert abs(ta.loss_value(ua) - tb.loss_value(ub)) < 1e-3
    moved = (ta.params - dev(p)).abs().mean()
    assert float(moved) > 0 and float((ta.params - tb.params).abs().mean()) < 0.02 * float(moved)
