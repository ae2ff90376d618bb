"""GPU tests of single kernels and dispatch branches at the sizes where they change, against
the FP64 oracle (gates of conftest: 1e-9 relative plus 1e-12 of the summed magnitudes)."""
import numpy as np
import pytest
import torch

from conftest import FLOOR, REL, newton_step_bound

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    assert torch.cuda.is_available(), "needs a GPU"
    from paper_1801_10277_amd import binding
    return binding


def say(*a):
    print("[case]", *a, flush=True)


def device(a):
    return torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")


@pytest.mark.parametrize("steps", [0, 1, 4])
@pytest.mark.parametrize("hess_mode,rows", [(0, 16), (0, 4), (1, 16)])
def test_newton_elbo_out_is_the_elbo_of_the_returned_point(B, O, synth, steps, hess_mode, rows):
    """celeste_newton's elbo_out is that of the last accepted point (both Hessian modes: the
    pixel-level gradient pass and the full one; 0 steps: the entry point)."""
    f = synth.tiny(S=3, n_bands=2, size=45, side=35, seed=311)
    plan = B.Plan(f)
    plan.set_launch(strip_rows=rows)
    plan.set_hessian_mode(hess_mode)
    for s in range(3):
        say("newton elbo_out steps", steps, "mode", hess_mode, "rows", rows, "source", s)
        th = device(f.theta)
        e, _ = plan.newton(th, [s], steps)
        th = th.cpu().numpy()
        others = [t for t in range(3) if t != s]
        np.testing.assert_array_equal(th[others], f.theta[others])
        if steps == 0:
            np.testing.assert_array_equal(th[s], f.theta[s])
        val, _, _ = O.source_grad(O.Problem(f, th), s)
        ref = val[0] + val[1]
        assert abs(float(e[s]) - ref) <= REL * abs(ref) + FLOOR * abs(val[2]), (s, float(e[s]), ref)


@pytest.mark.parametrize("epochs,mixture", [(1, False), (2, True), (4, False), (4, True)])
def test_source_kernels_over_passes_of_boxes(B, O, synth, epochs, mixture):
    """Gradient, HVP and dense Hessian of sources of 5, 10 and 20 boxes: the kernels that work
    a source's boxes off 16 (finalize) and 10 (Hessian assembly) at a time take one pass, an
    exactly full one, and a second, partial one; with and without the colour-prior mixture."""
    f = synth.sky_region(n_fx=1, n_fy=1, epochs=epochs, S=2, H=24, W=26, overlap=0, max_offset=1.0, seed=317)
    if mixture:
        f = synth.with_color_mixture(f, seed=5)
    n = 43 if mixture else 27
    assert len(f.boxes) == 2 * 5 * epochs
    plan, P = B.Plan(f), O.Problem(f)
    th = device(f.theta)
    v = np.zeros((2, 48))
    v[:, :n] = np.random.default_rng(3).standard_normal((2, n))
    say("source kernels epochs", epochs, "mixture", mixture)
    e, g = (t.cpu().numpy() for t in plan.elbo_grad(th))
    hv, g2 = (t.cpu().numpy() for t in plan.hvp(th, device(v), with_grad=True))
    H = plan.hessian(th, [1, 0]).cpu().numpy()
    e2 = plan.elbo(th).cpu().numpy()
    for s in range(2):
        val, gref, gabs = O.source_grad(P, s)
        href, habs = O.source_hvp(P, s, v[s])
        ref = val[0] + val[1]
        for got in (e[s], e2[s]):
            assert abs(got - ref) <= REL * abs(ref) + FLOOR * abs(val[2]), (s, got, ref)
        for got in (g, g2):
            assert np.all(np.abs(got[s, :n] - gref) <= REL * np.abs(gref) + FLOOR * gabs), s
            np.testing.assert_array_equal(got[s, n:], 0.0)
        assert np.all(np.abs(hv[s, :n] - href) <= REL * np.abs(href) + FLOOR * habs), s
        Href, Habs = O.source_hessian(P, s, with_abs=True)
        assert np.all(np.abs(H[1 - s] - Href) <= REL * np.abs(Href) + FLOOR * Habs), s


@pytest.mark.parametrize("mixture", [False, True])
@pytest.mark.parametrize("radius", [1e-6, 1e-2, 0.5, 40.0])
def test_trust_region_step_at_small_and_large_radii(B, synth, mixture, radius):
    """One Newton step from the smallest radii (the multiplier far above the spectrum) to one
    that leaves the interior step inside: within the derived one-step bound of the oracle's."""
    from oracle import newton as N
    from oracle import oracle as O
    O.build()
    f = synth.tiny(S=4, n_bands=3, size=25, side=15, seed=331)
    if mixture:
        f = synth.with_color_mixture(f, seed=2)
    plan = B.Plan(f)
    for s in range(4):
        say("trust region radius", radius, "mixture", mixture, "source", s)
        th = device(f.theta)
        rad = torch.full((4,), radius, dtype=torch.float64, device="cuda")
        _, rad = plan.newton(th, [s], 1, radius=rad)
        bound, row, _, R = newton_step_bound(N, f, f.theta, s, radius)
        diff = np.abs(th.cpu().numpy()[s, :len(row)] - row)
        assert np.all(diff <= bound), (s, float((diff / np.maximum(bound, 1e-300)).max()))
        assert float(rad[s]) == R


@pytest.mark.parametrize("rows", [4, 8, 16])
@pytest.mark.parametrize("eig", [(0.66, 0.66), (0.667, 0.667), (0.667, 4.0), (9.0, 9.0)])
def test_row_factors_at_the_psf_limit(B, O, synth, eig, rows):
    """ELBO, gradient, total ELBO and dense Hessian with PSF eigenvalues just below 2/3 px^2
    (row-ratio recurrence), just above it (row factors at their sharpest, also rotated by 45
    degrees) and far above, on boxes that reach tens of widths from the centre."""
    f = synth.tiny(S=3, n_bands=2, size=71, side=61, seed=347)
    a, b = eig
    f.img_psf[:, :, 3] = f.img_psf[:, :, 5] = 0.5 * (a + b)
    f.img_psf[:, :, 4] = 0.5 * (b - a)
    plan, P = B.Plan(f), O.Problem(f)
    plan.set_launch(strip_rows=rows)
    th = device(f.theta)
    say("row factors eig", eig, "rows", rows)
    e, g = (t.cpu().numpy() for t in plan.elbo_grad(th))
    H = plan.hessian(th, [0, 1, 2]).cpu().numpy()
    np.testing.assert_allclose(float(plan.total_elbo(th)[0]), O.total_elbo(P), rtol=1e-11)
    for s in range(3):
        val, gref, gabs = O.source_grad(P, s)
        ref = val[0] + val[1]
        assert abs(e[s] - ref) <= REL * abs(ref) + FLOOR * abs(val[2]), s
        assert np.all(np.abs(g[s, :27] - gref) <= REL * np.abs(gref) + FLOOR * gabs), s
        Href, Habs = O.source_hessian(P, s, with_abs=True)
        assert np.all(np.abs(H[s] - Href) <= REL * np.abs(Href) + FLOOR * Habs), s


# items of 16, 8 and 4 rows: 5, 5, 10; 90, 150, 275; 285, 495, 910; 520, 940, 1730; 850, 1485, 2800;
# 20380, 36485, 67880 (at most 1024: one wave per SIMD; at most 16384: 16)
@pytest.mark.parametrize("S,side,rows_eval,rows_newton", [(1, 60, 4, 4), (8, 160, 4, 4), (20, 200, 4, 4),
                                                          (30, 240, 8, 8), (50, 300, 16, 8),
                                                          (1100, 1000, 16, 16)])
def test_a_new_plan_takes_the_strip_height_of_its_size(B, synth, S, side, rows_eval, rows_newton):
    """A new plan's evaluations and its Newton, Hessian and sweep passes equal, bit for bit,
    those of a plan set to the height that the plan's size calls for; its reported items stay
    those of 16 rows, and setting the launch sets every pass."""
    f = synth.sdss_field(S, H=side, W=side, seed=353)
    new, ev, nt = B.Plan(f), B.Plan(f), B.Plan(f)
    assert new.info()["strip_rows"] == 16
    say("strip heights", S, "sources", new.info()["n_items"], "items")
    ev.set_launch(strip_rows=rows_eval)
    nt.set_launch(strip_rows=rows_newton)
    th = device(f.theta)
    v = device(np.random.default_rng(5).standard_normal(f.theta.shape))
    act = torch.zeros(S, dtype=torch.uint8, device="cuda")
    act[: (S + 1) // 2] = 1
    src = np.arange(0, S, 1 + S // 20, dtype=np.int32)

    def evaluations(p):
        out = [*p.elbo_grad(th), *p.elbo_grad_noalloc(th, active=act), p.elbo(th, active=act),
               p.total_elbo(th)]
        if S < 100:
            out += p.elbo_grad(th, mode=B.CELESTE_PLAIN)
        return out + list(p.hvp(th, v, with_grad=True))

    def steps(p):
        t = th.clone()
        e, r = p.newton(t, src, 2)
        t2 = th.clone()
        bp, bs = p.color_batches(3)
        return [p.hessian(th, src), t, e, r, p.sweep(t2, bp, bs, 1, B.tr_params(newton_steps=1)), t2]

    for a, b in zip(evaluations(new) + steps(new), evaluations(ev) + steps(nt)):
        np.testing.assert_array_equal(a.cpu().numpy(), b.cpu().numpy())
    new.set_launch()
    ev.set_launch()
    for a, b in zip(evaluations(new) + steps(new), evaluations(ev) + steps(ev)):
        np.testing.assert_array_equal(a.cpu().numpy(), b.cpu().numpy())


@pytest.mark.parametrize("rows,chunk,dynamic", [(4, 64, 0), (8, 192, 1), (16, 64, 0), (16, 1024, 1)])
@pytest.mark.parametrize("eig,mode", [((0.66, 0.66), 2), ((0.667, 0.667), 2), ((0.667, 4.0), 2), ((9.0, 9.0), 2),
                                      ((9.0, 9.0), 1)])
def test_hvp_over_stored_values(B, O, synth, eig, mode, rows, chunk, dynamic):
    """Hessian-vector products at the edges of the tangent pass over stored values (PSF
    eigenvalues from 2/3 px^2, the render that stores them) and of the recurrence it leaves
    the rest to: gradient and product per entry, boxes with a last strip of one row, items of
    one strip per lane and of several, one unmasked and one masked pixel."""
    f = synth.tiny(S=3, n_bands=2, size=71, side=49, seed=359)
    a, b = eig
    f.img_psf[:, :, 3] = f.img_psf[:, :, 5] = 0.5 * (a + b)
    f.img_psf[:, :, 4] = 0.5 * (b - a)
    f.x[37::211] = np.nan
    plan, P = B.Plan(f), O.Problem(f)
    plan.set_launch(strip_rows=rows, chunk=chunk, dynamic=dynamic, render_mode=mode)
    v = np.random.default_rng(11).standard_normal(f.theta.shape)
    say("hvp stored", eig, mode, rows, chunk)
    hv, g = (t.cpu().numpy() for t in plan.hvp(device(f.theta), device(v), with_grad=True))
    for s in range(3):
        _, gref, gabs = O.source_grad(P, s)
        href, habs = O.source_hvp(P, s, v[s])
        n = len(gref)
        assert np.all(np.abs(g[s, :n] - gref) <= REL * np.abs(gref) + FLOOR * gabs), s
        assert np.all(np.abs(hv[s, :n] - href) <= REL * np.abs(href) + FLOOR * habs), s


@pytest.mark.parametrize("n", [1, 64, 65, 256, 257, 1024, 1025])
def test_validation_of_lists_of_one_block_and_more(B, synth, n):
    """A bad row of a listed source refuses the call wherever it stands in the list, one of an
    unlisted source does not, and the next call starts with a clear status."""
    f = synth.tiny(S=1030, n_bands=1, size=64, side=5, seed=367)
    plan = B.Plan(f)
    src = np.arange(n, dtype=np.int32)
    say("validate", n)
    for bad in (0, n - 1, 1029):
        th = f.theta.copy()
        th[bad, 6] = 1.5
        if bad < n:
            with pytest.raises(B.CelesteError):
                plan.newton(device(th), src, 0)
        else:
            plan.newton(device(th), src, 0)
        plan.newton(device(f.theta), src, 0)


@pytest.mark.parametrize("S", [3, 64, 65, 66, 140])
@pytest.mark.parametrize("rows,chunk", [(4, 64), (8, 192), (16, 64)])
def test_backgrounds_of_crowded_boxes(B, O, synth, S, rows, chunk):
    """Dense Hessians over stored backgrounds and the total ELBO where boxes meet up to one, two
    and three waves' worth of other boxes, some on their edges only: each entry within its
    gate of the oracle's."""
    f = synth.tiny(S=S, n_bands=1, size=48, side=27, seed=373)
    plan, P = B.Plan(f), O.Problem(f)
    plan.set_launch(strip_rows=rows, chunk=chunk)
    src = sorted({0, S // 2, S - 1})
    say("crowded", S, "boxes", plan.info()["n_nbr"], "neighbours")
    H = plan.hessian(device(f.theta), src).cpu().numpy()
    for j, s in enumerate(src):
        Href, Habs = O.source_hessian(P, s, with_abs=True)
        assert np.all(np.abs(H[j] - Href) <= REL * np.abs(Href) + FLOOR * Habs), s
    np.testing.assert_allclose(float(plan.total_elbo(device(f.theta))[0]), O.total_elbo(P), rtol=1e-11)


@pytest.mark.parametrize("rows", [None, 4, 8, 16])
@pytest.mark.parametrize("sigma", [0.1, 0.2, 0.255, 0.26, 0.35, 0.55, 0.56])
def test_narrow_psfs_at_every_strip_height(B, O, synth, sigma, rows):
    """ELBO (batched and plain), gradient, Hessian-vector product, total ELBO and dense Hessian
    (both modes) with PSFs down to the narrowest accepted (0.1 px), the centre near the last row
    of a strip of any height, past it, and between rows: a component whose value underflows at
    a strip's top row must not vanish from the strip.  Both sides of the widths from which
    strips of 8 and of 16 rows are walked as such (7/27 and 15/27 px); below, a plan takes no
    more work items than at the height asked for."""
    f = synth.tiny(S=3, n_bands=2, size=51, side=33, seed=379)
    f.img_psf[:, :, 3] = f.img_psf[:, :, 5] = sigma ** 2
    f.img_psf[:, :, 4] = 0.0
    for s, past in enumerate((0.05, 0.45, -0.3)):
        box = f.boxes[f.patch_ptr[s]]
        f.theta[s, 0:2] = box[2] + 15 + past, box[1] + 15 + past
    plan, P = B.Plan(f), O.Problem(f)
    if rows:
        plan.set_launch(strip_rows=rows)
        info, (h, w) = plan.info(), np.asarray(f.boxes)[:, 3:5].T
        walked = min(rows, 16 if sigma > 15 / 27 else 8 if sigma > 7 / 27 else 4)
        assert plan.work_counts(device(f.theta))["strips"] == np.sum(w * -(-h // walked))
        assert (info["chunk"], info["strip_rows"]) == (64, rows)
        assert info["n_items"] <= np.sum(-(-w * -(-h // rows) // 64))
    th = device(f.theta)
    v = np.random.default_rng(13).standard_normal(f.theta.shape)
    say("narrow psf", sigma, "rows", rows)
    e, g = (t.cpu().numpy() for t in plan.elbo_grad(th))
    e2, g2 = (t.cpu().numpy() for t in plan.elbo_grad(th, mode=B.CELESTE_PLAIN))
    hv = plan.hvp(th, device(v)).cpu().numpy()
    H = [plan.hessian(th, [0, 1, 2]).cpu().numpy()]
    plan.set_hessian_mode(1)
    H.append(plan.hessian(th, [0, 1, 2]).cpu().numpy())
    np.testing.assert_allclose(float(plan.total_elbo(th)[0]), O.total_elbo(P), rtol=1e-11)
    for s in range(3):
        val, gref, gabs = O.source_grad(P, s)
        ref = val[0] + val[1]
        href, habs = O.source_hvp(P, s, v[s])
        Href, Habs = O.source_hessian(P, s, with_abs=True)
        for got in (e[s], e2[s]):
            assert abs(got - ref) <= REL * abs(ref) + FLOOR * abs(val[2]), s
        for got in (g[s, :27], g2[s, :27]):
            assert np.all(np.abs(got - gref) <= REL * np.abs(gref) + FLOOR * gabs), s
        assert np.all(np.abs(hv[s, :27] - href) <= REL * np.abs(href) + FLOOR * habs), s
        for got in H:
            assert np.all(np.abs(got[s] - Href) <= REL * np.abs(Href) + FLOOR * Habs), s


@pytest.mark.parametrize("S,side,rows", [(1, 60, 4), (8, 160, 4), (30, 240, 8), (50, 300, 16)])
def test_work_counts_are_those_of_the_strips_walked(B, synth, S, side, rows):
    """The work counts of a new plan are those of a plan set to the strip height that its
    evaluations take."""
    f = synth.sdss_field(S, H=side, W=side, seed=353)
    new, at = B.Plan(f), B.Plan(f)
    at.set_launch(strip_rows=rows)
    say("work counts", S, "rows", rows)
    assert new.work_counts(device(f.theta)) == at.work_counts(device(f.theta))


@pytest.mark.parametrize("S,side", [(8, 160), (50, 300), (500, 860), (1100, 1000)])
def test_tuning_the_gradient_leaves_the_newton_passes_their_strips(B, synth, S, side):
    """celeste_autotune times the batched gradient: afterwards the dense Hessians, Newton steps
    and sweeps of a plan still take the strips its size calls for (bit for bit a new plan's
    results, as long as the tuned render mode keeps the stored values they start from), a
    second tuning included; set_launch then sets every pass."""
    f = synth.sdss_field(S, H=side, W=side, seed=353)
    th = device(f.theta)
    src = np.arange(0, S, 1 + S // 20, dtype=np.int32)

    def steps(p):
        t = th.clone()
        e, r = p.newton(t, src, 2)
        t2 = th.clone()
        bp, bs = p.color_batches(3)
        p.sweep(t2, bp, bs, 1, B.tr_params(newton_steps=1))   # (its trace adds up the tuned tiles)
        return [x.cpu().numpy() for x in (p.hessian(th, src), t, e, r, t2)]

    new, tuned, again = B.Plan(f), B.Plan(f), B.Plan(f)
    ref = steps(new)
    for _ in range(2):
        say("tune", S, "sources")
        ms = tuned.autotune(th, reps=2)
        info = tuned.info()
        say("tuned", ms, info)
        for a, b in zip(steps(tuned), ref):
            if info["render_mode"] in (2, 3):
                np.testing.assert_array_equal(a, b)
            else:
                np.testing.assert_allclose(a, b, rtol=1e-9, atol=1e-9 * np.abs(b).max())
    tuned.set_launch()
    again.set_launch()
    for a, b in zip(steps(tuned), steps(again)):
        np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("mixture", [False, True])
@pytest.mark.parametrize("S", [1, 1023, 1025, 4097, 5200])
def test_total_elbo_of_few_and_many_sources_a_block(B, O, synth, S, mixture):
    """The total's KL terms where a block of the reduction gets none, one, a wave's share less
    or more one, and several passes of its waves: within the summation error of the oracle's."""
    f = synth.tiny(S=S, n_bands=1, size=90, side=3, seed=383)
    if mixture:
        f = synth.with_color_mixture(f, seed=3)
    say("total", S, "mixture", mixture)
    np.testing.assert_allclose(float(B.Plan(f).total_elbo(device(f.theta))[0]), O.total_elbo(O.Problem(f)), rtol=1e-11)
