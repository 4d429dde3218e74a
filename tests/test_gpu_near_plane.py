"""Gaussians just past the near plane whose centres project 1e3 to 1e5 pixels
off the image: their parameters' gradients against FP64.

The map from the nine screen-space sums to the parameters multiplies rounding
there by 1e3 and more (the sums of q d d^T are almost of rank one, and the
inverse covariance on both sides takes the large part out), so neither the
order of the additions nor FP32 storage of the sums is harmless.  The bound is
that of FP32 sums: 16 units in the last place of each sum's absolute terms,
pushed through the magnitudes of the Jacobian: up to many times the gradient of
these Gaussians, and a few 1e-4 of the others'."""
import numpy as np
import pytest
import torch

import synth
from oracle import binning, project, project_bwd, render
from oracle.params import RasterParams
from support import splat_as_oracle, splat_record

pytestmark = pytest.mark.gpu

RP = RasterParams()
NEAR, FAR = 24, 300
W, H, F = 160, 96, 300.0


def scene():
    rng = np.random.default_rng(31)
    p = synth.gaussians(NEAR + FAR, 31, logscale_mean=-3.3).astype(np.float64)
    cam = synth.look_at((2.4, -1.1, 1.3), fx=F, fy=F, width=W, height=H)
    tz = rng.uniform(0.205, 0.25, NEAR)
    r = 10 ** rng.uniform(3, 5, NEAR)
    phi = rng.uniform(0, 2 * np.pi, NEAR)
    t = np.stack([r * np.cos(phi) * tz / F, r * np.sin(phi) * tz / F, tz])
    p[0:3, :NEAR] = cam.R.T @ (t - cam.t[:, None])
    p[3:6, :NEAR] = np.log(rng.uniform(0.07, 0.14, (3, NEAR)))
    p[10, :NEAR] = rng.normal(-1, 0.5, NEAR)
    # SH colour within its clamp at this distance
    p[11:, :NEAR] *= 0.5
    return p.astype(np.float32), cam


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


def reference():
    p, cam = scene()
    pr = project.project(p, cam, RP)
    rec = splat_record(pr)
    q = splat_as_oracle(pr, rec)
    _, sv, ranges = binning.bin_and_sort(pr)
    xs, ys = render.dense_pixels(W, H)
    ref = render.render_pixels(q, sv, ranges, xs, ys, RP)
    g = np.random.default_rng(3).normal(size=(xs.size, 3)) * 1e-3
    g[ref["flag"]] = 0.0
    g2d, g2d_abs = render.render_pixels_bwd(q, sv, ranges, xs, ys, g, RP, with_abs=True)
    grad = project_bwd.project_bwd(p, cam, pr, g2d, RP)
    scale = np.zeros_like(grad)
    for k in range(9):
        e = np.zeros((9, p.shape[1]))
        e[k] = 1.0
        scale += np.abs(project_bwd.project_bwd(p, cam, pr, e, RP)) * g2d_abs[k][None, :]
    return p, cam, pr, rec, sv, ranges, xs, ys, ref, g, grad, scale


@pytest.mark.parametrize("variant", ["plain", "density", "deterministic"])
def test_parameter_gradients(variant):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_15924_amd import binding as B
    p, cam, pr, rec, sv, ranges, xs, ys, ref, g, grad, scale = reference()
    n, P, idx = p.shape[1], W * H, ys * W + xs
    out, dl, nc = np.zeros((P, 4), np.float32), np.zeros((P, 4), np.float32), np.zeros(P, np.int32)
    out[idx, :3], out[idx, 3], dl[idx, :3], nc[idx] = ref["rgb"], ref["T"], g, ref["n_contrib"]
    G = torch.zeros((n, 9), device="cuda")
    args = (dev(rec), dev(sv.view(np.int32)), dev(ranges.astype(np.int32)), pr["TX"], pr["TY"], W, H, None, None, None,
            pr["TX"] * pr["TY"], 256, B.raster_params(), dev(out), dev(nc), dev(dl), G)
    if variant == "plain":
        B.tgs_render_bwd(*args)
    elif variant == "density":
        B.tgs_render_bwd_density(*args, torch.zeros(P, device="cuda"), n, torch.zeros((n, 4), device="cuda"))
    else:
        ws = torch.empty(B.tgs_render_bwd_det_workspace_size(sv.size, 256, True), dtype=torch.uint8, device="cuda")
        B.tgs_render_bwd_deterministic(*args, None, None, dev(pr["depth32"]), dev(pr["rect"].T.astype(np.int32)), n,
                                       sv.size, ws)
    got = torch.zeros((59, n), device="cuda")
    clamp = (pr["clamp"].astype(np.uint8) * np.array([[1], [2], [4]], np.uint8)).sum(0).astype(np.uint8)
    B.tgs_project_bwd(dev(p), n, B.camera(cam), B.raster_params(), dev(pr["radius"].astype(np.int32)), dev(clamp), G, got)
    err = np.abs(got.cpu().numpy().astype(np.float64) - grad)
    bound = 1e-4 * np.abs(grad) + 16 * 2.0 ** -23 * scale + 1e-30
    live = np.abs(grad[:11]).max(0) > 0
    near = np.arange(n) < NEAR
    assert (live & near).sum() >= 12 and (live & ~near).sum() > 100
    assert (err <= bound).all(), np.argwhere(err > bound)[:5]
    # what the bound means: the map is ill-conditioned for the near ones only
    size = np.linalg.norm(grad[:11], axis=0)
    rel = np.linalg.norm(bound[:11], axis=0)[live] / size[live]
    assert np.median(rel[near[live]]) > 10 * np.median(rel[~near[live]])
    print(f"bound / gradient: near {np.median(rel[near[live]]):.2g}, others {np.median(rel[~near[live]]):.2g}; "
          f"error / gradient: near {np.median((np.linalg.norm(err[:11], axis=0) / size.clip(1e-300))[live & near]):.2g}, "
          f"others {np.median((np.linalg.norm(err[:11], axis=0) / size.clip(1e-300))[live & ~near]):.2g}")
