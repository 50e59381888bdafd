"""GPU parity of the HIP path (through the C ABI) with the CPU oracle.

Bit-exact: culling, tiles touched, tile rectangles, depth keys, the projected
means/conics/opacities (one correctly rounded fp32 operation sequence on both
sides), the number of pairs, the sorted per-tile lists, tile ids and ranges.
Images: abs 1e-5 + rel 1e-4 on every pixel whose decisions lie outside the
rounding bound of the oracle's margin; the others (flagged) are counted and
bounded, and get a zero upstream gradient on both sides.
Gradients (the fp32 tolerance of the workload): every element within 1e-3 |ref| + 1e-5 max|ref|
and relative L2 <= 1e-4 per tensor; the decoder paths as stated in MLP_GRADS.
"""
import numpy as np
import pytest

from paper_2609_05255_amd import inputs

import torch

from oracle import oracle as orc
from paper_2609_05255_amd import gsraster as gs
from parity import (GRAD_ELEM_FLOOR, GRAD_ELEM_RTOL, MLP_ATOL, MLP_HALF_ATOL, MLP_GRADS, NEURAL_FLIP, check_grads,
                    compare_image, compare_lists, compare_preprocess, flagged_pixels, grad_stats, lobe_color_atol,
                    report_grads, run_gpu, say, tiny_camera)

pytestmark = pytest.mark.gpu


def check_all(scene, cam, kind="sh3", sh_degree=3, label="", grads=True, capacity=None, max_flagged=None,
              cam_seed=0):
    say("case %s: n=%d %dx%d %s degree %d" % (label, scene.n, cam.width, cam.height, kind, sh_degree))
    latent = kind in ("latent", "neural", "neural_folded")
    # the decoder's operands are binary16: compare with the oracle that rounds them alike
    ref = orc.render(cam, scene, kind=kind, sh_degree=sh_degree, mode="f32", half_act=latent)
    flagged = flagged_pixels(ref["margin"], max_flagged)
    g = None
    if grads:
        g = (inputs.make_upstream_grad(cam.width, cam.height, cam_seed) * ~flagged[None]).astype(np.float32)
        ref["grads"] = orc.render_bwd(cam, scene, ref["pre"], ref["ranges"], ref["values"], g, kind=kind,
                                      sh_degree=sh_degree, mode="f32", half_act=latent)
    gpu = run_gpu(scene, cam, kind, sh_degree, g, capacity=capacity)
    flip = NEURAL_FLIP if kind in ("neural", "neural_folded") else None
    atol = (MLP_HALF_ATOL if latent else
            lobe_color_atol(scene, cam, kind, ref["pre"]["color"], sh_degree) if kind in ("nasg", "nasgabor") else 2e-6)
    compare_preprocess(gpu, ref["pre"], color_atol=atol, flip=flip)
    compare_lists(gpu, ref["values"], ref["tile_of"], ref["ranges"])
    if latent:
        compare_image(gpu, ref["image"], ref["final_T"], ref["n_contrib"], ref["margin"],
                      atol=flip[0] if flip else MLP_HALF_ATOL, rtol=0.0)
        exact = orc.render(cam, scene, kind=kind, sh_degree=sh_degree, mode="f32")
        err = np.abs(gpu["image"] - exact["image"])[:, exact["margin"] > 1.0]
        say("  latent image vs the exact decoder: max abs %.2e" % (err.max() if err.size else 0.0))
        assert err.size == 0 or err.max() <= MLP_ATOL
    else:
        compare_image(gpu, ref["image"], ref["final_T"], ref["n_contrib"], ref["margin"])
    say("  P=%d" % gpu["P"])
    if grads:
        st = grad_stats(gpu["grads"], ref["grads"])
        report_grads(st)
        if kind in ("latent", "neural"):
            check_grads(st, **MLP_GRADS)
        else:
            check_grads(st)
    return gpu, ref


def test_tiny_scene():
    sc = inputs.make_scene("tiny")
    cam = inputs.make_cameras("tiny")[0]
    check_all(sc, cam, label="tiny", max_flagged=0)


@pytest.mark.parametrize("degree", [0, 1, 2])
def test_tiny_scene_lower_sh_degrees(degree):
    sc = inputs.make_scene("tiny")
    check_all(sc, inputs.make_cameras("tiny")[0], sh_degree=degree, label="tiny", max_flagged=0)


def test_ragged_image_with_background():
    # 50x37 pixels: partial edge tiles on both axes; non-black background
    sc = inputs.make_scene("tiny")
    check_all(sc, tiny_camera(50, 37, bg=(0.25, 0.5, 0.75)), label="ragged")


@pytest.mark.parametrize("size", [(16, 16), (17, 9), (300, 20)])
def test_tile_grid_edge_cases(size):
    # one tile (no tile-sort pass), two tiles, and a 19x2 grid
    sc = inputs.make_scene("tiny")
    check_all(sc, tiny_camera(*size), label="grid%dx%d" % size)


def test_more_than_65536_tiles():
    # 4097 x 16 tiles: the tile ids no longer fit 16 bits, so the pair emission
    # and the tile sort carry 32-bit keys (below that they carry 16-bit ones)
    sc = inputs.make_scene("tiny").subset(np.arange(300))
    check_all(sc, tiny_camera(16 * 4097, 256), label="wide", grads=False)


@pytest.mark.parametrize("n,size", [(4097, (4096, 48)), (8193, (4097, 48)), (1 << 20, (64, 4096)),
                                    ((1 << 20) + 1, (64, 4097)), ((1 << 21) + 4097, (320, 240))])
def test_depth_sort_workgroups(n, size):
    # 4, 8 and 12 keys per thread of the depth sort's passes (to 2^20, to 2^21,
    # above), workgroups that are full, hold one key, or end inside a wave; tile
    # grids of 256 and 257 tiles a side, with rectangles packed in 32 bits or
    # gathered; equal depths (ties by index) and culled Gaussians among them
    sc = inputs.make_scene("tiny", n=n)
    sc.means[:, ::3] = np.round(sc.means[:, ::3] * 4) / 4
    sc.means[2, ::11] = -4.0
    cam = tiny_camera(*size)
    sc.log_scales[:] = np.float32(np.log(20.0 / cam.fx) if n < 10000 else np.log(0.1 / cam.fx))
    # the capacity also picks 8 (up to 12 << 20 pairs) or 16 entries per thread of the block sort
    gpu = run_gpu(sc, cam, capacity=1 << 18 if n < 10000 else 1 << 25)
    pre = orc.preprocess(cam, sc)
    values, tiles, ranges = orc.bin_sort(cam, pre)
    compare_lists(gpu, values, tiles, ranges)


@pytest.mark.parametrize("n,size", [(8192 * 1024, (320, 240)), (8192 * 1024 + 1, (320, 240)),
                                    (8192 * 1024 + 1, (64, 4112))])
def test_entry_offsets_of_many_chunks(n, size):
    # up to 8,192 chunks of 1,024 Gaussians every workgroup adds up the totals of the
    # chunks before its own, above that a launch scans them: both sides of the line,
    # with rectangles packed in 32 bits and (257 tiles a side) gathered; 128 copies of
    # the same Gaussians, so that every depth ties, three in four of them culled;
    # device and host mode, a capacity too small
    sc = inputs.make_scene("tiny", n=65537, appearance=("nasg",)).subset(np.arange(n) % 65537)
    sc.means[2, np.arange(n) % 4 != 1] = -4.0
    cam = tiny_camera(*size)
    sc.log_scales[:] = np.float32(np.log(0.1 / cam.fx))
    gpu = run_gpu(sc, cam, "nasg", 0, capacity=1 << 25)
    values, tiles, ranges = orc.bin_sort(cam, orc.preprocess(cam, sc, kind="nasg", sh_degree=0))
    compare_lists(gpu, values, tiles, ranges)
    cs, st, P = gs.camera_struct(cam), gpu["scene_tensors"], gpu["P"]
    for capacity in (P, P - 1):
        fr = gs.Frame(n, cam.width, cam.height, gs.GS_APP_NASG, capacity)
        gs.gs_preprocess(cs, st.gaussians(), st.appearance(gs.GS_APP_NASG, 0), fr.pre, fr.workspace, fr.ws_bytes,
                         sync_pairs=False)
        gs.gs_bin_sort(cs, fr.pre, n, gs.GS_PAIRS_ON_DEVICE, capacity, fr.values, None, fr.ranges, fr.workspace,
                       fr.ws_bytes)
        got = fr.ranges.cpu().numpy().reshape(-1, 2).astype(np.int64)
        if capacity == P:
            assert np.array_equal(got, ranges)
            assert np.array_equal(fr.values.cpu().numpy()[:P].astype(np.int64), values.astype(np.int64))
        else:
            assert not got.any() and int(fr.num_pairs.item()) == P


@pytest.mark.parametrize("n,size", [(1, (64, 64)), (1023, (64, 64)), (1025, (200, 90)), (2049, (200, 90)),
                                    (4097, (1000, 30)), (8193, (330, 200)),
                                    (12288, (330, 200)), (12289, (330, 200)), (24576, (640, 300)), (24577, (640, 300)),
                                    (12288, (4096, 1376)), (20000, (1920, 1080)), (3000, (2064, 2064))])
def test_few_gaussians_binning(n, size):
    # 1 to 12 Gaussians per thread of the sort, 1 to 24 of the search; the largest counts of the one-workgroup
    # depth sort and of the blocks' search, and the next; Gaussians times blocks at,
    # below and above its limit of 2^24; more tiles than it adds up; ties, culled
    # Gaussians, splats of many blocks; device and host mode, a capacity too small
    sc = inputs.make_scene("tiny", n=n)
    sc.means[:, ::3] = np.round(sc.means[:, ::3] * 4) / 4
    sc.means[2, 5::11] = -4.0
    cam = tiny_camera(*size)
    sc.log_scales[:] = np.float32(np.log(8.0 / cam.fx))
    sc.log_scales[:, ::97] = np.float32(np.log(60.0 / cam.fx))
    gpu = run_gpu(sc, cam, capacity=1 << 22)
    pre = orc.preprocess(cam, sc)
    values, tiles, ranges = orc.bin_sort(cam, pre)
    compare_lists(gpu, values, tiles, ranges)
    cs, st, P = gs.camera_struct(cam), gpu["scene_tensors"], gpu["P"]
    for capacity in (P, P - 1) if P > 1 else ():
        fr = gs.Frame(n, cam.width, cam.height, gs.GS_APP_SH3, max(capacity, 1))
        gs.gs_preprocess(cs, st.gaussians(), st.appearance(gs.GS_APP_SH3), fr.pre, fr.workspace, fr.ws_bytes,
                         sync_pairs=False)
        gs.gs_bin_sort(cs, fr.pre, n, gs.GS_PAIRS_ON_DEVICE, capacity, fr.values, None, fr.ranges, fr.workspace,
                       fr.ws_bytes)
        got = fr.ranges.cpu().numpy().reshape(-1, 2).astype(np.int64)
        if capacity == P:
            assert np.array_equal(got, ranges)
            assert np.array_equal(fr.values.cpu().numpy()[:P].astype(np.int64), values.astype(np.int64))
        else:
            assert not got.any() and int(fr.num_pairs.item()) == P


@pytest.mark.parametrize("n,size", [(1, (64, 64)), (65, (50, 40)), (257, (16, 16)), (1025, (64, 64)), (4097, (70, 64)),
                                    (12288, (64, 64)), (12289, (64, 64)), (12289, (768, 64)), (12289, (832, 64)),
                                    (24576, (384, 256)), (24576, (64, 1536))])
def test_few_gaussians_whole_image(n, size):
    # every Gaussian in every tile: lists of all Gaussians out of one block, of
    # 2 x 2 blocks with tiles outside the image, and of the fewest blocks (one for
    # every 1,024 Gaussians) that more than 12,288 Gaussians are searched in
    sc = inputs.make_scene("tiny", n=n)
    sc.means[:] *= np.float32(0.2)
    cam = tiny_camera(*size)
    sc.log_scales[:] = np.float32(np.log(3.0 * max(size) / cam.fx))
    gpu = run_gpu(sc, cam, capacity=n * -(-size[0] // 16) * -(-size[1] // 16))
    values, tiles, ranges = orc.bin_sort(cam, orc.preprocess(cam, sc))
    assert values.size == n * len(ranges)
    compare_lists(gpu, values, tiles, ranges)


@pytest.mark.parametrize("tiles_x", [2048, 2049])
def test_backward_tile_order_limit(tiles_x):
    # 2048 x 16 = 32768 tiles, the largest image whose backward launches its
    # tiles longest walk first (as every other case here), and 2049 x 16, the
    # smallest that keeps the plain tile order
    sc = inputs.make_scene("tiny").subset(np.arange(300))
    check_all(sc, tiny_camera(16 * tiles_x, 256), label="wide-bwd-%d" % tiles_x)


@pytest.mark.parametrize("tiles", [(16, 16), (1, 257), (48, 32), (29, 53), (64, 32), (3, 683), (64, 48), (7, 439)])
def test_pixels_per_lane_limits(tiles):
    # 1536, 2048 and 3072 tiles and the next sizes above them, where the blend
    # kernels take more pixels per lane, and 256 tiles, above which the backward
    # orders its tiles: clustered splats (long lists, a count
    # that is no multiple of the splats per step, saturated pixels) and a
    # background that stays in sight
    w, h = 16 * tiles[0] - 5, 16 * tiles[1] - 3
    sc = inputs.make_scene("medium", n=3001)
    sc.log_scales += np.float32(0.8)
    sc.opacity_logits += np.float32(1.5)
    check_all(sc, tiny_camera(w, h, bg=(0.2, 0.4, 0.1)), label="pix-%dx%d" % tiles)


def thin_scene(n, cam, long_px, short_px, seed=5):
    """n splats of about long_px x short_px pixels (sigma), at every angle in the image plane, in the middle of the view."""
    sc = inputs.make_scene("tiny", n=n)
    r = np.random.default_rng(seed)
    sc.means[0], sc.means[1], sc.means[2] = (r.uniform(-b, b, n) for b in (0.8, 0.5, 0.01))
    sc.log_scales[0], sc.log_scales[1:] = np.log(3.0 * long_px / cam.fx), np.log(3.0 * short_px / cam.fx)
    half = r.uniform(0, np.pi, n) / 2
    sc.quats[:] = 0
    sc.quats[0], sc.quats[3] = np.cos(half), np.sin(half)
    sc.opacity_logits[:] = r.uniform(-2.5, -0.5, n)
    return sc


def smooth_upstream(cam, seed=3):
    """An upstream gradient that varies slowly over the image, as a loss's does (white noise averages out in the sums
    over a splat's pixels, and with it the cancellation between them)."""
    r = np.random.default_rng(seed)
    y, x = np.mgrid[0:cam.height, 0:cam.width]
    wave = [np.sin(2 * np.pi * (r.uniform(0.5, 2) * x / cam.width + r.uniform(0.5, 2) * y / cam.height) +
                   r.uniform(0, 6)) for _ in range(3)]
    return (1e-3 * (1 + 0.5 * np.stack(wave))).astype(np.float32)


@pytest.mark.parametrize("long_px,short_px,size", [
    (10, 1, (480, 320)), (10, 1, (800, 608)), (10, 1, (1600, 1064)),
    (40, 4, (480, 320)), (40, 4, (800, 608)), (40, 4, (1600, 1064)),
    (60, 0.5, (480, 320)), (60, 0.5, (800, 608)), (60, 0.5, (1600, 1064)),
    (300, 0.1, (480, 320)), (300, 0.1, (800, 608))])
def test_mean_gradient_of_long_thin_splats(long_px, short_px, size):
    # dL/dmean2d of a long thin splat is a difference of terms up to the conic's
    # condition number larger, with the conic of the record that was blended. The
    # three sizes take the three numbers of pixels per lane. The measure is the
    # error that fp32 leaves in any case: the oracle with each pixel's power and
    # alpha in fp32, its products and sums in fp64. Products rounded where the terms
    # are small add at most about as much again, independently of it: together
    # sqrt(2) times, 1.5 with the medians' spread. The additions of the waves' sums
    # round to 2^-24 of the running sum, which is up to 16 times the result (the
    # splat's two sides of its mean cancel): 1e-6 more. Combined from the finished
    # sums the errors were 3e-6 to 7e-6 at 40 x 4, 2e-5 at 10 x 1 in the largest image.
    cam = tiny_camera(*size)
    sc = thin_scene(160, cam, long_px, short_px)
    pre = orc.preprocess(cam, sc)
    values, _, ranges = orc.bin_sort(cam, pre)
    margin = orc.render_fwd(cam, pre, ranges, values)[3]
    g = (smooth_upstream(cam) * (margin > 1.0)[None]).astype(np.float32)
    ref = orc.render_bwd(cam, sc, pre, ranges, values, g, mode="f64")["dmean2d"]
    fp32 = orc.render_bwd(cam, sc, pre, ranges, values, g, mode="f32")["dmean2d"]
    gpu = run_gpu(sc, cam, "sh3", 3, g, capacity=values.size)["grads"]["dmean2d"]

    def error(d):
        return np.median(np.linalg.norm(d - ref, axis=0) / np.linalg.norm(ref, axis=0))
    say("case thin %g x %g px, %dx%d: dmean2d error %.2e, in fp32 in any case %.2e" % (long_px, short_px, *size,
                                                                                      error(gpu), error(fp32)))
    assert error(gpu) <= 1.5 * error(fp32) + 1e-6


@pytest.mark.parametrize("size", [(480, 320), (800, 608), (1600, 1064)])
def test_opacity_gradient_of_long_thin_splats(size):
    # the quadratic form of a long thin splat is a difference of terms up to kappa =
    # ac / (ac - b^2) larger. A constant of the form that is rounded once per splat
    # errs alike at every pixel: c's, by a relative d, moves the sum that is the
    # opacity's gradient by d kappa / 2 (the mean of c dy^2 / 2 over the splat), and
    # |d| of one product is 2.1e-8 in the median (a quarter of 2^-23, over mantissas
    # from 1 to 2). Roundings that differ from pixel to pixel average out: 1.5 times
    # the one constant's share. (With a's, b's and c's rounded 2.6e-8 to 3.0e-8.)
    cam = tiny_camera(*size)
    sc = thin_scene(160, cam, 60, 0.5)
    pre = orc.preprocess(cam, sc)
    values, _, ranges = orc.bin_sort(cam, pre)
    margin = orc.render_fwd(cam, pre, ranges, values)[3]
    g = (smooth_upstream(cam) * (margin > 1.0)[None]).astype(np.float32)
    ref = orc.render_bwd(cam, sc, pre, ranges, values, g, mode="f64")["dopacity_logits"].reshape(-1)
    gpu = run_gpu(sc, cam, "sh3", 3, g, capacity=values.size)["grads"]["dopacity_logits"].reshape(-1)
    a, b, c = pre["conic"]
    error = np.median(np.abs(gpu - ref) / np.abs(ref) * (1 - b * b / (a * c)))
    say("case thin opacity %dx%d: dopacity_logits error %.2e kappa" % (*size, error))
    assert error <= 1.5 * 2.1e-8 / 2


@pytest.mark.parametrize("n,tiles", [(1, (1, 1)), (127, (1, 1)), (255, (2, 1)), (256, (1, 2)), (257, (1, 1)),
                                     (1025, (2, 2)), (128, (32, 49)), (129, (39, 40)), (300, (40, 39))])
def test_backward_spans(n, tiles):
    # the waves of a tile add up their sums over 256 list entries (128 above 1,536
    # tiles): lists that end at, before and behind such a span's end, walked to
    # their end by every wave, or by some (a part of the splats is opaque or small)
    w, h = 16 * tiles[0] - 3, 16 * tiles[1] - 5
    cam = tiny_camera(w, h, bg=(0.2, 0.4, 0.1))
    sc = inputs.make_scene("tiny", n=n)
    sc.means[:] *= np.float32(0.2)
    sc.log_scales[:] = np.float32(np.log(6.0 * max(w, h) / cam.fx))
    sc.opacity_logits[:] = -4.8
    sc.log_scales[:, ::5] = np.float32(np.log(6.0 / cam.fx))
    sc.log_scales[:] -= np.float32([[0.0], [0.3], [0.6]])   # equal scales would have no rotation gradient
    sc.opacity_logits[7::50] = 1.0
    # flat splats cross a threshold slowly: the pixels within the rounding bound are
    # a strip of up to 0.1 pixels along n / 5 contours of up to 2 (w + h)
    check_all(sc, cam, label="spans-%d-%dx%d" % (n, *tiles), max_flagged=max(n // 5 * 2 * (w + h) // 10, w * h // 250))


@pytest.mark.parametrize("value", [np.inf, np.nan])
@pytest.mark.parametrize("tiles", [(4, 4), (40, 40), (64, 49)])
def test_backward_keeps_a_pixel_to_its_splats(tiles, value):
    # an infinite or undefined upstream gradient at one pixel (1, 2 and 4 pixels per
    # lane): the Gaussians that are blended there take it, and no other Gaussian's
    # gradient changes, also of those that share its lane, wave and list
    cam = tiny_camera(16 * tiles[0], 16 * tiles[1])
    sc = inputs.make_scene("tiny")
    pre = orc.preprocess(cam, sc)
    values, _, ranges = orc.bin_sort(cam, pre)
    n_contrib, margin = orc.render_fwd(cam, pre, ranges, values)[2:]
    y, x = np.unravel_index(np.argmax(np.where(margin > 1.0, n_contrib, -1)), margin.shape)
    g = inputs.make_upstream_grad(cam.width, cam.height)
    g[:, y, x] = 0.0
    one = np.zeros_like(g)
    one[:, y, x] = 1.0
    there = orc.render_bwd(cam, sc, pre, ranges, values, one)["dcolor"].any(axis=0)
    listed = ranges[y // 16 * tiles[0] + x // 16] @ (-1, 1)
    clean = run_gpu(sc, cam, "sh3", 3, g, capacity=values.size)["grads"]
    g[:, y, x] = value
    got = run_gpu(sc, cam, "sh3", 3, g, capacity=values.size)["grads"]
    say("case one pixel %s of %dx%d tiles: %d Gaussians blended there, %d in its tile's list, of %d" % (
        value, *tiles, there.sum(), listed, sc.n))
    assert 0 < there.sum() < listed and not np.isfinite(got["dsh"][:3, there]).any()
    for k, ref in clean.items():
        # the atomics' order: as the parity bar
        bound = GRAD_ELEM_RTOL * np.abs(ref) + GRAD_ELEM_FLOOR * np.abs(ref).max()
        assert (np.abs(got[k] - ref) <= bound)[..., ~there].all(), k


@pytest.mark.parametrize("degree", [3, 1])
def test_sh3_backward_without_the_colour_jacobian(degree):
    # gs_preprocessed.color_jac NULL: the preprocess writes no view-direction
    # Jacobian and the backward re-reads the SH coefficients instead. The same
    # gradients as with it (the oracle checks the Jacobian path in every other
    # SH3 case), to the float atomics' summation order and a few ulp of the two
    # evaluation orders of the direction term.
    sc = inputs.make_scene("medium")
    cam = inputs.make_cameras("medium")[6]
    say("case SH3 backward from the coefficients, degree %d" % degree)
    up = torch.from_numpy(inputs.make_upstream_grad(cam.width, cam.height, 6)).cuda()
    st = gs.SceneTensors(sc)
    cs = gs.camera_struct(cam)
    out = []
    for jac in (True, False):
        fr = gs.Frame(sc.n, cam.width, cam.height, gs.GS_APP_SH3, 1 << 22)
        if not jac:
            fr.pre.color_jac = None
        fr.forward(cs, st, degree)
        fr.backward(cs, st, up, degree)
        torch.cuda.synchronize()
        out.append({k: getattr(fr, k).clone() for k in ("dmeans", "dlog_scales", "dquats", "dopacity_logits", "dsh")})
        out[-1]["image"] = fr.image.clone()
    assert torch.equal(out[0]["image"], out[1]["image"])
    for k in ("dmeans", "dlog_scales", "dquats", "dopacity_logits", "dsh"):
        a, b = out[0][k], out[1][k]
        scale = float(b.abs().max())
        err = float((a - b).abs().max())
        say("  %s: max |diff| %.2e of max |grad| %.2e" % (k, err, scale))
        assert bool(((a - b).abs() <= 1e-4 * b.abs() + 1e-6 * scale).all()), k


def test_capacity_retry():
    sc = inputs.make_scene("tiny")
    check_all(sc, inputs.make_cameras("tiny")[0], capacity=100, label="capacity")


def test_empty_and_culled_scenes():
    sc = inputs.make_scene("tiny")
    empty = sc.subset(np.arange(0))
    gpu, ref = check_all(empty, tiny_camera(40, 24, bg=(0.3, 0.6, 0.9)), label="empty")
    assert np.all(gpu["image"][0] == np.float32(0.3))
    # camera looking away from every Gaussian
    away = inputs.look_at_camera([0.0, 0.0, -3.0], 64, 64, target=(0.0, 0.0, -6.0))
    gpu, ref = check_all(sc, away, label="culled")
    assert gpu["P"] == 0 and np.all(gpu["tiles"] == 0)
    for k, v in gpu["grads"].items():
        assert np.all(v == 0), k


@pytest.mark.parametrize("cam_index", range(8))
def test_medium_scene(cam_index):
    # every camera of the medium workload (200k Gaussians, 1280x720)
    sc = inputs.make_scene("medium")
    check_all(sc, inputs.make_cameras("medium")[cam_index], label="medium cam %d" % cam_index, cam_seed=cam_index)


def test_mlp_eval_matches_oracle():
    rng = np.random.default_rng(31)
    rows = 1000                                 # 15 full waves and a ragged one
    x = rng.normal(0.0, 0.5, size=(rows, 17))
    x[:, 14:] /= np.linalg.norm(x[:, 14:], axis=1, keepdims=True)
    x[7] = 0.0                                  # all-zero input: every hidden unit at 0
    xb = x.astype(np.float16).view(np.uint16)
    w = inputs.make_mlp_weights(5)
    say("case mlp_eval rows=%d" % rows)
    xt = torch.from_numpy(xb.view(np.int16)).cuda()
    wt = torch.from_numpy(w.view(np.int16)).cuda()
    out = torch.empty(rows, 3, device="cuda")
    gs.gs_mlp_eval(xt, rows, wt, out)
    torch.cuda.synchronize()
    got = out.cpu().numpy()
    err = np.abs(got - orc.mlp_eval(xb, w))
    err_half = np.abs(got - orc.mlp_eval(xb, w, half_act=True))
    say("  max abs error %.2e (exact decoder), %.2e (binary16 activations)" % (err.max(), err_half.max()))
    assert err.max() <= MLP_ATOL
    assert err_half.max() <= MLP_HALF_ATOL
    assert np.all(got[7] == 0.5)


def test_tiny_scene_latent():
    sc = inputs.make_scene("tiny", appearance=("latent",))
    check_all(sc, inputs.make_cameras("tiny")[0], kind="latent", label="tiny latent", max_flagged=0)


def test_ragged_latent_with_background():
    sc = inputs.make_scene("tiny", appearance=("latent",))
    check_all(sc, tiny_camera(50, 37, bg=(0.25, 0.5, 0.75)), kind="latent", label="ragged latent")


@pytest.mark.parametrize("cam_index", [2, 6])
def test_medium_scene_latent(cam_index):
    sc = inputs.make_scene("medium", appearance=("latent",))
    check_all(sc, inputs.make_cameras("medium")[cam_index], kind="latent", label="medium latent cam %d" % cam_index,
              cam_seed=cam_index)


@pytest.mark.parametrize("degree", [0, 1, 2, 3])
def test_tiny_scene_neural(degree):
    # the paper's neural appearance; degree 0 has the residual off
    sc = inputs.make_scene("tiny", appearance=("neural",))
    check_all(sc, tiny_camera(), kind="neural", sh_degree=degree, label="tiny-neural", max_flagged=0)


def test_ragged_neural_with_background():
    sc = inputs.make_scene("tiny", appearance=("neural",))
    check_all(sc, tiny_camera(50, 37, bg=(0.1, 0.5, 0.9)), kind="neural", label="ragged-neural")


def test_medium_scene_neural():
    sc = inputs.make_scene("medium", appearance=("neural",))
    check_all(sc, inputs.make_cameras("medium")[2], kind="neural", label="medium-neural")


def test_binning_one_tile_and_huge_gaussians():
    # 6000 Gaussians so small that nearly all touch one tile (a window of 64
    # consecutive pairs then holds up to 64 Gaussians), plus a few so large
    # they cover the whole 96x80 image; pairs span several emission chunks
    import dataclasses
    # (the scene's own anisotropic log-scales, shifted: with equal axes the
    # covariance would not depend on the rotation and the exact quaternion
    # gradient would be zero, leaving only rounding to compare)
    sc = inputs.make_scene("tiny", n=6000)
    ls = (sc.log_scales - np.float32(3.5)).astype(np.float32)
    ls[:, ::997] += np.float32(6.0)
    sc = dataclasses.replace(sc, log_scales=ls)
    check_all(sc, tiny_camera(96, 80), label="one-tile+huge")


# ---- the folded neural form (render only) ---------------------------------------

def folded_preact_check(sc, got):
    """GPU pre-activations against the oracle's fold (binary16 inputs, fp64 sum,
    rounded to binary16). The GPU's sin/cos (fp32) may round an input to the
    neighbouring binary16 value (spacing <= 2^-11 below 1), which moves a sum
    by at most max|W1| 2^-11, and it sums in fp32 (17 terms, error far below
    1e-5); the final rounding then adds at most one binary16 spacing. Both are
    rare: nearly every value is bit-equal."""
    ref = orc.neural_fold(sc.features, sc.neural_w).T          # [n][16]
    g = got.view(np.float16).astype(np.float64)
    assert g.shape == ref.shape
    w1 = np.abs(sc.neural_w.view(np.float16).astype(np.float64)[:512])
    spacing = np.spacing(np.abs(ref).astype(np.float16)).astype(np.float64)
    diff = np.abs(g - ref)
    bound = spacing + w1.max() * 2.0 ** -11 + 1e-5
    assert np.all(diff <= bound), float((diff / bound).max())
    flips = int((diff > 0).sum())
    say("  fold: %d of %d pre-activations on the neighbouring binary16 value" % (flips, ref.size))
    assert flips <= max(2, ref.size // 1000)


@pytest.mark.parametrize("n", [1, 63, 1000, 4096])
def test_neural_fold(n):
    sc = inputs.make_scene("tiny", n=n, appearance=("neural",))
    st = gs.SceneTensors(sc)
    got = st.fold_neural().cpu().numpy().view(np.uint16)
    torch.cuda.synchronize()
    folded_preact_check(sc, got)


def test_neural_fold_empty():
    sc = inputs.make_scene("tiny", n=1, appearance=("neural",))
    st = gs.SceneTensors(sc)
    st.preact = torch.full((1, 16), 7, dtype=torch.int16, device="cuda")
    gs.gs_neural_fold(st.features, st.neural_w, 0, st.preact)   # n = 0 touches nothing
    torch.cuda.synchronize()
    assert np.all(st.preact.cpu().numpy() == 7)


@pytest.mark.parametrize("degree", [0, 1, 2, 3])
def test_tiny_scene_neural_folded(degree):
    sc = inputs.make_scene("tiny", appearance=("neural",))
    check_all(sc, tiny_camera(), kind="neural_folded", sh_degree=degree, label="tiny-folded", grads=False)


def test_ragged_neural_folded_with_background():
    sc = inputs.make_scene("tiny", n=1000, appearance=("neural",))
    check_all(sc, tiny_camera(50, 37, bg=(0.3, 0.2, 0.1)), kind="neural_folded", label="ragged-folded",
              grads=False)


def test_medium_scene_neural_folded():
    sc = inputs.make_scene("medium", appearance=("neural",))
    check_all(sc, inputs.make_cameras("medium")[2], kind="neural_folded", label="medium-folded", grads=False)


# ---- NASG and NASGabor lobes ------------------------------------------------------

@pytest.mark.parametrize("kind", ["nasg", "nasgabor"])
@pytest.mark.parametrize("degree", [0, 1])
def test_tiny_scene_lobe(kind, degree):
    sc = inputs.make_scene("tiny", appearance=(kind,))
    check_all(sc, tiny_camera(), kind=kind, sh_degree=degree, label="tiny-" + kind)


@pytest.mark.parametrize("kind", ["nasg", "nasgabor"])
def test_ragged_lobe_with_background(kind):
    sc = inputs.make_scene("tiny", n=999, appearance=(kind,))
    check_all(sc, tiny_camera(50, 37, bg=(0.6, 0.1, 0.4)), kind=kind, label="ragged-" + kind)


@pytest.mark.parametrize("kind", ["nasg", "nasgabor"])
def test_medium_scene_lobe(kind):
    sc = inputs.make_scene("medium", appearance=(kind,))
    check_all(sc, inputs.make_cameras("medium")[5], kind=kind, label="medium-" + kind)


@pytest.mark.parametrize("degree", [0, 3])
def test_tiny_scene_sh_y0_folded(degree):
    # the paper's implementation: DC coefficients stored with Y0 folded in
    sc = inputs.make_scene("tiny")
    sc.sh = sc.sh.copy()
    sc.sh[0:3] *= np.float32(0.28209479177387814)
    sc.sh_y0_folded = True
    check_all(sc, tiny_camera(), sh_degree=degree, label="tiny-sh-y0-folded")


# ---- the neural decoder configurations of the paper's architecture table ---------

@pytest.mark.parametrize("arch", [(1, 16, 0), (3, 16, 0), (2, 16, 1), (3, 16, 1), (2, 32, 0)])
def test_tiny_scene_neural_configurations(arch):
    sc = inputs.make_scene("tiny", appearance=("neural",), neural_arch=arch)
    check_all(sc, tiny_camera(), kind="neural", sh_degree=3, label="tiny-neural-%d-%d-%d" % arch)


@pytest.mark.parametrize("degree", [0, 1, 2])
def test_tiny_scene_neural_32_wide_degrees(degree):
    # degree masking of the direction inputs (degree 0: the residual is off)
    sc = inputs.make_scene("tiny", appearance=("neural",), neural_arch=(2, 32, 0))
    check_all(sc, tiny_camera(), kind="neural", sh_degree=degree, label="tiny-neural-2-32-0")


def test_ragged_neural_32_wide_with_background():
    sc = inputs.make_scene("tiny", appearance=("neural",), neural_arch=(2, 32, 0))
    check_all(sc, tiny_camera(50, 37, bg=(0.1, 0.5, 0.9)), kind="neural", label="ragged-neural-2-32-0")


def test_medium_scene_neural_32_wide():
    sc = inputs.make_scene("medium", appearance=("neural",), neural_arch=(2, 32, 0))
    check_all(sc, inputs.make_cameras("medium")[2], kind="neural", label="medium-neural-2-32-0")


def test_medium_scene_neural_three_layers():
    sc = inputs.make_scene("medium", appearance=("neural",), neural_arch=(3, 16, 0))
    check_all(sc, inputs.make_cameras("medium")[2], kind="neural", label="medium-neural-3-16-0")


# ---- degenerate Gaussians ----------------------------------------------------------

def degenerate_scene():
    """The tiny scene with extreme members: needle-thin and screen-sized scales,
    opacities at the alpha cap and far below 1/255, means behind the camera,
    just beyond the near plane, on tile and pixel boundaries, and one Gaussian
    that projects far outside the image (guard band)."""
    sc = inputs.make_scene("tiny")
    f32 = np.float32
    m, ls, lg = sc.means, sc.log_scales, sc.opacity_logits
    ls[:, 0:20] = f32(-12.0)                   # far below a pixel
    ls[:, 20:30] = f32(0.5)                    # covering the whole image
    ls[0, 30:40] = f32(-1.0)                   # needles: one long axis
    ls[1:, 30:40] = f32(-9.0)
    lg[40:60] = f32(25.0)                      # opacity 1 -> alpha capped at 0.99
    lg[60:80] = f32(-25.0)                     # opacity ~ 1e-11, never 1/255
    m[:, 80:90] = np.array([[0.1], [0.2], [-3.5]], f32)          # behind the camera (it sits at z = -3)
    m[:, 90:100] = np.array([[0.0], [0.0], [-2.8 + 1e-4]], f32)  # just beyond the near plane 0.2
    cam = tiny_camera()
    # means whose projections land on tile corners and pixel centres
    fx = cam.fx
    for k, (u, v) in enumerate([(16, 16), (32, 48), (0.5, 0.5), (63.5, 31.5), (48, 0)]):
        # at depth 3 (z = 0 in the world) these land on tile corners and pixel
        # centres (the camera's x axis points along world -x, so u is mirrored)
        m[:, 100 + k] = np.array([(u - cam.cx) * 3.0 / fx, (v - cam.cy) * 3.0 / fx, 0.0], f32)
    m[:, 110] = np.array([3.0, 0.0, 0.0], f32)   # projects far to the side
    ls[:, 110] = f32(-0.5)
    return sc, cam


@pytest.mark.parametrize("kind", ["sh3", "neural", "nasg"])
def test_degenerate_gaussians(kind):
    sc, cam = degenerate_scene()
    if kind != "sh3":
        extra = inputs.make_scene("tiny", appearance=(kind,))
        sc.base_color = extra.base_color
        sc.features, sc.neural_w, sc.lobes, sc.lobes_gabor = (extra.features, extra.neural_w, extra.lobes,
                                                              extra.lobes_gabor)
    check_all(sc, cam, kind=kind, label="degenerate-" + kind)


# ---- the pair count read on the device -------------------------------------------

@pytest.mark.parametrize("size", [(64, 64), (16, 16)])
def test_device_pair_count(size):
    # gs_bin_sort in device mode (no read-back of P): the same lists, ranges and
    # image as the host mode; with a capacity below P nothing is listed, every
    # range is empty, the image is the background, the gradients are zero, and
    # pre->num_pairs keeps the P needed for the retry
    sc = inputs.make_scene("tiny")
    cam = tiny_camera(*size, bg=(0.2, 0.4, 0.6))
    say("case device pair count %dx%d" % size)
    cs = gs.camera_struct(cam)
    st = gs.SceneTensors(sc)
    g = torch.from_numpy(inputs.make_upstream_grad(cam.width, cam.height, 0)).cuda()
    host = gs.Frame(sc.n, cam.width, cam.height, gs.GS_APP_SH3, 1 << 14, want_tile_ids=True)
    P = host.forward(cs, st)
    dev = gs.Frame(sc.n, cam.width, cam.height, gs.GS_APP_SH3, 1 << 14, want_tile_ids=True)
    assert dev.forward(cs, st, sync_pairs=False) is None
    torch.cuda.synchronize()
    assert int(dev.num_pairs.item()) == P and not dev.pairs_overflowed()
    for k in ("values", "tile_ids"):
        assert torch.equal(getattr(dev, k)[:P], getattr(host, k)[:P]), k
    for k in ("ranges", "image", "final_T", "n_contrib"):
        assert torch.equal(getattr(dev, k), getattr(host, k)), k
    host.backward(cs, st, g)
    dev.backward(cs, st, g)
    torch.cuda.synchronize()
    for k in ("dmeans", "dlog_scales", "dquats", "dopacity_logits", "dsh"):
        a, b = getattr(dev, k).double(), getattr(host, k).double()
        assert torch.allclose(a, b, rtol=1e-5, atol=1e-12 + 1e-6 * float(b.abs().max())), k
    # overflow found on the device
    small = gs.Frame(sc.n, cam.width, cam.height, gs.GS_APP_SH3, P // 3)
    small.forward(cs, st, sync_pairs=False)
    torch.cuda.synchronize()
    assert small.pairs_overflowed() and int(small.num_pairs.item()) == P
    assert int(small.ranges.abs().sum().item()) == 0
    bg = torch.tensor([0.2, 0.4, 0.6], device="cuda").view(3, 1, 1).expand_as(small.image)
    assert torch.equal(small.image, bg.float())
    assert bool((small.final_T == 1).all()) and int(small.n_contrib.sum().item()) == 0
    small.backward(cs, st, g)
    torch.cuda.synchronize()
    for k in ("dmeans", "dlog_scales", "dquats", "dopacity_logits", "dsh"):
        assert int(torch.count_nonzero(getattr(small, k)[..., : sc.n]).item()) == 0, k
    # a host-mode count that understates P, with a capacity to match it: the
    # lists need more than the capacity, which is found on the device, and every
    # range comes out empty (nothing is written past the capacity)
    low = gs.Frame(sc.n, cam.width, cam.height, gs.GS_APP_SH3, P // 2)
    gs.gs_preprocess(cs, st.gaussians(), st.appearance(gs.GS_APP_SH3, 3), low.pre, low.workspace, low.ws_bytes,
                     sync_pairs=False)
    guard = torch.full((64,), -7, dtype=torch.int32, device="cuda")
    values = torch.cat([low.values, guard])
    gs.gs_bin_sort(cs, low.pre, sc.n, P // 2, P // 2, values, None, low.ranges, low.workspace, low.ws_bytes)
    torch.cuda.synchronize()
    assert int(low.ranges.abs().sum().item()) == 0
    assert torch.equal(values[P // 2:], guard)
    # retry with room for every pair
    retry = gs.Frame(sc.n, cam.width, cam.height, gs.GS_APP_SH3, P, want_tile_ids=True)
    retry.forward(cs, st, sync_pairs=False)
    torch.cuda.synchronize()
    assert not retry.pairs_overflowed()
    assert torch.equal(retry.values[:P], host.values[:P]) and torch.equal(retry.image, host.image)


# ---- the blend's work counts (measurement) ------------------------------------------

@pytest.mark.parametrize("case", ["tiny", "ragged", "medium"])
def test_render_work_counts(case):
    # gs_render_work: blended and visited entries against the oracle's
    # per-pixel counts (exactly where no pixel is flagged; otherwise within the
    # flagged pixels' list lengths), the listed entries equal to the sum of the
    # GPU's own n_contrib, and evaluated counts between them
    if case == "medium":
        sc, cam = inputs.make_scene("medium"), inputs.make_cameras("medium")[3]
    else:
        sc = inputs.make_scene("tiny")
        cam = inputs.make_cameras("tiny")[0] if case == "tiny" else tiny_camera(50, 37)
    say("case render work %s" % case)
    ref = orc.render(cam, sc, mode="f32")
    gpu = run_gpu(sc, cam)
    fr = gpu["frame"]
    counts = torch.zeros(5, dtype=torch.int64, device="cuda")
    gs.gs_render_work(gs.camera_struct(cam), fr.pre, sc.n, fr.values, fr.ranges, counts)
    torch.cuda.synchronize()
    blended, listed, ev_bwd, ev_fwd, walked = (int(v) for v in counts.cpu().numpy())
    say("  blended %d listed %d evaluated bwd %d fwd %d visited fwd %d" % (blended, listed, ev_bwd, ev_fwd, walked))
    assert listed == int(gpu["n_contrib"].astype(np.int64).sum())
    flagged = ref["margin"] <= 1.0
    ref_blended = int(ref["n_blended"].astype(np.int64).sum())
    ref_walked = int(ref["n_walked"].astype(np.int64).sum())
    tiles_x = (cam.width + 15) // 16
    ys, xs = np.mgrid[0:cam.height, 0:cam.width]
    lens = (ref["ranges"][:, 1] - ref["ranges"][:, 0])[(ys // 16) * tiles_x + xs // 16]
    slack = int(ref["n_contrib"][flagged].astype(np.int64).sum() + gpu["n_contrib"][flagged].astype(np.int64).sum())
    if not flagged.any():
        assert blended == ref_blended and walked == ref_walked
    assert abs(blended - ref_blended) <= slack
    assert abs(walked - ref_walked) <= int(lens[flagged].astype(np.int64).sum())
    assert blended <= ev_bwd <= listed and ev_bwd <= ev_fwd <= walked and listed <= walked


# ---- decoder weights far from their initialisation -----------------------------------

@pytest.mark.parametrize("kind,arch,factor", [("latent", None, 4.0), ("neural", (2, 16, 0), 4.0),
                                              ("neural", (3, 16, 0), 4.0), ("neural", (2, 32, 0), 4.0),
                                              ("neural", (3, 16, 0), 16.0)])
def test_decoder_large_weights(kind, arch, factor):
    # every decoder weight times 4 or 16 (exact in binary16): the backward's hidden-
    # layer gradients grow by the layers' norms on the way back and must stay
    # within binary16 range (the chunk's gradient scale accounts for them).
    # The binary16 rounding flips of the forward grow with the weights too, so
    # the colour and gradient bars are those of the decoder path scaled by the
    # weights' growth along the network (the factor per layer).
    sc = inputs.make_scene("tiny", appearance=(kind,), neural_arch=arch)
    attr = "mlp_w" if kind == "latent" else "neural_w"
    w = getattr(sc, attr).view(np.float16).astype(np.float32) * factor
    setattr(sc, attr, w.astype(np.float16).view(np.uint16))
    layers = 3 if kind == "latent" else arch[0] + 1
    growth = factor ** layers
    cam = tiny_camera()
    say("case large weights %s %s x%g" % (kind, arch, factor))
    ref = orc.render(cam, sc, kind=kind, sh_degree=3, mode="f32", half_act=True)
    flagged = flagged_pixels(ref["margin"])
    g = (inputs.make_upstream_grad(cam.width, cam.height, 0) * ~flagged[None]).astype(np.float32)
    grads = orc.render_bwd(cam, sc, ref["pre"], ref["ranges"], ref["values"], g, kind=kind, sh_degree=3, mode="f32",
                           half_act=True)
    gpu = run_gpu(sc, cam, kind, 3, g)
    vis = ref["pre"]["tiles"] > 0
    err = np.abs(gpu["splat"]["color"][:, vis] - ref["pre"]["color"][:, vis])
    say("  colours: max abs %.2e" % err.max())
    assert err.max() <= MLP_HALF_ATOL * growth
    for k, v in gpu["grads"].items():
        assert np.all(np.isfinite(v)), k
    st = grad_stats(gpu["grads"], grads)
    report_grads(st)
    for k, (rel, _, _, _) in st.items():
        assert rel <= 5e-3, (k, rel)
