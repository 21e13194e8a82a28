"""Parity of the HIP path (through the C ABI) with the FP64 oracle on the
parity scene (2,000 Gaussians, SH degree 0, four 128x128 views) and on small
edge cases.

Tolerances (FP32 kernels vs FP64 oracle):
  - images: |C - C_ref| <= 1e-4 |C_ref| + 1e-6 on pixels the oracle does not
    flag as near a decision threshold;
  - gradients: per attribute group ||g - g_ref|| / ||g_ref|| <= 1e-3;
  - projection: 1e-5 relative (a few FP32 rounding steps);
  - Adam / consensus: 1e-6 relative + small absolute (a handful of FP32 ops);
  - binning: bit-exact against a stable sort of the same integer keys.
"""
import math

import numpy as np
import pytest

import oracle
from paper_2405_13943_amd import scenes

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2405_13943_amd import gs  # noqa: E402

LOG2E = 1.0 / math.log(2.0)
GROUPS = {"p": [0, 1, 2], "q": [3, 4, 5, 6], "s": [7, 8, 9], "o": [10]}


def group_planes(A):
    d = dict(GROUPS)
    d["f"] = list(range(11, A))
    return d


def make_frame(scene, cfg, views=None, weight=None):
    views = list(range(len(scene.cams))) if views is None else views
    n = scene.params.shape[1]
    w = weight if weight is not None else 1.0 / len(views)
    jobs = [gs.JobSpec(v, 0, n, w) for v in views]
    return gs.Frame(scene.cams, jobs, cfg)


def frame_target(frame, scene, views):
    return torch.cat([torch.from_numpy(scene.targets[v]).reshape(-1) for v in views]).cuda()


@pytest.fixture(scope="module")
def cfg1():
    return scenes.config1()


@pytest.fixture(scope="module")
def gpu1(cfg1):
    print("\n[gpu] config-1 forward (2000 G, 4 x 128x128)", flush=True)
    cfg = gs.raster_cfg((16, 16))
    frame = make_frame(cfg1, cfg)
    params = torch.from_numpy(cfg1.params).cuda()
    buf = gs.rasterize(params, frame, cfg)
    torch.cuda.synchronize()
    return cfg, frame, params, buf


@pytest.fixture(scope="module")
def ref1(cfg1):
    return [oracle.render(cfg1.params, c) for c in cfg1.cams]


def images(frame, buf):
    return [frame.image(buf.rgb, i).cpu().numpy().astype(np.float64) for i in range(frame.n_jobs)]


def assert_image_close(got, ref, flags, rtol=1e-4, atol=1e-6):
    ok = flags == 0
    err = np.abs(got - ref["rgb"])
    bad = (err > rtol * np.abs(ref["rgb"]) + atol) & ok[None]
    assert not bad.any(), f"{bad.sum()} pixel-channels off, max err {err[:, ok].max():.3e}"


# ---------------------------------------------------------------------------

def test_project_matches_oracle(cfg1, gpu1):
    cfg, frame, params, buf = gpu1
    rec = buf.rec.view(-1, gs.REC_WORDS).cpu().numpy().astype(np.float64)
    meta = buf.meta.view(-1, gs.META_WORDS).cpu().numpy().view(np.uint32)
    for v in range(4):
        pr = oracle.project(cfg1.params, cfg1.cams[v])
        r = rec[v * 2000:(v + 1) * 2000]
        m = meta[v * 2000:(v + 1) * 2000]
        vis = m[:, 1] > 0
        assert vis.sum() > 500
        assert pr["valid"][vis].all()
        np.testing.assert_allclose(r[vis, 0:2], pr["mean2d"][vis], rtol=0, atol=2e-4)
        conic = np.stack([r[:, 2] / (-0.5 * LOG2E), r[:, 3] / -LOG2E, r[:, 4] / (-0.5 * LOG2E)], axis=1)
        scale = np.abs(pr["conic"][vis]).max(axis=1, keepdims=True)
        np.testing.assert_allclose(conic[vis] / scale, pr["conic"][vis] / scale, atol=2e-5)
        np.testing.assert_allclose(2.0 ** r[vis, 5], pr["opacity"][vis], rtol=2e-6)
        np.testing.assert_allclose(r[vis, 6:9], pr["rgb"][vis], atol=2e-6)
        np.testing.assert_allclose(m[vis, 0].view(np.float32), pr["depth"][vis], rtol=1e-6)
        # moment frame: the conic's largest-eigenvalue axis (cos, sin), cos >= 0
        t = r[vis, 9]
        cs, sn = (1 - t * t) / (1 + t * t), 2 * t / (1 + t * t)
        a, b, c = (pr["conic"][vis, k] for k in range(3))
        d11 = a * cs * cs + 2 * b * cs * sn + c * sn * sn
        d22 = a * sn * sn - 2 * b * cs * sn + c * cs * cs
        d12 = (c - a) * cs * sn + b * (cs * cs - sn * sn)
        spread = np.sqrt((a - c) ** 2 + 4 * b * b)
        assert (np.abs(t) <= 1.0 + 1e-6).all()
        assert (np.abs(d12) <= 1e-3 * spread + 1e-6 * (a + c)).all()
        assert (d11 - d22 >= -1e-3 * spread - 1e-6 * (a + c)).all()


def _bins_check(frame, buf):
    meta = buf.meta.view(-1, gs.META_WORDS).cpu().numpy().view(np.uint32)
    c = gs.read_counters(buf)
    rects = np.stack([meta[:, 2] & 0xFFFF, meta[:, 2] >> 16, meta[:, 3] & 0xFFFF, meta[:, 3] >> 16], axis=1)
    rects = rects.astype(np.int64)
    rects[meta[:, 1] == 0] = [1, 1, 0, 0]
    job_of = np.zeros(frame.n_records, np.int64)
    for j in range(frame.n_jobs):
        job_of[frame.job(j).rec0: frame.job(j).rec0 + frame.job(j).g1 - frame.job(j).g0] = j
    tb = [frame.job(j).tile0 for j in range(frame.n_jobs)]
    tx = [frame.job(j).tiles_x for j in range(frame.n_jobs)]
    vals, ranges = oracle.bin_reference(rects, meta[:, 0], tb, tx, job_of, frame.n_tiles)
    assert c["status"] == 0
    assert c["pairs"] == len(vals)
    assert c["visible"] == int((meta[:, 1] > 0).sum())
    got = buf.vals[:len(vals)].cpu().numpy().view(np.uint32)
    np.testing.assert_array_equal(got, vals)
    np.testing.assert_array_equal(buf.ranges.view(-1, 2).cpu().numpy().view(np.uint32), ranges)


def test_bins_bit_exact(gpu1):
    cfg, frame, params, buf = gpu1
    _bins_check(frame, buf)


def plan_check(frame, cfg, buf):
    """The compositing plan: a permutation of the tiles grouped by their
    wavefront count (4 above 4x the mean list length, 2 above 1.25x, never
    more than the tile's quadrants), the counts in front; inside a group the
    lists by bucket of half the mean length, longest first (last bucket
    open-ended).  Which of several tiles of one bucket comes first is free."""
    nt = frame.n_tiles
    order = buf.tile_order.cpu().numpy().view(np.uint32)
    rg = buf.ranges.view(-1, 2).cpu().numpy().view(np.uint32).astype(np.int64)
    n = rg[:nt, 1] - rg[:nt, 0]
    pairs = int(gs.read_counters(buf)["pairs"])
    quads = (cfg.tile_w // 8) * (cfg.tile_h // 8)
    a = 4 * n * nt
    waves = np.minimum(np.where(a > 16 * pairs, 4, np.where(a > 5 * pairs, 2, 1)), quads)
    n4, n2, n1 = (int(v) for v in order[:3])
    assert (n4, n2, n1) == tuple(int((waves == w).sum()) for w in (4, 2, 1))
    lst = order[4:4 + nt].astype(np.int64)
    assert np.array_equal(np.sort(lst), np.arange(nt))
    bucket = np.minimum(2 * n * nt // max(pairs, 1), 15)
    for lo, hi, w in ((0, n4, 4), (n4, n4 + n2, 2), (n4 + n2, nt, 1)):
        part = lst[lo:hi]
        assert (waves[part] == w).all()
        assert (np.diff(bucket[part]) <= 0).all()


@pytest.mark.parametrize("tile", [(16, 16), (32, 8), (16, 8)])
def test_compositing_plan(cfg1, tile):
    cfg = gs.raster_cfg((*tile, -1, -1))
    frame = make_frame(cfg1, cfg)
    buf = gs.rasterize(torch.from_numpy(cfg1.params).cuda(), frame, cfg)
    plan_check(frame, cfg, buf)
    assert int(buf.tile_order[0]) + int(buf.tile_order[1]) > 0      # some tiles split


@pytest.mark.parametrize("n", [300, 1500, 3000, 6000, 9000])
def test_bins_bit_exact_long_tile_lists(n):
    """Large Gaussians in front of a small view put n entries in every tile
    (above 256: the in-LDS merge sort, 4 keys per thread up to 1024 and 16
    beyond, the capacity making the frame dense; above 4096: the long-list
    kernel; above 8192: its chunks and merges), with many equal depths (ties
    ordered by record), against the reference."""
    p = scenes.gaussians(n, 0, 4100 + n, [-0.3, -0.3, -0.3], [0.3, 0.3, 0.3], 0.0, 0.1)
    p[scenes.MEAN + 2, ::3] = 0.25                  # every third Gaussian at the same depth
    params = torch.from_numpy(p).cuda()
    cam = scenes.look_at([0.0, 0.0, 3.0], [0, 0, 0], 64, 48, 60.0, 60.0)
    for tile in [(16, 16), (8, 8)]:
        cfg = gs.raster_cfg(tile)
        frame = gs.Frame([cam], [gs.JobSpec(0, 0, n, 1.0)], cfg)
        buf = gs.rasterize(params, frame, cfg, capacity=n * frame.n_tiles + 1024)
        lens = np.diff(buf.ranges.view(-1, 2).cpu().numpy().view(np.uint32), axis=1)
        assert lens.max() > min(n - 10, 256)
        _bins_check(frame, buf)


@pytest.mark.parametrize("n", [1500, 3000])
def test_bins_bit_exact_long_lists_in_sparse_frame(n):
    """A cluster of n small Gaussians in a 1600x1066 view: a few tiles hold
    about n entries while the mean list stays short, so the tile sort keeps
    its small form (8 keys per thread, lists up to 2048 on chip) and sends
    the longer lists to the long-list kernel; bins against the reference."""
    p = scenes.gaussians(n, 0, 4400 + n, [-0.01, -0.01, -0.3], [0.01, 0.01, 0.3], -5.0, 0.3)
    p[scenes.MEAN + 2, ::4] = 0.1                   # every fourth Gaussian at the same depth
    params = torch.from_numpy(p).cuda()
    cam = scenes.look_at([0.0, 0.0, 3.0], [0, 0, 0], 1600, 1066, 1200.0, 1200.0)
    cfg = gs.raster_cfg((16, 16))
    frame = gs.Frame([cam], [gs.JobSpec(0, 0, n, 1.0)], cfg)
    buf = gs.rasterize(params, frame, cfg, capacity=64 * n + 1024)
    assert buf.capacity <= frame.n_tiles * 1024        # the sparse form of the tile sort
    lens = np.diff(buf.ranges.view(-1, 2).cpu().numpy().view(np.uint32), axis=1)
    assert lens.max() > min(n - 100, 2048) and lens.mean() < 64
    _bins_check(frame, buf)


@pytest.mark.parametrize("size", [(16, 16), (17, 16), (48, 16), (200, 16)])
def test_bins_bit_exact_few_tiles(size):
    """1, 2, 3 and 13 tiles: no radix pass at all, then one pass of a 1-, 2-
    and 4-bit digit; every Gaussian in front of the camera."""
    n = 400
    p = scenes.gaussians(n, 0, 4300, [-0.4, -0.2, -0.2], [0.4, 0.2, 0.2], 0.0, 0.3)
    params = torch.from_numpy(p).cuda()
    w, h = size
    cam = scenes.look_at([0.0, 0.0, 3.0], [0, 0, 0], w, h, 40.0, 40.0)
    cfg = gs.raster_cfg((16, 16))
    frame = gs.Frame([cam], [gs.JobSpec(0, 0, n, 1.0)], cfg)
    buf = gs.rasterize(params, frame, cfg)
    assert frame.n_tiles == (w + 15) // 16 and gs.read_counters(buf)["pairs"] > 0
    _bins_check(frame, buf)


def test_bins_bit_exact_large_pair_capacity():
    """A pair capacity above 2^22 takes the tile radix sort's large form (16
    keys per thread and iteration, here over many iterations and a ragged
    last one); the bins do not change."""
    n = 1500
    p = scenes.gaussians(n, 0, 4200, [-0.3, -0.3, -0.3], [0.3, 0.3, 0.3], 0.0, 0.1)
    params = torch.from_numpy(p).cuda()
    cam = scenes.look_at([0.0, 0.0, 3.0], [0, 0, 0], 64, 48, 60.0, 60.0)
    cfg = gs.raster_cfg((8, 8))
    frame = gs.Frame([cam], [gs.JobSpec(0, 0, n, 1.0)], cfg)
    buf = gs.rasterize(params, frame, cfg, capacity=(1 << 22) + 4096)
    assert gs.read_counters(buf)["pairs"] > 4096 * 8
    _bins_check(frame, buf)


@pytest.mark.parametrize("tile", [(8, 8), (16, 8), (32, 8)])
def test_bins_bit_exact_other_tiles(cfg1, tile):
    cfg = gs.raster_cfg(tile)
    frame = make_frame(cfg1, cfg)
    buf = gs.rasterize(torch.from_numpy(cfg1.params).cuda(), frame, cfg)
    _bins_check(frame, buf)


def test_render_fwd_matches_oracle(gpu1, ref1):
    cfg, frame, params, buf = gpu1
    nflag = 0
    for v, img in enumerate(images(frame, buf)):
        ref = ref1[v]
        nflag += int((ref["flags"] != 0).sum())
        assert_image_close(img, ref, ref["flags"])
        T = frame.plane(buf.T, v).cpu().numpy()
        ok = ref["flags"] == 0
        np.testing.assert_allclose(T[ok], ref["T"][ok], rtol=1e-4, atol=1e-6)
    assert nflag < 50


def test_tile_shape_and_batch_invariance(cfg1, gpu1):
    """Forward images are bit-identical across tile shapes, wavefronts per
    tile, and whether views are rendered batched or one at a time."""
    cfg, frame, params, buf = gpu1
    base = images(frame, buf)
    for tile in [(8, 8), (16, 8), (32, 8), (16, 8, 2), (16, 16, 2), (16, 16, 4), (32, 8, 2), (32, 8, 4),
                 (16, 16, -1), (32, 8, -1), (16, 8, -1), (8, 8, -1)]:
        c2 = gs.raster_cfg(tile)
        f2 = make_frame(cfg1, c2)
        b2 = gs.rasterize(params, f2, c2)
        for a, b in zip(base, images(f2, b2)):
            np.testing.assert_array_equal(a, b)
    for v in range(4):
        f1 = make_frame(cfg1, cfg, [v])
        b1 = gs.rasterize(params, f1, cfg)
        np.testing.assert_array_equal(images(f1, b1)[0], base[v])


def test_forward_deterministic(gpu1):
    cfg, frame, params, buf = gpu1
    a = buf.rgb.clone()
    gs.rasterize(params, frame, cfg, buf)
    assert torch.equal(a, buf.rgb)


def _oracle_dldc(scene, views, ref, weight):
    """L1 gradient from the oracle image, zero at flagged pixels and where
    |C - target| is within rounding of the kink."""
    out = []
    for v in views:
        C = ref[v]["rgb"]
        d = C - scene.targets[v]
        g = weight * np.sign(d) / d.size
        g[:, ref[v]["flags"] != 0] = 0
        g[np.abs(d) < 1e-5] = 0
        out.append(g)
    return out


def test_contribution_count_matches_oracle(cfg1, gpu1, ref1):
    """gs_render_fwd_stats counts the (pixel, Gaussian) contributions of
    Eq. 2: the oracle's per-pixel contributor counts summed over the frame,
    up to one per flagged pixel; the image is the plain forward's."""
    cfg, frame, params, buf = gpu1
    rgb = buf.rgb.clone()
    kept = gs.render_fwd_stats(frame, cfg, buf)
    assert torch.equal(buf.rgb, rgb)
    n_ref = sum(int(r["n"].sum()) for r in ref1)
    flagged = sum(int(np.count_nonzero(r["flags"])) for r in ref1)
    assert n_ref > 10_000
    assert abs(kept - n_ref) <= flagged, (kept, n_ref, flagged)


def test_render_bwd_matches_oracle(cfg1, gpu1, ref1):
    cfg, frame, params, buf = gpu1
    views = list(range(4))
    dl = _oracle_dldc(cfg1, views, ref1, 0.25)
    g_ref = sum(oracle.backward(cfg1.params, cfg1.cams[v], dl[v]) for v in views)
    gin = torch.cat([torch.from_numpy(d.astype(np.float32)).reshape(-1) for d in dl]).cuda()
    grad = torch.empty_like(params)
    gs.render_bwd(params, frame, cfg, buf, grad, gs.LOSS_EXTERNAL, gin)
    g = grad.cpu().numpy().astype(np.float64)
    for name, planes in group_planes(params.shape[0]).items():
        num = np.linalg.norm(g[planes] - g_ref[planes])
        den = np.linalg.norm(g_ref[planes])
        assert den > 0, name
        assert num / den <= 1e-3, (name, num / den)
    # determinism of the backward (no float atomics on the gradient path)
    grad2 = torch.empty_like(params)
    gs.render_bwd(params, frame, cfg, buf, grad2, gs.LOSS_EXTERNAL, gin)
    assert torch.equal(grad, grad2)


@pytest.mark.parametrize("tile", [(16, 16, 2), (16, 16, 4), (32, 8, 4), (16, 8, 2), (16, 16, 2, -1), (32, 8, 1, -1),
                                  (16, 8, 2, -1), (8, 8, 1, -1)])
def test_render_bwd_sub_tile_waves_match_oracle(cfg1, ref1, tile):
    """Several wavefronts per tile (fixed, or per tile from its list length),
    each storing its own partials per pair: gradients against the FP64
    oracle as for one wavefront per tile, and deterministic."""
    cfg = gs.raster_cfg(tile)
    frame = make_frame(cfg1, cfg)
    params = torch.from_numpy(cfg1.params).cuda()
    buf = gs.rasterize(params, frame, cfg)
    views = list(range(4))
    dl = _oracle_dldc(cfg1, views, ref1, 0.25)
    g_ref = sum(oracle.backward(cfg1.params, cfg1.cams[v], dl[v]) for v in views)
    gin = torch.cat([torch.from_numpy(d.astype(np.float32)).reshape(-1) for d in dl]).cuda()
    grad = torch.empty_like(params)
    gs.render_bwd(params, frame, cfg, buf, grad, gs.LOSS_EXTERNAL, gin)
    g = grad.cpu().numpy().astype(np.float64)
    for name, planes in group_planes(params.shape[0]).items():
        num = np.linalg.norm(g[planes] - g_ref[planes])
        assert num / np.linalg.norm(g_ref[planes]) <= 1e-3, (name, tile)
    grad2 = torch.empty_like(params)
    gs.render_bwd(params, frame, cfg, buf, grad2, gs.LOSS_EXTERNAL, gin)
    assert torch.equal(grad, grad2)


@pytest.mark.parametrize("tile", [(16, 16, -1), (16, 16, 1), (16, 16, 2, 1), (16, 16, 1, 4), (16, 16, 4, 2),
                                  (32, 8, 2, 4), (32, 8, -1, 1), (16, 8, 2, 1), (8, 8, 1), (16, 16, -1, 2)])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_quadrant_masks_from_forward_equal_recomputed(cfg1, tile, dtype):
    """The backward reading the forward's per-entry quadrant masks (bins.qmask)
    gives the gradients it gives when it recomputes them, bit for bit, and the
    same loss, whatever the forward's and the backward's wavefront splits."""
    if dtype == torch.float64 and tile != (16, 16, 2, 1):
        pytest.skip("FP64 on one split pair")
    cfg = gs.raster_cfg(tile)
    frame = make_frame(cfg1, cfg)
    params = torch.from_numpy(cfg1.params).to("cuda", dtype)
    buf = gs.rasterize(params, frame, cfg)
    target = frame_target(frame, cfg1, range(4)).to(dtype)
    out = []
    for share in (True, False):
        buf.share_qmask = share
        g = torch.empty_like(params)
        loss = torch.zeros(4, dtype=dtype, device="cuda")
        gs.render_bwd(params, frame, cfg, buf, g, gs.LOSS_L1, target, loss)
        out.append((g, loss))
    buf.share_qmask = True
    assert torch.equal(out[0][0], out[1][0]), tile
    # the per-job loss is added with atomics in no fixed order
    torch.testing.assert_close(out[0][1], out[1][1], rtol=1e-6, atol=0)


@pytest.mark.parametrize("tile", [(16, 16), (16, 16, -1), (32, 8, -1), (8, 8, -1)])
def test_l1_loss_mode(cfg1, tile):
    """GS_LOSS_L1 equals the external mode fed the oracle's dL/dC of the
    L1 part of Eq. 3 (w sign(C - target) / 3HW on the GPU's own image), and
    the fused loss equals the oracle's w mean |C - target| per job: with one
    wavefront per tile, and with the wavefronts from the plan (whose
    workgroups mix tiles of the four jobs and add their sums per job)."""
    from oracle.raster import l1_loss_and_grad
    cfg = gs.raster_cfg(tile)
    frame = make_frame(cfg1, cfg)
    params = torch.from_numpy(cfg1.params).cuda()
    buf = gs.rasterize(params, frame, cfg)
    target = frame_target(frame, cfg1, range(4))
    loss = torch.zeros(4, dtype=torch.float32, device="cuda")
    g1 = torch.empty_like(params)
    gs.render_bwd(params, frame, cfg, buf, g1, gs.LOSS_L1, target, loss)
    n = 3 * 128 * 128
    rgb, tg = buf.rgb.cpu().numpy(), target.cpu().numpy()
    ref = [l1_loss_and_grad(rgb[i * n:(i + 1) * n], tg[i * n:(i + 1) * n], 0.25) for i in range(4)]
    dl = torch.from_numpy(np.concatenate([r[1] for r in ref]).astype(np.float32)).cuda()
    g2 = torch.empty_like(params)
    gs.render_bwd(params, frame, cfg, buf, g2, gs.LOSS_EXTERNAL, dl)
    torch.testing.assert_close(g1, g2, rtol=1e-6, atol=1e-12)
    np.testing.assert_allclose(loss.cpu().numpy(), [r[0] for r in ref], rtol=1e-5)


def _adam_bounds(x, g, m, v, w, lr, rho, step, mask, b1, b2, eps):
    """Per-element FP32 rounding bounds of one Adam + ADMM update, from the
    magnitudes of the terms each result sums (u = 2^-24, a few ops each):
    m' = b1 m + (1-b1) g' can cancel, so its bound scales with
    b1|m| + (1-b1)|g'|, not with |m'|; the step inherits m''s error."""
    from oracle.admm import penalty_groups
    u = 2.0 ** -24
    grp = penalty_groups(x.shape[0])
    x, g, m, v = (np.asarray(a, np.float64) for a in (x, g, m, v))
    r = np.asarray(rho)[grp][:, None] * (1.0 if mask is None else mask[None, :]) if w is not None else 0.0
    gp_terms = np.abs(g) + (np.abs(r) * (np.abs(x) + np.abs(w)) if w is not None else 0.0)
    gp = g + (r * (x - w) if w is not None else 0.0)
    sm = b1 * np.abs(m) + (1 - b1) * gp_terms
    m1 = b1 * m + (1 - b1) * gp
    v1 = b2 * v + (1 - b2) * gp * gp
    bc1, bc2 = 1 - b1 ** step, 1 - b2 ** step
    den = np.sqrt(v1 / bc2) + eps
    lrp = np.asarray(lr)[grp][:, None]
    ratio = np.abs(m1 / bc1) / den
    bm = 16 * u * sm
    bv = 16 * u * (b2 * v + (1 - b2) * gp_terms ** 2)
    bx = 16 * u * np.abs(x) + lrp * (16 * u * ratio + bm / bc1 / den + ratio * bv / (2 * v1 + 1e-300))
    return bx, bm, bv


def test_adam_admm_matches_oracle():
    rng = np.random.default_rng(31)
    A, N = 59, 10_003                      # ragged tail (not a multiple of 4)
    x, g, m, w = (rng.standard_normal((A, N)).astype(np.float32) for _ in range(4))
    v = np.abs(rng.standard_normal((A, N))).astype(np.float32)
    mask = (rng.random(N) < 0.5).astype(np.float32)
    lr, rho = [1e-3, 2e-3, 3e-3, 4e-3, 5e-3], [1e-3, 1e4, 1e4, 1e3, 1e4]
    # the kernel receives its hyper-parameters as FP32; the oracle gets the same values
    f32 = lambda v: [float(np.float32(a)) for a in v]  # noqa: E731
    hp = dict(beta1=f32([0.9])[0], beta2=f32([0.999])[0], eps=f32([1e-8])[0])
    for use_w, use_mask in [(False, False), (True, False), (True, True)]:
        t = {k: torch.from_numpy(a.copy()).cuda() for k, a in dict(x=x, g=g, m=m, v=v, w=w).items()}
        tm = torch.from_numpy(mask).cuda() if use_mask else None
        gs.adam_admm(t["x"], t["g"], t["m"], t["v"], t["w"] if use_w else None, tm, gs.adam_cfg(lr, rho, 7))
        ww, mm = (w if use_w else None), (mask if use_mask else None)
        rx, rm, rv = oracle.adam_admm(x, g, m, v, ww, f32(lr), f32(rho), 7, mask=mm, **hp)
        bx, bm, bv = _adam_bounds(x, g, m, v, ww, f32(lr), f32(rho), 7, mm, hp["beta1"], hp["beta2"], hp["eps"])
        for name, got, ref, bnd in [("x", t["x"], rx, bx), ("m", t["m"], rm, bm), ("v", t["v"], rv, bv)]:
            err = np.abs(got.cpu().numpy() - ref)
            assert (err <= bnd).all(), (name, use_w, use_mask, int((err > bnd).sum()), float((err / bnd).max()))
    # unaligned stride: scalar path
    xs = torch.from_numpy(np.ascontiguousarray(x[:, :N - 1])).cuda()
    big = torch.zeros((A, N), device="cuda")
    big[:, :N - 1] = xs
    sub = big[:, :N - 1]
    gg = torch.from_numpy(np.ascontiguousarray(g[:, :N - 1])).cuda()
    mm = torch.zeros_like(gg)
    vv = torch.zeros_like(gg)
    gs.adam_admm(sub, gg, mm, vv, None, None, gs.adam_cfg(lr, rho, 1))
    z = 0 * g[:, :N - 1]
    rx, _, _ = oracle.adam_admm(x[:, :N - 1], g[:, :N - 1], z, z, None, f32(lr), f32(rho), 1, **hp)
    bx, _, _ = _adam_bounds(x[:, :N - 1], g[:, :N - 1], z, z, None, f32(lr), f32(rho), 1, None, hp["beta1"],
                            hp["beta2"], hp["eps"])
    assert (np.abs(sub.cpu().numpy() - rx) <= bx).all()


def _random_holders(rng, K, G, max_holders, unheld=0.0):
    """Holder CSR over K blocks: each global id is held by 1..max_holders
    blocks (a fraction ``unheld`` by none), locals laid out block by block in
    ascending global id with a padding column after every 97th local copy
    (a column no holder set names)."""
    held = []
    for _ in range(G):
        n = 0 if rng.random() < unheld else int(rng.integers(1, max_holders + 1))
        held.append(sorted(rng.choice(K, n, replace=False)) if n else [])
    cols, local_of, L = [], {}, 0
    for k in range(K):
        for gid in range(G):
            if k in held[gid]:
                local_of[(gid, k)] = L
                cols.append(L)
                L += 1
                if L % 97 == 0:
                    L += 1
    ptr = np.zeros(G + 1, np.int64)
    idx = []
    for gid in range(G):
        idx += [local_of[(gid, k)] for k in held[gid]]
        ptr[gid + 1] = len(idx)
    return ptr, np.asarray(idx, np.int64), L


@pytest.mark.parametrize("deg,max_holders", [(0, 2), (1, 4), (2, 6), (3, 2), (3, 5)])
def test_consensus_matches_oracle(deg, max_holders):
    """z, u, w and the per-group residual sums against the oracle for every
    SH degree (plane count), the 1-2 / 3-4 / more-holder paths, with and
    without over-relaxation and residuals; single-holder duals and columns
    of no holder set keep their values."""
    rng = np.random.default_rng(32 + deg)
    K, G = 6, 2500
    A = 11 + 3 * (deg + 1) ** 2
    ptr, idx, L = _random_holders(rng, K, G, max_holders, unheld=0.02)
    x = rng.standard_normal((A, L)).astype(np.float32)
    u = (0.1 * rng.standard_normal((A, L))).astype(np.float32)
    zp = rng.standard_normal((A, G)).astype(np.float32)
    w0 = rng.standard_normal((A, L)).astype(np.float32)
    held = np.sort(idx)
    free = np.setdiff1d(np.arange(L), held)
    unheld_g = np.nonzero(np.diff(ptr) == 0)[0]
    single = idx[ptr[:-1][np.diff(ptr) == 1]]
    assert len(free) and len(unheld_g) and len(single)
    dptr, didx = torch.from_numpy(ptr).cuda(), torch.from_numpy(idx).cuda()
    for relax in (1.0, 1.6):
        for want_resid in (True, False):
            tx, tu = torch.from_numpy(x).cuda(), torch.from_numpy(u.copy()).cuda()
            tw, tz = torch.from_numpy(w0.copy()).cuda(), torch.from_numpy(zp.copy()).cuda()
            res = torch.zeros(10, device="cuda") if want_resid else None
            gs.consensus(tx, tu, tw, tz, dptr, didx, relax, res)
            rz, ru, rw = oracle.consensus(x, u, ptr, idx, G, relax=relax, z_prev=zp)
            gz, gu, gw = (t.cpu().numpy() for t in (tz, tu, tw))
            hg = np.diff(ptr) > 0
            np.testing.assert_allclose(gz[:, hg], rz[:, hg], rtol=1e-6, atol=1e-6)
            np.testing.assert_allclose(gu[:, held], ru[:, held], rtol=1e-6, atol=1e-6)
            np.testing.assert_allclose(gw[:, held], rw[:, held], rtol=1e-6, atol=1e-6)
            # untouched: columns of no holder, z of unheld ids, u of single holders (bitwise)
            assert np.array_equal(gu[:, free], u[:, free]) and np.array_equal(gw[:, free], w0[:, free])
            assert np.array_equal(gz[:, unheld_g], zp[:, unheld_g])
            assert np.array_equal(gu[:, single], u[:, single])
            if want_resid:
                rp, rd = oracle.residual_sums(x, rz, zp, ptr, idx, G)
                got = res.cpu().numpy().astype(np.float64)
                np.testing.assert_allclose(got[:5], rp, rtol=2e-5)
                np.testing.assert_allclose(got[5:], rd, rtol=2e-5)


def test_dual_rescale_matches_oracle():
    """u *= scale per group, w = z - u over held copies after a consensus
    (groups at scale 1 and zero duals untouched bitwise)."""
    rng = np.random.default_rng(40)
    K, G, deg = 4, 3000, 3
    A = 11 + 3 * (deg + 1) ** 2
    ptr, idx, L = _random_holders(rng, K, G, 3)
    x = rng.standard_normal((A, L)).astype(np.float32)
    u = (0.1 * rng.standard_normal((A, L))).astype(np.float32)
    u[:, idx[ptr[:-1][np.diff(ptr) == 1]]] = 0                  # single holders: duals stay zero
    zp = rng.standard_normal((A, G)).astype(np.float32)
    tx, tu = torch.from_numpy(x).cuda(), torch.from_numpy(u.copy()).cuda()
    tw, tz = torch.zeros_like(tu), torch.from_numpy(zp.copy()).cuda()
    dptr, didx = torch.from_numpy(ptr).cuda(), torch.from_numpy(idx).cuda()
    gs.consensus(tx, tu, tw, tz, dptr, didx, 1.0, None)
    u1, w1, z1 = tu.cpu().numpy(), tw.cpu().numpy(), tz.cpu().numpy()
    scale = (2.0, 0.5, 1.0, 4.0, 0.25)
    gs.dual_rescale(tu, tw, tz, dptr, didx, scale)
    ru, rw = oracle.rescale_duals(u1, z1, ptr, idx, G, scale)
    held = np.sort(idx)
    gu, gw = tu.cpu().numpy(), tw.cpu().numpy()
    np.testing.assert_allclose(gu[:, held], ru[:, held], rtol=1e-6, atol=1e-7)
    np.testing.assert_allclose(gw[:, held], rw[:, held], rtol=1e-6, atol=1e-6)
    s_planes = np.asarray(oracle.penalty_groups(A)) == 2          # group s has scale 1
    assert np.array_equal(gu[s_planes], u1[s_planes]) and np.array_equal(gw[s_planes], w1[s_planes])
    zero = u1 == 0
    assert zero.sum() > 0 and np.array_equal(gw[zero], w1[zero])
    with pytest.raises(gs.GsError, match="scale"):
        gs.dual_rescale(tu, tw, tz, dptr, didx, (1.0, 0.0, 1.0, 1.0, 1.0))


def test_capacity_overflow_reported_then_grown(cfg1):
    cfg = gs.raster_cfg((16, 16))
    frame = make_frame(cfg1, cfg)
    params = torch.from_numpy(cfg1.params).cuda()
    buf = gs.Buffers(frame, 100)
    gs.project(params, frame, cfg, buf)
    gs.bin_sort(frame, cfg, buf)
    c = gs.read_counters(buf)
    assert c["status"] & gs.GS_STATUS_PAIR_OVERFLOW and c["pairs"] > 100
    gs.rasterize(params, frame, cfg, buf)
    assert buf.capacity >= c["pairs"]
    _bins_check(frame, buf)


def test_ragged_image_and_empty_frame():
    """A 100x70 image (partial tiles on both edges) and a frame whose
    Gaussians are all behind the camera."""
    s = scenes.config1()
    cam = scenes.look_at([0.0, 0.4, 2.5], [0, 0, 0], 100, 70, 90.0, 90.0)
    cfg = gs.raster_cfg((16, 16))
    p = s.params[:, :500].copy()
    frame = gs.Frame([cam], [gs.JobSpec(0, 0, 500, 1.0)], cfg)
    buf = gs.rasterize(torch.from_numpy(p).cuda(), frame, cfg)
    ref = oracle.render(p, cam)
    assert_image_close(frame.image(buf.rgb, 0).cpu().numpy().astype(np.float64), ref, ref["flags"])
    behind = p.copy()
    behind[2] += 10.0                       # all Gaussians behind the camera at z = 2.5
    b2 = gs.rasterize(torch.from_numpy(behind).cuda(), frame, cfg)
    assert gs.read_counters(b2)["pairs"] == 0
    assert torch.count_nonzero(b2.rgb).item() == 0
    assert torch.all(b2.T == 1).item()
    grad = torch.empty((p.shape[0], 500), device="cuda")
    gs.render_bwd(torch.from_numpy(behind).cuda(), frame, cfg, b2, grad, gs.LOSS_L1,
                  torch.rand(3 * 100 * 70, device="cuda"))
    assert torch.count_nonzero(grad).item() == 0


def test_f64_path_against_finite_differences():
    """FP64 instantiation of the same kernels: central differences h = 1e-6 of
    L = sum W * C on the 200-Gaussian, 64x64, SH-3 adjoint scene, on every
    one of its 59 x 200 = 11,800 parameters (coordinates whose keep/stop
    decisions flip inside [-h, h] are discarded and counted)."""
    from fd_batch import finite_differences
    s = scenes.config4a()
    cam = s.cams[0]
    cfg = gs.raster_cfg((16, 16))
    frame = gs.Frame([cam], [gs.JobSpec(0, 0, 200, 1.0)], cfg)
    p64 = torch.from_numpy(s.params.astype(np.float64)).cuda()
    rng = np.random.default_rng(41)
    Wt = torch.from_numpy(rng.standard_normal(3 * 64 * 64)).cuda()
    buf = gs.rasterize(p64, frame, cfg)
    grad = torch.empty_like(p64)
    gs.render_bwd(p64, frame, cfg, buf, grad, gs.LOSS_EXTERNAL, Wt)
    g = grad.cpu().numpy()
    # against the oracle's reverse mode (both FP64)
    g_ref = oracle.backward(s.params.astype(np.float64), cam, Wt.cpu().numpy().reshape(3, 64, 64))
    np.testing.assert_allclose(g, g_ref, rtol=1e-7, atol=1e-9 * np.abs(g_ref).max())
    coords = [(a, i) for a in range(59) for i in range(200)]
    print(f"\n[gpu] finite differences on {len(coords)} coordinates", flush=True)
    fd, noise, flipped = finite_differences(p64, cam, Wt, coords, cfg)
    ga = np.array([g[a, i] for a, i in coords])
    bad = (np.abs(fd - ga) > 1e-5 * np.abs(ga) + 1e-9 * np.abs(g).max() + noise) & ~flipped
    used = int((~flipped).sum())
    print(f"[gpu] {used} coordinates compared, {int(flipped.sum())} flipped", flush=True)
    assert used >= 0.9 * len(coords)
    assert (np.abs(ga[~flipped]) > 0).sum() > 5000
    assert not bad.any(), [(coords[k], fd[k], ga[k]) for k in np.nonzero(bad)[0][:10]]


def test_disjoint_and_shared_job_paths_agree(cfg1, gpu1):
    """Four views of one block (jobs share Gaussians: per-Gaussian accumulation
    over jobs) against the same four views on four disjoint copies of the
    block (one thread per record): the copies' gradients sum to the shared
    gradient, and each copy's image equals the shared-job image bit for bit."""
    cfg, frame, params, buf = gpu1
    n = params.shape[1]
    rep = params.repeat(1, 4).contiguous()
    jobs = [gs.JobSpec(v, v * n, (v + 1) * n, 0.25) for v in range(4)]
    f4 = gs.Frame(cfg1.cams, jobs, cfg)
    assert f4.jobs_disjoint == 1 and frame.jobs_disjoint == 0
    b4 = gs.rasterize(rep, f4, cfg)
    for a, b in zip(images(frame, buf), images(f4, b4)):
        np.testing.assert_array_equal(a, b)
    target = frame_target(frame, cfg1, range(4))
    g_shared = torch.empty_like(params)
    gs.render_bwd(params, frame, cfg, buf, g_shared, gs.LOSS_L1, target)
    g_copies = torch.empty_like(rep)
    gs.render_bwd(rep, f4, cfg, b4, g_copies, gs.LOSS_L1, target)
    summed = sum(g_copies[:, v * n:(v + 1) * n].double() for v in range(4))
    torch.testing.assert_close(summed, g_shared.double(), rtol=1e-5, atol=1e-9)
    # Gaussians outside every job get zero gradients
    f2 = gs.Frame(cfg1.cams, [gs.JobSpec(0, 0, n // 2, 1.0)], cfg)
    b2 = gs.rasterize(params, f2, cfg)
    g2 = torch.full_like(params, 7.0)
    gs.render_bwd(params, f2, cfg, b2, g2, gs.LOSS_L1, target[: 3 * 128 * 128])
    assert torch.count_nonzero(g2[:, n // 2:]).item() == 0
    assert torch.count_nonzero(g2[:, : n // 2]).item() > 0


@pytest.mark.parametrize("tile", [(16, 16), (16, 16, -1), (32, 8, 1), (16, 8), (8, 8, -1)])
@pytest.mark.parametrize("size", [(16, 8, 1), (250, 130, 1), (512, 513, 1), (608, 592, 1), (900, 480, 2)])
def test_wavefronts_by_tile_count(cfg1, tile, size):
    """Frames on both sides of the tile counts where the launch's wavefronts
    per tile change: images as with two wavefronts per tile set outright
    (bit for bit; 8x8 tiles: with the plan), gradients equal up to the order
    of their sums, and the same loss.  2,000 Gaussians of the parity scene,
    one of them spanning the image."""
    w, h, views = size
    p = cfg1.params.copy()
    p[scenes.LOGSCALE:scenes.LOGSCALE + 3, 7] = -0.5
    params = torch.from_numpy(p).cuda()
    cams = [scenes.look_at([3 * math.sin(a), 0.0, 3 * math.cos(a)], [0, 0, 0], w, h, 1.2 * w, 1.2 * w)
            for a in (0.3, 1.7)[:views]]
    gen = torch.Generator().manual_seed(5)
    target = torch.rand(3 * w * h * views, generator=gen).cuda()
    out = []
    for t in (tile, (16, 16, 2) if tile[:2] == (16, 16) else (8, 8, 1)):
        cfg = gs.raster_cfg(t)
        frame = gs.Frame(cams, [gs.JobSpec(k, 0, p.shape[1], 0.5) for k in range(views)], cfg)
        buf = gs.rasterize(params, frame, cfg)
        grad = torch.full_like(params, float("nan"))
        loss = torch.zeros(views, device="cuda")
        gs.render_bwd(params, frame, cfg, buf, grad, gs.LOSS_L1, target, loss)
        out.append((buf.rgb.clone(), buf.T.clone(), buf.ncontrib.clone(), grad, loss))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
    if tile[:2] == (16, 16):
        assert torch.equal(out[0][2], out[1][2])
    # the same FP32 terms in another order: per plane, against the plane's norm
    a, b = out[0][3].double(), out[1][3].double()
    assert ((a - b).norm(dim=1) <= 1e-4 * b.norm(dim=1) + 1e-12).all()
    torch.testing.assert_close(out[0][4], out[1][4], rtol=1e-5, atol=0)


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("views", [1, 4])
def test_l1_loss_with_and_without_room_for_its_sum(cfg1, dtype, views):
    """The loss summed per tile in the free end of the backward workspace
    (the same bits every call) and, with a pair capacity of exactly the
    frame's pairs, by the wavefronts' own atomics: both add w mean |C -
    target| to what loss_out holds, and the gradients are the same."""
    cfg = gs.raster_cfg((16, 16))
    frame = make_frame(cfg1, cfg, list(range(views)))
    params = torch.from_numpy(cfg1.params).to("cuda", dtype)
    target = frame_target(frame, cfg1, range(views)).to(dtype)
    pairs = gs.read_counters(gs.rasterize(params, frame, cfg))["pairs"]
    got = []
    for capacity in (pairs, pairs + 1, 4 * pairs, 4 * pairs):
        buf = gs.rasterize(params, frame, cfg, gs.Buffers(frame, capacity, dtype))
        assert buf.capacity == capacity
        loss = torch.full((views,), 0.25, dtype=dtype, device="cuda")
        grad = torch.empty_like(params)
        gs.render_bwd(params, frame, cfg, buf, grad, gs.LOSS_L1, target, loss)
        got.append((loss, grad))
    ref = [0.25 + (frame.image(buf.rgb, k).double() - frame.image(target, k).double()).abs().mean().item() / views
           for k in range(views)]
    for loss, grad in got:
        np.testing.assert_allclose(loss.cpu().numpy(), ref, rtol=2e-6 if dtype == torch.float32 else 1e-13)
        assert torch.equal(grad, got[0][1])
    assert torch.equal(got[2][0], got[3][0])


@pytest.mark.parametrize("form", ["waves", "blocks", "dense"])
@pytest.mark.parametrize("depths", ["uniform", "equal", "clusters", "octaves", "ulps"])
def test_bins_bit_exact_list_lengths_and_depths(form, depths):
    """Tile lists at the edges of the sort's forms (1 .. 64 .. 512 .. 2048 ..
    4096 entries and beyond; the form follows from the pair capacity per
    tile), with depths that spread, all coincide, crowd into two buckets,
    span the exponent range and differ by single bits, on records written
    here: bins against the reference."""
    rng = np.random.default_rng(5)
    lengths = [0, 1, 2, 3, 63, 64, 65, 128, 129, 256, 257, 511, 512, 513, 1025, 2047, 2048, 2049]
    if form != "waves":
        lengths += [4095, 4096, 4097, 9000]
    cam = scenes.look_at([0.0, 0.0, 3.0], [0, 0, 0], 16 * 8, 16 * 10, 100.0, 100.0)
    cfg = gs.raster_cfg((16, 16, -1))
    nt = (cam.width // 16) * (cam.height // 16)
    tiles = rng.permutation(np.repeat(np.arange(len(lengths)), lengths))      # record -> tile
    n = len(tiles)
    d = {"uniform": 1.0 + 3.0 * rng.random(n), "equal": np.full(n, 2.5),
         "clusters": np.where(rng.random(n) < 0.5, 1.0, 4.0) + 1e-6 * rng.random(n),
         "octaves": 2.0 ** rng.uniform(-2, 120, n), "ulps": np.full(n, 2.0)}[depths].astype(np.float32)
    bits = d.view(np.uint32).copy()
    if depths == "ulps":
        bits += rng.integers(0, 40, n).astype(np.uint32)
    lo = ((tiles % 8) | ((tiles // 8) << 16)).astype(np.uint32)
    meta = np.stack([bits, np.ones(n, np.uint32), lo, lo], axis=1)
    frame = gs.Frame([cam], [gs.JobSpec(0, 0, n, 1.0)], cfg)
    assert frame.n_tiles == nt
    per_tile = {"waves": 150, "blocks": 1024, "dense": 1200}[form]
    assert n <= per_tile * nt
    buf = gs.Buffers(frame, per_tile * nt)
    buf.meta.copy_(torch.from_numpy(meta.view(np.int32).reshape(-1)))
    gs.bin_sort(frame, cfg, buf)
    _bins_check(frame, buf)


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("views", [2, 3, 4, 5, 9])
@pytest.mark.parametrize("n", [1, 63, 64, 129, 700])
def test_shared_gaussians_backward_adds_the_jobs(dtype, views, n):
    """Jobs that share Gaussians, over whole and partial overlapping ranges:
    the gradient equals the sum, in job order, of each job's own (a frame of
    that job alone), over a buffer of NaN; Gaussians in no job get zero."""
    p = scenes.gaussians(n, 2, 77, [-1, -1, -1], [1, 1, 1], -2.5, 0.5)
    params = torch.from_numpy(p).to("cuda", dtype)
    cfg = gs.raster_cfg((16, 16))
    cams = [scenes.look_at([3 * math.sin(a), 0.2, 3 * math.cos(a)], [0, 0, 0], 48, 40, 60.0, 60.0)
            for a in np.linspace(0.1, 5.0, views)]
    jobs = [gs.JobSpec(k, (k % 3) * (n // 5), n - (k % 2) * (n // 7) - n // 10, 0.5 + k) for k in range(views)]
    frame = gs.Frame(cams, jobs, cfg)
    assert not frame.jobs_disjoint
    dl = torch.randn(3 * frame.n_pixels, generator=torch.Generator().manual_seed(n)).to("cuda", dtype)
    buf = gs.rasterize(params, frame, cfg)
    grad = torch.full_like(params, float("nan"))
    gs.render_bwd(params, frame, cfg, buf, grad, gs.LOSS_EXTERNAL, dl)
    total = torch.zeros_like(params)
    for k in range(views):
        fk = gs.Frame([cams[k]], [gs.JobSpec(0, jobs[k].g0, jobs[k].g1, 1.0)], cfg)
        bk = gs.rasterize(params, fk, cfg)
        gk = torch.empty_like(params)
        gs.render_bwd(params, fk, cfg, bk, gk, gs.LOSS_EXTERNAL, frame.image(dl, k).reshape(-1).contiguous())
        total += gk
    assert torch.equal(grad, total)


def _holder_runs(rng, G):
    """Holder CSR of G ids in runs of one holder set with consecutive columns:
    runs of 1 .. 300 ids (inside a lane's four, over several wavefronts), 0 to
    3 holders, columns that jump between runs.  Returns (ptr, idx, columns)."""
    sets, nxt = [], 0
    while len(sets) < G:
        n = min(int(rng.choice([1, 2, 3, 4, 5, 7, 64, 130, 300])), G - len(sets))
        first = []
        for _ in range(int(rng.choice([0, 1, 1, 1, 2, 2, 2, 3]))):
            nxt += int(rng.integers(0, 3))
            first.append(nxt)
            nxt += n
        sets += [[c + i for c in first] for i in range(n)]
    ptr = np.concatenate([[0], np.cumsum([len(h) for h in sets])]).astype(np.int64)
    return ptr, np.asarray([c for h in sets for c in h], np.int64), nxt + 3


def _consensus(x, u, z, ptr, idx, relax):
    """gs.consensus on copies; w starts at 7.  Returns u, w, z, residual sums."""
    t = [torch.from_numpy(v.reshape(-1).copy().reshape(v.shape)).cuda() for v in (x, u, np.full_like(u, 7.0), z)]
    res = torch.zeros(10, device="cuda")
    dev = [torch.from_numpy(v.copy() if len(v) else np.zeros(1, np.int64)).cuda() for v in (ptr, idx)]
    gs.consensus(*t, *dev, relax, res)
    return [v.cpu().numpy() for v in t[1:]] + [res.cpu().numpy()]


@pytest.mark.parametrize("relax", [1.0, 1.6])
@pytest.mark.parametrize("G,deg", [(1, 0), (3, 3), (257, 2), (1029, 3), (1029, 1)])
def test_consensus_runs_of_ids_match_oracle(G, deg, relax):
    """z, u, w and the residual sums against the oracle, columns of no holder
    and ids of no holder untouched, and the same bits as the same ids in
    another order."""
    rng = np.random.default_rng(G + deg)
    A = 11 + 3 * (deg + 1) ** 2
    ptr, idx, L = _holder_runs(rng, G)
    x = rng.standard_normal((A, L)).astype(np.float32)
    u = (0.1 * rng.standard_normal((A, L))).astype(np.float32)
    zp = rng.standard_normal((A, G)).astype(np.float32)
    held, hg = np.sort(idx), np.diff(ptr) > 0
    gu, gw, gz, res = _consensus(x, u, zp, ptr, idx, relax)
    perm = rng.permutation(G)
    pptr = np.concatenate([[0], np.cumsum(np.diff(ptr)[perm])])
    pidx = np.concatenate([idx[ptr[g]:ptr[g + 1]] for g in perm])
    pu, pw, pz, _ = _consensus(x, u, zp[:, perm], pptr, pidx, relax)
    assert np.array_equal(gu, pu) and np.array_equal(gw, pw)
    assert np.array_equal(gz[:, perm][:, hg[perm]], pz[:, hg[perm]])
    rz, ru, rw = oracle.consensus(x, u, ptr, idx, G, relax=relax, z_prev=zp)
    np.testing.assert_allclose(gz[:, hg], rz[:, hg], rtol=1e-6, atol=1e-6)
    np.testing.assert_allclose(gu[:, held], ru[:, held], rtol=1e-6, atol=1e-6)
    np.testing.assert_allclose(gw[:, held], rw[:, held], rtol=1e-6, atol=1e-6)
    free = np.setdiff1d(np.arange(L), held)
    assert np.array_equal(gu[:, free], u[:, free]) and (gw[:, free] == 7.0).all()
    assert np.array_equal(gz[:, ~hg], zp[:, ~hg])
    rp, rd = oracle.residual_sums(x, rz, zp, ptr, idx, G)
    np.testing.assert_allclose(res[:5], rp, rtol=2e-5, atol=1e-6)
    np.testing.assert_allclose(res[5:], rd, rtol=2e-5, atol=1e-6)


@pytest.mark.parametrize("relax", [1.0, 1.6])
@pytest.mark.parametrize("deg", [0, 1, 2, 3])
def test_consensus_of_many_ids_equals_its_parts(deg, relax):
    """Past 131,072 ids (lanes of four ids) the bits equal those of two calls
    on parts of the ids below that (one id per lane), and the residual sums
    agree to their rounding."""
    rng = np.random.default_rng(deg)
    G, A = 131_072 + 1029, 11 + 3 * (deg + 1) ** 2
    ptr, idx, L = _holder_runs(rng, G)
    x = rng.standard_normal((A, L), dtype=np.float32)
    u = 0.1 * rng.standard_normal((A, L), dtype=np.float32)
    zp = rng.standard_normal((A, G), dtype=np.float32)
    gu, gw, gz, res = _consensus(x, u, zp, ptr, idx, relax)
    half, total = 70_001, np.zeros(10)
    wu, ww, wz = u.copy(), np.full_like(u, 7.0), zp.copy()
    for a, b in ((0, half), (half, G)):
        ha, hb = ptr[a], ptr[b]
        pu, pw, pz, pr = _consensus(x, u, np.ascontiguousarray(zp[:, a:b]), ptr[a:b + 1] - ha, idx[ha:hb], relax)
        cols = idx[ha:hb]
        wu[:, cols], ww[:, cols], wz[:, a:b] = pu[:, cols], pw[:, cols], pz
        total += pr
    assert np.array_equal(gu, wu) and np.array_equal(gw, ww) and np.array_equal(gz, wz)
    np.testing.assert_allclose(res, total, rtol=1e-4)


@pytest.mark.parametrize("jobs", [1, 3])
@pytest.mark.parametrize("n", [1, 255, 256, 257, 512, 513, 2047, 2048, 2049, 8192, 8193])
@pytest.mark.parametrize("room", ["all", "exact", "half", "one"])
def test_bins_of_small_frames(n, jobs, room):
    """Frames on both sides of the record counts where one launch makes the
    bins (2048 and 8192 records a job; more: by strips): most records in
    one tile, the others' rectangles up to the whole image, culled ones among
    them, depths with ties.  Bins, first pairs and counters against pairs
    listed here in record order; with fewer pairs of capacity than the frame
    has, the lists of the first `capacity` pairs, and the overflow is
    reported and counted."""
    rng = np.random.default_rng(n + jobs)
    cams = [scenes.look_at([0.0, 0.0, 3.0], [0, 0, 0], 100 + 30 * k, 70, 100.0, 100.0) for k in range(jobs)]
    cfg = gs.raster_cfg((16, 16))
    frame = gs.Frame(cams, [gs.JobSpec(k, 0, n, 1.0) for k in range(jobs)], cfg)
    meta = np.zeros((frame.n_records, 4), np.uint32)
    lists, first = [], []
    for k in range(jobs):
        j = frame.job(k)
        x0, y0 = rng.integers(0, j.tiles_x, n), rng.integers(0, j.tiles_y, n)
        x1 = np.minimum(x0 + rng.integers(0, 3, n), j.tiles_x - 1)
        y1 = np.minimum(y0 + rng.integers(0, 3, n), j.tiles_y - 1)
        one = rng.random(n) < 0.8
        x0[one], x1[one], y0[one], y1[one] = 1, 1, 2, 2
        x0[n // 2], x1[n // 2], y0[n // 2], y1[n // 2] = 0, j.tiles_x - 1, 0, j.tiles_y - 1
        m = meta[j.rec0:j.rec0 + n]
        m[:, 0] = (1.0 + rng.integers(0, 50, n) / 16.0).astype(np.float32).view(np.uint32)
        m[:, 1] = (x1 - x0 + 1) * (y1 - y0 + 1)
        m[:, 2], m[:, 3] = x0 | (y0 << 16), x1 | (y1 << 16)
        culled = rng.random(n) < 0.1
        culled[n // 2] = False
        m[culled] = [0xffffffff, 0, 0, 0]
        for i in range(n):
            first.append(len(lists))
            if not culled[i]:
                lists += [(j.tile0 + y * j.tiles_x + x, int(m[i, 0]), j.rec0 + i)
                          for y in range(y0[i], y1[i] + 1) for x in range(x0[i], x1[i] + 1)]
    pairs = len(lists)
    capacity = {"all": 2 * pairs + 7, "exact": pairs, "half": (pairs + 1) // 2, "one": 1}[room]
    buf = gs.Buffers(frame, capacity)
    buf.meta.copy_(torch.from_numpy(meta.view(np.int32).reshape(-1)))
    buf.ranges.fill_(99)
    for call in (1, 2):
        gs.bin_sort(frame, cfg, buf)
    c = gs.read_counters(buf)
    over = pairs > buf.capacity
    assert (c["visible"], c["pairs"]) == (int((meta[:, 1] > 0).sum()), pairs)
    assert bool(c["status"] & gs.GS_STATUS_PAIR_OVERFLOW) == over and c["overflowed"] == (2 if over else 0)
    kept = sorted(lists[:buf.capacity])
    vals = buf.vals.cpu().numpy().view(np.uint32)
    assert vals[:len(kept)].tolist() == [r for _, _, r in kept]
    tiles = np.asarray([t for t, _, _ in kept])
    ranges = np.zeros((frame.n_tiles, 2), np.int64)
    for t in np.unique(tiles):
        at = np.nonzero(tiles == t)[0]
        ranges[t] = at[0], at[-1] + 1
    np.testing.assert_array_equal(buf.ranges.view(-1, 2).cpu().numpy(), ranges)
    vis = meta[:, 1] > 0
    np.testing.assert_array_equal(buf.pair_off.cpu().numpy()[vis], np.asarray(first)[vis])


def _bins_of(frame, cfg, meta, capacity):
    buf = gs.Buffers(frame, capacity)
    buf.meta.copy_(torch.from_numpy(meta.view(np.int32).reshape(-1)))
    buf.ranges.fill_(99)
    gs.bin_sort(frame, cfg, buf)
    return buf


def _expect_bins(frame, buf, meta):
    """vals, ranges, first pairs and counters against the first `capacity` of
    all pairs, listed here in record order."""
    n = meta[:, 1].astype(np.int64)
    rec = np.repeat(np.arange(len(meta)), n)
    first = np.cumsum(n) - n
    k = np.arange(len(rec)) - first[rec]                          # pair of its record
    x0, y0 = (meta[rec, 2] & 0xFFFF).astype(np.int64), (meta[rec, 2] >> 16).astype(np.int64)
    w = (meta[rec, 3] & 0xFFFF) - x0 + 1
    tile = np.empty(len(rec), np.int64)
    for j in range(frame.n_jobs):
        b = frame.job(j)
        own = (rec >= b.rec0) & (rec < b.rec0 + b.g1 - b.g0)
        tile[own] = b.tile0 + (y0[own] + k[own] // w[own]) * b.tiles_x + x0[own] + k[own] % w[own]
    c = gs.read_counters(buf)
    over = len(rec) > buf.capacity
    assert (c["visible"], c["pairs"], c["overflowed"]) == (int((n > 0).sum()), len(rec), int(over))
    rec, tile = rec[:buf.capacity], tile[:buf.capacity]
    order = np.lexsort((rec, meta[rec, 0], tile))
    got = buf.vals[:len(rec)].cpu().numpy().view(np.uint32)
    np.testing.assert_array_equal(got, rec[order])
    ranges = np.zeros((frame.n_tiles, 2), np.int64)
    count = np.bincount(tile, minlength=frame.n_tiles)
    ranges[:, 1] = np.cumsum(count)
    ranges[:, 0] = ranges[:, 1] - count
    ranges[count == 0] = 0
    np.testing.assert_array_equal(buf.ranges.view(-1, 2).cpu().numpy(), ranges)
    np.testing.assert_array_equal(buf.pair_off.cpu().numpy()[n > 0], first[n > 0])
    plan = np.sort(buf.tile_order[4:4 + frame.n_tiles].cpu().numpy())
    assert np.array_equal(plan, np.arange(frame.n_tiles))


@pytest.mark.parametrize("room", ["all", "exact", "half"])
@pytest.mark.parametrize("n,w,h,jobs", [(8193, 16, 16, 1), (8193, 17, 16, 2), (9000, 16 * 191, 16, 1),
                                        (9000, 16 * 193, 16, 2), (5000, 700, 420, 2), (20000, 330, 500, 1),
                                        (20227, 160, 128, 1), (65535, 800, 410, 1), (65537, 800, 410, 1),
                                        (32768, 790, 400, 2)])
def test_bins_by_strips(n, w, h, jobs, room):
    """Frames of some thousand records (up to 65,536, or 20,224 in 80 tiles):
    strips of one tile to a whole row, ragged at the row's end, strips' lists
    on both sides of 4096 entries and tiles' of 2048 and 8192, rectangles from
    one tile to the image, equal depths, culled records."""
    rng = np.random.default_rng(n + w)
    cams = [scenes.look_at([0.0, 0.0, 3.0], [0, 0, 0], w + 16 * k, h, 100.0, 100.0) for k in range(jobs)]
    cfg = gs.raster_cfg((16, 16, -1))
    frame = gs.Frame(cams, [gs.JobSpec(k, 0, n, 1.0) for k in range(jobs)], cfg)
    meta = np.zeros((frame.n_records, 4), np.uint32)
    for k in range(jobs):
        j = frame.job(k)
        x0, y0 = rng.integers(0, j.tiles_x, n), rng.integers(0, j.tiles_y, n)
        one = rng.random(n) < 0.2 + 0.3 * k                       # these crowd into one tile
        x0[one], y0[one] = j.tiles_x // 2, j.tiles_y // 2
        x1 = np.minimum(x0 + np.where(one, 0, rng.integers(0, 4, n)), j.tiles_x - 1)
        y1 = np.minimum(y0 + np.where(one, 0, rng.integers(0, 3, n)), j.tiles_y - 1)
        full = rng.random(n) < 4.0 / n
        x0[full], y0[full], x1[full], y1[full] = 0, 0, j.tiles_x - 1, j.tiles_y - 1
        m = meta[j.rec0:j.rec0 + n]
        m[:, 0] = (1.0 + rng.integers(0, 500, n) / 16.0).astype(np.float32).view(np.uint32)
        m[:, 1], m[:, 2], m[:, 3] = (x1 - x0 + 1) * (y1 - y0 + 1), x0 | (y0 << 16), x1 | (y1 << 16)
        m[rng.random(n) < 0.1] = [0xffffffff, 0, 0, 0]
    pairs = int(meta[:, 1].sum())
    buf = _bins_of(frame, cfg, meta, {"all": 2 * pairs + 7, "exact": pairs, "half": pairs // 2}[room])
    _expect_bins(frame, buf, meta)


@pytest.mark.parametrize("size", [(16, 16), (32, 16), (48, 16), (13 * 16, 16), (16 * 16, 16 * 17), (16 * 96, 16 * 87)])
@pytest.mark.parametrize("mean", [40, 300, 1000, 1100])
def test_bins_of_many_records(size, mean):
    """More records than go by strips (most of them culled): no radix pass to
    two, tile lists at the edges of every form of the tile sort, which follows
    from the pair capacity per tile and the number of tiles."""
    rng = np.random.default_rng(size[0] + mean)
    cam = scenes.look_at([0.0, 0.0, 3.0], [0, 0, 0], *size, 100.0, 100.0)
    cfg = gs.raster_cfg((16, 16, -1))
    tx, nt = size[0] // 16, size[0] // 16 * (size[1] // 16)
    lengths = [0, 1, 2, 3, 63, 64, 65, 128, 129, 256, 257, 511, 512, 513, 1025, 2047, 2048, 2049, 4096, 4097, 9000]
    tiles = np.repeat(rng.permutation(max(nt, len(lengths)))[:len(lengths)], lengths) % nt
    n = 70_000
    rec = np.sort(rng.permutation(n)[:len(tiles)])
    tiles = rng.permutation(tiles)
    meta = np.zeros((n, 4), np.uint32)
    meta[:, 0] = 0xffffffff
    meta[rec, 0] = (1.0 + rng.integers(0, 3000, len(rec)) / 16.0).astype(np.float32).view(np.uint32)
    meta[rec, 1] = 1
    meta[rec, 2] = meta[rec, 3] = (tiles % tx) | (tiles // tx << 16)
    frame = gs.Frame([cam], [gs.JobSpec(0, 0, n, 1.0)], cfg)
    assert frame.n_tiles == nt
    buf = _bins_of(frame, cfg, meta, max(mean * nt, len(rec)))
    _expect_bins(frame, buf, meta)


@pytest.mark.parametrize("room", ["all", "half"])
@pytest.mark.parametrize("jobs,n,tx,ty", [(1, 9000, 1, 2000), (3, 3000, 2, 200), (16, 300, 4, 100), (64, 200, 4, 5),
                                          (65, 200, 4, 4), (200, 50, 3, 3), (130, 60, 17, 1), (2, 5000, 200, 3),
                                          (24, 2048, 1, 1), (25, 2000, 1, 1)])
def test_bins_by_strips_of_many_and_narrow_views(jobs, n, tx, ty, room):
    """Strips that hold several rows of a view, strips of up to 200 views,
    views of different sizes; records over one tile to the whole view; and
    views of a few tiles on both sides of the 49,152 records up to which one
    launch makes the bins."""
    rng = np.random.default_rng(n + tx)
    cams = [scenes.look_at([0.0, 0.0, 3.0], [0, 0, 0], 16 * (tx + k % 3), 16 * (ty + k % 2), 100.0, 100.0)
            for k in range(jobs)]
    cfg = gs.raster_cfg((16, 16, -1))
    frame = gs.Frame(cams, [gs.JobSpec(k, 0, n, 1.0) for k in range(jobs)], cfg)
    meta = np.zeros((frame.n_records, 4), np.uint32)
    for k in range(jobs):
        j = frame.job(k)
        x0, y0 = rng.integers(0, j.tiles_x, n), rng.integers(0, j.tiles_y, n)
        x1 = np.minimum(x0 + rng.integers(0, 4, n), j.tiles_x - 1)
        y1 = np.minimum(y0 + rng.integers(0, 12, n), j.tiles_y - 1)
        x0[0], y0[0], x1[0], y1[0] = 0, 0, j.tiles_x - 1, j.tiles_y - 1
        m = meta[j.rec0:j.rec0 + n]
        m[:, 0] = (1.0 + rng.integers(0, 50, n) / 16.0).astype(np.float32).view(np.uint32)
        m[:, 1], m[:, 2], m[:, 3] = (x1 - x0 + 1) * (y1 - y0 + 1), x0 | (y0 << 16), x1 | (y1 << 16)
        m[rng.random(n) < 0.1] = [0xffffffff, 0, 0, 0]
    pairs = int(meta[:, 1].sum())
    _expect_bins(frame, _bins_of(frame, cfg, meta, 2 * pairs if room == "all" else pairs // 2), meta)


@pytest.mark.parametrize("form", ["waves", "blocks", "dense"])
@pytest.mark.parametrize("depths", ["uniform", "equal", "clusters", "octaves", "ulps"])
def test_tile_sort_forms_by_list_length_and_depths(form, depths):
    """As test_bins_bit_exact_list_lengths_and_depths on frames that take the
    tile sort: 70,000 records, most of them culled, so that neither one launch
    nor strips make the bins, and for the wavefronts' form 2,080 tiles with
    pair capacity for 150 entries each (workgroups of 256: 1024, of 512:
    1200, in 80 tiles).  Wavefronts' lists of 2 to 512 entries have crowded
    buckets (equal depths, clusters, octaves) and depths within fewer values
    than buckets (ulps)."""
    rng = np.random.default_rng(7)
    lengths = [0, 1, 2, 3, 63, 64, 65, 128, 129, 200, 256, 257, 400, 511, 512, 513, 1025, 2047, 2048, 2049]
    tx, ty, per_tile = {"waves": (40, 52, 150), "blocks": (8, 10, 1024), "dense": (8, 10, 1200)}[form]
    if form != "waves":
        lengths += [4095, 4096, 4097, 9000]
    cam = scenes.look_at([0.0, 0.0, 3.0], [0, 0, 0], 16 * tx, 16 * ty, 100.0, 100.0)
    cfg = gs.raster_cfg((16, 16, -1))
    at = rng.permutation(tx * ty)[:len(lengths)]
    tiles = rng.permutation(np.repeat(at, lengths))               # of the visible records, in order
    n, m = 70_000, len(tiles)
    d = {"uniform": 1.0 + 3.0 * rng.random(m), "equal": np.full(m, 2.5),
         "clusters": np.where(rng.random(m) < 0.5, 1.0, 4.0) + 1e-6 * rng.random(m),
         "octaves": 2.0 ** rng.uniform(-2, 120, m), "ulps": np.full(m, 2.0)}[depths].astype(np.float32)
    bits = d.view(np.uint32).copy()
    if depths == "ulps":
        bits += rng.integers(0, 40, m).astype(np.uint32)
    meta = np.zeros((n, 4), np.uint32)
    meta[:, 0] = 0xffffffff
    rec = np.sort(rng.permutation(n)[:m])
    meta[rec, 0], meta[rec, 1] = bits, 1
    meta[rec, 2] = meta[rec, 3] = (tiles % tx) | (tiles // tx << 16)
    frame = gs.Frame([cam], [gs.JobSpec(0, 0, n, 1.0)], cfg)
    assert frame.n_tiles == tx * ty and m <= per_tile * tx * ty
    gs.profile_set(["k_tile_sort", "k_bin_small", "k_bin_strips"])
    try:
        buf = _bins_of(frame, cfg, meta, per_tile * tx * ty)
        ran = [gs.profile_get(k)[1] for k in ("k_tile_sort", "k_bin_small", "k_bin_strips")]
    finally:
        gs.profile_set(None)
    assert ran == [1, 0, 0]
    _expect_bins(frame, buf, meta)


@pytest.fixture(scope="module")
def many_tiles(cfg1):
    """2,000 Gaussians of the parity scene, one of them spanning the image, in
    3,776 tiles: above every tile count up to which a launch takes more
    wavefronts than the configuration's one or the plan's."""
    w, h = 1024, 944
    p = cfg1.params.copy()
    p[scenes.LOGSCALE:scenes.LOGSCALE + 3, 7] = -0.5
    cam = scenes.look_at([3 * math.sin(0.3), 0.0, 3 * math.cos(0.3)], [0, 0, 0], w, h, 1.2 * w, 1.2 * w)
    target = torch.rand(3 * w * h, generator=torch.Generator().manual_seed(5))

    def run(tile, dtype, share):
        params = torch.from_numpy(p).to("cuda", dtype)
        cfg = gs.raster_cfg(tile)
        frame = gs.Frame([cam], [gs.JobSpec(0, 0, p.shape[1], 1.0)], cfg)
        assert frame.n_tiles > 3600
        buf = gs.Buffers(frame, 1 << 18, dtype)
        buf.share_qmask = share
        gs.rasterize(params, frame, cfg, buf)
        assert 2 * gs.read_counters(buf)["pairs"] < buf.capacity          # room for the loss's sum
        grad = torch.full_like(params, float("nan"))
        loss = torch.zeros(1, dtype=dtype, device="cuda")
        gs.render_bwd(params, frame, cfg, buf, grad, gs.LOSS_L1, target.to("cuda", dtype), loss)
        return buf.rgb, buf.T, buf.ncontrib, grad, loss

    return run


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("tile", [(16, 16, 1), (16, 16, -1), (16, 16, 1, -1), (16, 16, -1, 1), (16, 16, 4, 1),
                                  (16, 16, 1, 4), (16, 16, 4, -1), (32, 8, 1), (32, 8, -1), (32, 8, -1, 2)])
def test_one_wavefront_and_the_plan_in_frames_of_many_tiles(many_tiles, tile, dtype):
    """The kernels of one wavefront per tile and of the plan, which smaller
    frames do not reach, in both precisions and mixed with splits: the images
    of two wavefronts per tile set outright bit for bit, its gradients up to
    the order of their sums, its loss; and the same bits, the loss's among
    them, whether the backward takes the forward's quadrant masks or makes
    its own."""
    rgb, T, nc, grad, loss = many_tiles(tile, dtype, True)
    ref = many_tiles((*tile[:2], 2), dtype, True)
    assert torch.equal(rgb, ref[0]) and torch.equal(T, ref[1]) and torch.equal(nc, ref[2])
    # the same terms in another order: per plane, against the plane's norm
    bound = 1e-4 if dtype == torch.float32 else 1e-12
    a, b = grad.double(), ref[3].double()
    assert ((a - b).norm(dim=1) <= bound * b.norm(dim=1) + 1e-12).all()
    torch.testing.assert_close(loss, ref[4], rtol=1e-5 if dtype == torch.float32 else 1e-12, atol=0)
    own = many_tiles(tile, dtype, False)
    assert all(torch.equal(x, y) for x, y in zip((rgb, T, nc, grad, loss), own))
