"""Renders of 2^18 to 2^20 rays, which take two lanes per ray by default: whole
frames against the oracle, in one view and in several, with image sizes that
leave remainders of the 16 x 8 pixel tiles, every record width (a D that is
filled up, an exact one, one beyond the widest record), world and NDC rays,
stratified samples, no termination and a single sample."""
import dataclasses

import numpy as np
import pytest

import oracle
from paper_2204_02585_amd import scenes
from tests import parity_util as pu

pytestmark = pytest.mark.gpu

CASES = [
    dict(width=515, height=511, n_samples=48, D=8, dtype="f16"),
    dict(width=641, height=410, n_samples=33, D=4, dtype="f16", sigma_dtype="f32", n_poses=1),
    dict(width=300, height=293, n_samples=40, D=12, dtype="f32", n_poses=3, stratified=True),
    dict(width=515, height=513, n_samples=48, D=16, dtype="f16", t_eps=0.0),
    dict(width=520, height=505, n_samples=20, D=20, dtype="f32"),
    dict(width=513, height=512, n_samples=1, D=1, dtype="f16", stratified=True),
    dict(width=517, height=509, n_samples=64, D=8, dtype="f32", forward=True),
    dict(width=362, height=365, n_samples=31, D=13, dtype="f16", forward=True, n_poses=2),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"{c['width']}x{c['height']}x{c.get('n_poses', 1)}-D{c['D']}")
def test_whole_frames(case):
    base = scenes.CONFIGS["llff_tiny" if case.get("forward") else "tiny"]
    cfg = dataclasses.replace(base, name="two_lanes", number=300 + case["D"], n_p=61, n_blobs=24, sigma_max=200.0,
                              focal=(0.8 if case.get("forward") else 1.25) * case["width"], **case)
    rays = cfg.width * cfg.height * cfg.n_poses
    assert 1 << 18 <= rays < 1 << 20
    sc = scenes.make_scene(cfg)
    gpu = pu.gpu_render(sc)
    ref = oracle.render_scene(sc)
    pu.compare(gpu, ref, np.arange(ref.size), pu.scene_atol(sc), f"two lanes {case}")


@pytest.mark.parametrize("D", [1, 7, 8, 9, 12, 16, 17, 32])
@pytest.mark.parametrize("dtypes", [("f16", "f32"), ("f32", "f16")])
def test_filled_records_equal_padded_input(D, dtypes):
    """A D below the stored width renders as the same arrays padded with zero
    components by the caller (uvw and beta of different types: both widths
    of the fill; Eq. 5 maps padded alike)."""
    import torch
    from paper_2204_02585_amd import binding
    rng = np.random.Generator(np.random.PCG64(D))
    tmap = {"f16": torch.float16, "f32": torch.float32}
    DS = 8 if D <= 8 else (16 if D <= 16 else D)
    n_p, nt, nph = 37, 5, 9
    cfg = dataclasses.replace(scenes.CONFIGS["tiny"], n_p=n_p, number=400 + D)
    blobs = scenes.make_blobs(16, 200.0, 0.1, 0.4, 1)
    poses = torch.from_numpy(scenes.spiral_poses(2)).cuda()
    uvw = [rng.uniform(-1, 1, (n_p, n_p, 3, D)).astype(np.float32) for _ in range(3)]
    beta = rng.uniform(-1, 1, (nt, nph, D)).astype(np.float32)
    dec = scenes.linear_decoder(3, D, 50.0, 5)

    def tensors(width):
        pad = [(0, 0)] * 3 + [(0, width - D)]
        u = [torch.from_numpy(np.pad(a, pad).reshape(n_p, n_p, 3 * width)).cuda().to(tmap[dtypes[0]]) for a in uvw]
        return u, torch.from_numpy(np.pad(beta, pad[1:])).cuda().to(tmap[dtypes[1]])

    def decoder(width):
        w = np.zeros((3, width, 3, width), np.float32)
        w[:, :D, :, :D] = dec.w_uvw.reshape(3, D, 3, D)
        return scenes.LinearDecoder(dec.w_sigma, dec.b_sigma, w.reshape(3, width, 3 * width),
                                    np.pad(dec.b_uvw, [(0, 0), (0, width - D)]))

    for linear in (False, True):
        planes = (scenes.bake_linear_sigma_planes(n_p, blobs, 3) if linear else scenes.bake_sigma_planes(n_p, blobs))
        sig = [torch.from_numpy(p).cuda() for p in planes]
        out = []
        for width in (D, DS):
            u, b = tensors(width)
            caches = binding.Caches(sig, u, b, scenes.BOX_MIN, scenes.BOX_MAX, decoder=decoder(width) if linear else None)
            try:
                rgb, depth = caches.render(poses, dict(fx=60.0, fy=60.0, cx=24.0, cy=20.0, width=48, height=40),
                                           2.0, 6.0, 64)
                torch.cuda.synchronize()
                out.append((rgb.cpu().numpy(), depth.cpu().numpy()))
            finally:
                caches.close()
        assert np.abs(out[0][0]).max() > 0.0
        # the same kernel on the same records; the order of the binary64 sums
        # of a ray may differ by a unit in the last place of binary32
        assert np.abs(out[0][0] - out[1][0]).max() <= 1e-7, (D, linear)
        assert np.abs(out[0][1] - out[1][1]).max() <= 1e-6, (D, linear)


def test_recreate_keeps_records_the_block_has_no_room_to_fill():
    """A handle whose block fits D = 7 records only as they are (a larger grid
    than it was made for) still takes them."""
    import torch
    from paper_2204_02585_amd import binding
    small = dataclasses.replace(scenes.CONFIGS["tiny"], n_p=64, D=8, dtype="f16", number=501)
    large = dataclasses.replace(small, n_p=67, D=7, number=502)
    handle = binding.caches_from_scene(scenes.make_scene(small))
    try:
        sc = scenes.make_scene(large)
        dev = lambda a: torch.from_numpy(a).cuda()  # noqa: E731
        handle.recreate([dev(a) for a in sc.sigma], [dev(a) for a in sc.uvw], dev(sc.beta), sc.bbox_min, sc.bbox_max,
                        t_eps=large.t_eps, seed=sc.seed)
        P = dev(sc.poses)
        rgb, depth, st = handle.render_stats(P, sc.intrinsics, sc.near, sc.far, large.n_samples)
        torch.cuda.synchronize()
        gpu = (rgb.cpu().numpy().reshape(-1, 3), depth.cpu().numpy().reshape(-1),
               st.cpu().numpy().view(np.uint32).reshape(-1, 4))
        ref = oracle.render_scene(sc)
        pu.compare(gpu, ref, np.arange(ref.size), pu.scene_atol(sc), "recreate without fill")
    finally:
        handle.close()
