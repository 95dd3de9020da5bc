"""Create-time preparation at the sizes where its tiles, caps and remainders
can go wrong.  Distances: a march that leaps by the distance fields (and the
linear decoder's cell grid) must find the very samples that a dense march of
the same handle finds, which reads no distance; sparse planes make the
distances reach the 255-texel cap.  Records and copies, which both marches
read: whole frames against the CPU oracle, which reads the caller's arrays.
"""
import numpy as np
import pytest

import oracle
from paper_2204_02585_amd import scenes
from tests import parity_util as pu

pytestmark = pytest.mark.gpu


def _planes(n_p, rng, density, channels=0):
    """Planes that are zero but for a few texels (and NaN in one, which counts
    as occupied for the distances and as empty for the density)."""
    out = []
    for j in range(3):
        live = rng.random((n_p, n_p)) < density
        # a band along each axis keeps some rays occupied in all planes
        live[n_p // 3:n_p // 3 + 2 + n_p // 40, :] = True
        live[:, n_p // 2:n_p // 2 + 2 + n_p // 40] = True
        if channels:
            p = rng.uniform(0.2, 1.0, (n_p, n_p, channels)) * live[..., None]
        else:
            p = rng.uniform(1.0, 4.0, (n_p, n_p)) * live
        if j == 1:
            p[n_p - 1, 0] = np.nan
        out.append(p.astype(np.float32))
    return out


def _renders(caches, poses, n):
    import torch
    intr = dict(fx=30.0, fy=30.0, cx=12.0, cy=9.5, width=24, height=19)
    got = []
    for skip in (True, False):
        caches.set_empty_space_skipping(skip)
        rgb, depth, stats = caches.render_stats(poses, intr, 2.0, 6.0, n)
        torch.cuda.synchronize()
        got.append([t.cpu().numpy() for t in (rgb, depth, stats)])
    return got


def _check(caches, poses, n, label):
    (rgb, depth, stats), (rgb_d, depth_d, stats_d) = _renders(caches, poses, n)
    print(f"[prepare {label}] occupied samples {int(stats_d[..., 2].sum())}", flush=True)
    assert np.array_equal(stats, stats_d), label
    # the same samples in another order of the binary64 sums: a few units in
    # the last place of binary32 (rgb <= 1, depth <= 6)
    assert np.abs(rgb - rgb_d).max() <= 1e-6 and np.abs(depth - depth_d).max() <= 6e-6, label
    return rgb, stats


# below, at and past the 16-row, 64- and 256-column tiles and the cap
SIZES = (2, 3, 15, 16, 17, 65, 255, 256, 257, 300, 531)


@pytest.mark.parametrize("n_p", SIZES)
@pytest.mark.parametrize("dtype", ["f16", "f32"])
def test_leaps_by_the_distances_miss_no_sample(n_p, dtype):
    import torch
    from paper_2204_02585_amd import binding
    rng = np.random.Generator(np.random.PCG64(n_p))
    tdt = torch.float16 if dtype == "f16" else torch.float32
    D = (1, 3, 8)[n_p % 3]
    poses = torch.from_numpy(scenes.spiral_poses(2)).cuda()
    handle = None
    try:
        for density in (0.0, 2e-4, 0.05):
            sig = [torch.from_numpy(p).cuda().to(tdt) for p in _planes(n_p, rng, density)]
            uvw = [torch.from_numpy(rng.uniform(-1, 1, (n_p, n_p, 3 * D)).astype(np.float32)).cuda().to(tdt)
                   for _ in range(3)]
            beta = torch.from_numpy(rng.uniform(-1, 1, (3, 5, D)).astype(np.float32)).cuda().to(tdt)
            caches = binding.Caches(sig, uvw, beta, scenes.BOX_MIN, scenes.BOX_MAX)
            want = _check(caches, poses, 96, f"n_p={n_p} {dtype} density={density}")
            # the same arrays through recreate, into a handle that held others
            if handle is None:
                handle = caches
                continue
            handle.recreate(sig, uvw, beta, scenes.BOX_MIN, scenes.BOX_MAX)
            got = _check(handle, poses, 96, f"recreate n_p={n_p} {dtype} density={density}")
            assert np.array_equal(want[0], got[0]) and np.array_equal(want[1], got[1])
            caches.close()
    finally:
        if handle is not None:
            handle.close()


@pytest.mark.parametrize("n_p", [2, 5, 16, 17, 64, 130, 257, 300])
@pytest.mark.parametrize("channels,dtype", [(1, "f32"), (12, "f16"), (64, "f32")])
def test_linear_leaps_miss_no_sample(n_p, channels, dtype):
    """(64 binary32 channels: one wave per workgroup folds them; small grids
    with D = 1 take a scratch allocation of their own.)"""
    import torch
    from paper_2204_02585_amd import binding
    rng = np.random.Generator(np.random.PCG64(1000 * channels + n_p))
    tdt = torch.float16 if dtype == "f16" else torch.float32
    D = (1, 4, 8)[n_p % 3]
    poses = torch.from_numpy(scenes.spiral_poses(2)).cuda()
    for density in (0.0, 3e-3):
        sig = [torch.from_numpy(p).cuda().to(tdt) for p in _planes(n_p, rng, density, channels)]
        uvw = [torch.from_numpy(rng.uniform(-1, 1, (n_p, n_p, 3 * D)).astype(np.float32)).cuda().to(tdt)
               for _ in range(3)]
        beta = torch.from_numpy(rng.uniform(-1, 1, (3, 5, D)).astype(np.float32)).cuda().to(tdt)
        # live only where all three planes are: about 0.6 per live channel
        dec = scenes.LinearDecoder(rng.uniform(2.0, 3.0, 3 * channels).astype(np.float32), -3.6 * channels,
                                   rng.uniform(-0.3, 0.3, (3, D, 3 * D)).astype(np.float32),
                                   rng.uniform(-0.1, 0.1, (3, D)).astype(np.float32))
        caches = binding.Caches(sig, uvw, beta, scenes.BOX_MIN, scenes.BOX_MAX, decoder=dec)
        try:
            _check(caches, poses, 96, f"linear n_p={n_p} channels={channels} {dtype} density={density}")
        finally:
            caches.close()


@pytest.mark.parametrize("shift", [1, 3, 4, 8])
def test_arrays_that_start_between_16_byte_pieces(shift):
    """Views into larger buffers, `shift` binary16 values past an aligned
    start, hold the same caches as aligned arrays."""
    import torch
    from paper_2204_02585_amd import binding
    rng = np.random.Generator(np.random.PCG64(shift))
    n_p, D = 36, 8
    sig = [torch.from_numpy(p).cuda().half() for p in _planes(n_p, rng, 0.02)]
    uvw = [torch.from_numpy(rng.uniform(-1, 1, (n_p, n_p, 3 * D)).astype(np.float16)).cuda() for _ in range(3)]
    beta = torch.from_numpy(rng.uniform(-1, 1, (3, 5, D)).astype(np.float16)).cuda()

    def moved(t):
        buf = torch.zeros(t.numel() + shift, dtype=t.dtype, device="cuda")
        buf[shift:] = t.reshape(-1)
        return buf[shift:].view(t.shape)

    poses = torch.from_numpy(scenes.single_pose()).cuda()
    out = []
    for f in (lambda t: t, moved):
        caches = binding.Caches([f(t) for t in sig], [f(t) for t in uvw], f(beta), scenes.BOX_MIN, scenes.BOX_MAX)
        try:
            out.append(_check(caches, poses, 64, f"shift={shift}"))
        finally:
            caches.close()
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])


def _against_oracle(sig, uvw, beta, decoder, label):
    """A small frame of these arrays (numpy, in their storage types) with the
    handle's records against the oracle's, every ray and statistic."""
    import torch
    from paper_2204_02585_amd import binding
    intr = dict(fx=30.0, fy=30.0, cx=12.0, cy=9.5, width=24, height=19)
    poses, n = scenes.spiral_poses(2), 96
    dev = lambda a: torch.from_numpy(a).cuda()  # noqa: E731
    caches = binding.Caches([dev(a) for a in sig], [dev(a) for a in uvw], dev(beta), scenes.BOX_MIN, scenes.BOX_MAX,
                            decoder=decoder)
    try:
        rgb, depth, st = caches.render_stats(dev(poses), intr, 2.0, 6.0, n)
        torch.cuda.synchronize()
    finally:
        caches.close()
    ref = oracle.render(sig, uvw, beta, poses, intr, 2.0, 6.0, n, scenes.BOX_MIN, scenes.BOX_MAX, decoder=decoder)
    assert int(ref["n_occ"].sum()) > 0, label
    gpu = (rgb.cpu().numpy().reshape(-1, 3), depth.cpu().numpy().reshape(-1),
           st.cpu().numpy().view(np.uint32).reshape(-1, 4))
    # binary32 values, sums in binary64
    pu.compare(gpu, ref, np.arange(ref.size), 1e-5, label)


def _arrays(n_p, rng, D, dtype, channels=0):
    ndt = np.float16 if dtype == "f16" else np.float32
    # the oracle takes finite values, as the entry point documents
    sig = [np.nan_to_num(p).astype(ndt) for p in _planes(n_p, rng, 0.05, channels)]
    uvw = [rng.uniform(-1, 1, (n_p, n_p, 3 * D)).astype(ndt) for _ in range(3)]
    return sig, uvw, rng.uniform(-1, 1, (3, 5, D)).astype(ndt)


# the copies' runs of 32 KiB: whole ones with a tail (67, 129, 257), a part of
# one (2, 17), none left over (256); records filled up and as they are
@pytest.mark.parametrize("n_p", [2, 17, 67, 129, 256, 257])
@pytest.mark.parametrize("dtype", ["f16", "f32"])
def test_records_and_copies(n_p, dtype):
    rng = np.random.Generator(np.random.PCG64(2000 + n_p))
    for D in (1, 3, 8, 16):
        _against_oracle(*_arrays(n_p, rng, D, dtype), None, f"records n_p={n_p} D={D} {dtype}")


@pytest.mark.parametrize("n_p", [2, 17, 64, 130, 257])
@pytest.mark.parametrize("channels,dtype", [(1, "f32"), (12, "f16"), (64, "f32"), (64, "f16")])
def test_folded_records(n_p, channels, dtype):
    rng = np.random.Generator(np.random.PCG64(3000 * channels + n_p))
    for D in (1, 8):
        dec = scenes.LinearDecoder(rng.uniform(2.0, 3.0, 3 * channels).astype(np.float32), -3.6 * channels,
                                   rng.uniform(-0.3, 0.3, (3, D, 3 * D)).astype(np.float32),
                                   rng.uniform(-0.1, 0.1, (3, D)).astype(np.float32))
        _against_oracle(*_arrays(n_p, rng, D, dtype, channels), dec, f"folded n_p={n_p} D={D} {channels} {dtype}")
