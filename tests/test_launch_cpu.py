"""Choices of the library's host code, on the CPU (tests/fake_hip.py): which
kernel a render launches, what tuning keeps, whether every accepted size is a
legal launch, and what a create does when memory is short."""
import pytest

from tests import fake_hip

# 800 x 800 x 256 of a 512 cache, ms per launch in each shape
COSTS = """
for part, ms in ((b"render_kernel_hybrid", 0.145), (b"ELi1ELb1ELb0", 0.149), (b"ELi2ELb1ELb0", 0.122),
                 (b"ELi4ELb1ELb0", 0.135), (b"ELi8ELb1ELb0", 0.174)):
    fake.fake_cost(part, ms)
"""


def test_tuning_keeps_the_automatic_two_lanes_where_they_are_fastest():
    """The shape that a render takes without tuning is among the candidates, so
    tuning never leaves a handle in a slower one."""
    got = fake_hip.run("""
d = desc(512, 8, sigma="f32")
a = arrays(d)
h = ctypes.c_void_p()
assert lib.sqn_create_caches(ctypes.byref(d), a[0], a[1], a[2], None, ctypes.byref(h)) == 0
out = []
for w, n in ((800, 1), (400, 3), (200, 1), (1600, 1)):
    it = intrinsics(w, w)
    poses, rgb, depth = alloc(48 * n), alloc(12 * w * w * n), alloc(4 * w * w * n)
    fake.fake_reset()
""" + COSTS.replace("\n", "\n    ") + """
    lanes, centre = ctypes.c_int32(-7), ctypes.c_float(-7)
    assert lib.sqn_tune_lanes_per_ray(h, poses, n, ctypes.byref(it), 2.0, 6.0, 256, rgb, depth, None,
                                      ctypes.byref(lanes), ctypes.byref(centre)) == 0
    launches()
    assert lib.sqn_render(h, poses, n, ctypes.byref(it), 2.0, 6.0, 256, rgb, depth, None) == 0
    out.append([lanes.value, centre.value, launches()])
print(json.dumps(out))
""")
    # one view and three views between 2^18 and 2^20 rays: two lanes, by the
    # automatic choice; outside, where it is eight or one lanes, what is
    # fastest of the lane counts that can be set
    for lanes, centre, log in got[:2]:
        assert (lanes, centre) == (0, 0.0) and len(log) == 1 and "ELi2ELb1ELb0" in log[0], got
    for lanes, centre, log in got[2:]:
        assert (lanes, centre) == (4, 0.0) and "ELi4ELb1ELb0" in log[0], got


# D, uvw, NDC, views, width, height, leaps -> lanes
LANES = [
    (8, "f16", 0, 1, 512, 511, 1, 8), (8, "f16", 0, 1, 512, 512, 1, 2), (8, "f32", 0, 1, 1024, 1023, 1, 2),
    (8, "f16", 0, 1, 1024, 1024, 1, 1), (16, "f32", 0, 1, 512, 512, 1, 2), (12, "f16", 0, 1, 512, 512, 1, 2),
    # no leaps, and D without a kernel of its own
    (8, "f16", 0, 1, 800, 800, 0, 4), (24, "f16", 0, 1, 800, 800, 1, 4), (17, "f32", 1, 1, 512, 512, 1, 4),
    (32, "f32", 0, 1, 512, 511, 1, 8), (24, "f16", 0, 1, 1024, 1024, 1, 1),
    # two lanes from 3 * 2^17 rays
    (8, "f16", 0, 2, 512, 383, 1, 4), (8, "f16", 0, 2, 512, 384, 1, 2), (8, "f32", 0, 3, 300, 300, 1, 4),
    (8, "f16", 1, 1, 768, 511, 1, 4), (8, "f16", 1, 1, 768, 512, 1, 2), (8, "f16", 1, 2, 512, 383, 1, 4),
    (16, "f32", 1, 1, 768, 511, 1, 4), (16, "f32", 1, 1, 768, 512, 1, 2),
    # the same kinds in the other type or D, from 2^18
    (8, "f32", 1, 1, 512, 512, 1, 2), (8, "f32", 1, 2, 512, 383, 1, 2), (16, "f16", 1, 1, 512, 512, 1, 2),
    (16, "f16", 0, 2, 512, 383, 1, 2), (16, "f32", 0, 2, 512, 383, 1, 2),
]


def test_automatic_lanes():
    """Lanes per ray by rays, views, D, uvw type and ray space: the name of the
    launched kernel carries them."""
    got = fake_hip.run(r"""
import re
out = []
for D, uvw, ndc, views, w, height, skip in DATA:
    d = desc(64, D, uvw=uvw)
    a = arrays(d)
    h = ctypes.c_void_p()
    assert lib.sqn_create_caches(ctypes.byref(d), a[0], a[1], a[2], None, ctypes.byref(h)) == 0
    assert lib.sqn_set_ndc(h, 1.0 if ndc else 0.0) == 0 and lib.sqn_set_empty_space_skipping(h, skip) == 0
    it = intrinsics(w, height)
    poses, rgb, depth = alloc(48 * views), alloc(12 * w * height * views), alloc(4 * w * height * views)
    fake.fake_reset()
    assert lib.sqn_render(h, poses, views, ctypes.byref(it), 0.5, 1.0, 64, rgb, depth, None) == 0
    log = launches()
    assert len(log) == 1, log
    out.append(int(re.search(r"render_kernelI\w+?Li\d+ELb0ELi(\d+)E", log[0]).group(1)))
    lib.sqn_destroy(h)
    for p in (poses, rgb, depth):
        fake.hipFree(p)
    free(a)
print(json.dumps(out))
""", data=[c[:7] for c in LANES])
    assert [(c, lanes) for c, lanes in zip(LANES, got) if lanes != c[7]] == []


def test_stored_components():
    """Which records are filled up: the handle's bytes and the kernel's D."""
    cases = [("f16", 1, 0, 0), ("f32", 1, 0, 0), ("f16", 2, 0, 8), ("f32", 2, 0, 0), ("f16", 3, 0, 8), ("f32", 3, 0, 8),
             ("f16", 8, 0, 8), ("f16", 9, 0, 16), ("f32", 16, 0, 16), ("f16", 17, 0, 0), ("f16", 1, 1, 8),
             ("f32", 2, 1, 8), ("f32", 12, 1, 16), ("f16", 31, 1, 0)]
    got = fake_hip.run(r"""
import re
import numpy as np
out = []
for uvw, D, linear, _ in DATA:
    d = desc(64, D, uvw=uvw)
    a = arrays(d)
    h = ctypes.c_void_p()
    if linear:
        w = [np.zeros(n, np.float32) for n in (3, 9 * D * D, 3 * D)]
        dec = B.LinearDecoder(1, 0.5, *[x.ctypes.data for x in w])
        s = lib.sqn_create_linear_caches(ctypes.byref(d), ctypes.byref(dec), a[0], a[1], a[2], None, ctypes.byref(h))
    else:
        s = lib.sqn_create_caches(ctypes.byref(d), a[0], a[1], a[2], None, ctypes.byref(h))
    assert s == 0, B.last_error()
    it = intrinsics(64, 64)
    poses, rgb, depth = alloc(48), alloc(12 * 4096), alloc(4 * 4096)
    fake.fake_reset()
    assert lib.sqn_render(h, poses, 1, ctypes.byref(it), 0.5, 1.0, 64, rgb, depth, None) == 0
    out.append([int(re.search(r"render_kernelI\w+?Li(\d+)ELb0E", launches()[0]).group(1)), lib.sqn_cache_device_bytes(h)])
    lib.sqn_destroy(h)
    for p in (poses, rgb, depth):
        fake.hipFree(p)
    free(a)
print(json.dumps(out))
""", data=cases)
    for (uvw, D, linear, kernel), (launched, nbytes) in zip(cases, got):
        assert launched == kernel, (uvw, D, linear, launched)
        if not linear:
            # 64 x 64 texels in three planes (4-byte sigma records), 256
            # directions in binary16; every part a multiple of 256 bytes
            stored = kernel or D
            assert nbytes == 3 * 4096 * (4 + 3 * stored * (2 if uvw == "f16" else 4)) + 256 * stored * 2, (uvw, D)


@pytest.mark.parametrize("linear", [0, 1])
def test_create_without_memory_for_filled_records(linear):
    """Too little memory for records of D = 4 filled up to 8, enough for them as
    they are: the create succeeds with the narrow ones; with less it reports
    it and keeps nothing."""
    got = fake_hip.run(r"""
import re
import numpy as np
D, n_p = 4, 64
d = desc(n_p, D)
a = arrays(d)
rng = np.random.Generator(np.random.PCG64(1))
w = [rng.uniform(-1, 1, n).astype(np.float32) for n in (3, 9 * D * D, 3 * D)]
dec = B.LinearDecoder(1, 0.5, *[x.ctypes.data for x in w])
def create():
    h = ctypes.c_void_p()
    if DATA:
        s = lib.sqn_create_linear_caches(ctypes.byref(d), ctypes.byref(dec), a[0], a[1], a[2], None, ctypes.byref(h))
    else:
        s = lib.sqn_create_caches(ctypes.byref(d), a[0], a[1], a[2], None, ctypes.byref(h))
    return s, h
before = fake.fake_used()
s, h = create()
assert s == 0
filled = lib.sqn_cache_device_bytes(h)
lib.sqn_destroy(h)
assert fake.fake_used() == before
out = dict(filled=filled, tries=[])
it = intrinsics(64, 64)
poses, rgb, depth = alloc(48), alloc(12 * 4096), alloc(4 * 4096)
before = fake.fake_used()
for room in (filled + (1 << 20), filled - 1, 3 * n_p * n_p * 4):
    fake.fake_limit(before + room)
    s, h = create()
    kernel, same = None, None
    if s == 0:
        if DATA:
            # the maps as the kernels read them, at the stored width
            buf = (ctypes.c_ubyte * (1 << 20))()
            n = fake.fake_copied(buf)
            DS = 8 if lib.sqn_cache_device_bytes(h) == filled else 4
            want = np.zeros((9 * DS + 3, DS), np.float32)
            want[:9 * DS].reshape(3, 3, DS, DS)[:, :, :D, :D] = w[1].reshape(3, D, 3, D).transpose(0, 2, 3, 1)
            want[9 * DS:, :D] = w[2].reshape(3, D)
            same = n == want.nbytes and bytes(buf[:n]) == want.tobytes()
        fake.fake_reset()
        assert lib.sqn_render(h, poses, 1, ctypes.byref(it), 0.5, 1.0, 64, rgb, depth, None) == 0
        kernel = int(re.search(r"render_kernelI\w+?Li(\d+)ELb0E", launches()[0]).group(1))
        bytes_ = lib.sqn_cache_device_bytes(h)
        lib.sqn_destroy(h)
    else:
        assert not h.value
        bytes_ = 0
    out["tries"].append([s, kernel, bytes_, same, fake.fake_used() - before])
print(json.dumps(out))
""", data=linear)
    first, short, none = got["tries"]
    assert first[:3] == [0, 8, got["filled"]] and first[4] == 0
    narrow = got["filled"] - 3 * 64 * 64 * 12 * 2 - 256 * 4 * 2
    if linear:
        narrow = short[2]       # its maps are smaller too
        assert 0 < narrow < got["filled"] - 3 * 64 * 64 * 12 * 2
        assert first[3] and short[3]
    assert short[:3] == [0, 0, narrow] and short[4] == 0
    assert none[0] == 2 and none[4] == 0       # SQN_ERR_OUT_OF_MEMORY


def test_recreate_scratch_lies_in_the_block():
    """The preparation's row distances and their minima end inside the handle's
    block, behind its sigma records, for every small grid and the largest,
    with the narrowest records there are."""
    got = fake_hip.run(r"""
import re
out = []
for n_p in list(range(2, 130)) + [255, 256, 257, 1023, 1025, 2047, 2048]:
    for D, uvw in ((1, "f16"), (1, "f32"), (2, "f32"), (3, "f16")):
        d = desc(n_p, D, n_theta=2, n_phi=2, uvw=uvw)
        a = arrays(d)
        h = ctypes.c_void_p()
        assert lib.sqn_create_caches(ctypes.byref(d), a[0], a[1], a[2], None, ctypes.byref(h)) == 0
        fake.fake_reset()
        assert lib.sqn_recreate_caches(h, ctypes.byref(d), a[0], a[1], a[2], None) == 0
        f, f_min, n, pitch = [int(x) for x in [l for l in launches() if l.startswith("scratch")][0].split()[1:]]
        base, size = ctypes.c_void_p(), ctypes.c_size_t()
        fake.hipMemGetAddressRange(ctypes.byref(base), ctypes.byref(size), ctypes.c_void_p(f))
        sigma = 3 * -(-(4 * n_p * (-(-n_p // 4) * 4)) // 256) * 256      # 4-byte records, rows padded to four
        rows = -(-n_p // 16)
        ok = (n == n_p and size.value == lib.sqn_cache_device_bytes(h) and base.value + sigma <= f
              and f + 3 * rows * 16 * pitch <= f_min and f_min + 3 * rows * pitch <= base.value + size.value)
        if not ok:
            out.append([n_p, D, uvw, f - base.value, f_min - base.value, pitch, size.value])
        lib.sqn_destroy(h)
        free(a)
print(json.dumps(out))
""")
    assert got == []


def test_every_direction_grid_is_a_legal_launch():
    """Generation and creation over the direction grids that validation accepts,
    up to 2^31 nodes of D = 1: the launches stay within 2^32 work items per
    dimension (the stand-in for the runtime refuses others), and all nodes are
    covered."""
    grids = [(2, 2), (192, 256), (193, 256), (4096, 4096), (16384, 16383), (16384, 16384), (20000, 20000),
             (65536, 32767), (44431, 48333)]
    got = fake_hip.run(r"""
import numpy as np
def mlp(sizes):
    m = B.MLPDesc()
    m.n_hidden, m.width, m.n_in, m.n_out = len(sizes) - 2, sizes[1], sizes[0], sizes[-1]
    ws = [np.zeros((o, i), np.uint16) for i, o in zip(sizes[:-1], sizes[1:])]
    bs = [np.zeros(o, np.float32) for o in sizes[1:]]
    w = (ctypes.c_void_p * len(ws))(*[x.ctypes.data for x in ws])
    b = (ctypes.c_void_p * len(bs))(*[x.ctypes.data for x in bs])
    m.weights, m.biases = ctypes.cast(w, type(m.weights)), ctypes.cast(b, type(m.biases))
    return m, (ws, bs, w, b)
out = []
D = 1
pos, keep = zip(*[mlp([2 * (1 + 2 * 10), 256, 2 + 6 * D]) for _ in range(3)])
dirn, keep_d = mlp([3 * (1 + 2 * 4), 128, D])
nets = ctypes.c_void_p()
assert lib.sqn_create_networks((B.MLPDesc * 3)(*pos), ctypes.byref(dirn), D, 10, 4, None, ctypes.byref(nets)) == 0
for nt, nph in DATA:
    for n_p in (8, 128):
        d = desc(n_p, D, n_theta=nt, n_phi=nph)
        a = arrays(d)
        fake.fake_reset()
        s = lib.sqn_generate_caches(nets, ctypes.byref(d), a[0], a[1], a[2], None)
        log = [l.split() for l in launches()]
        own = [l for l in log if "direction_kernel" in l[0]]
        nodes = sum(int(l[1]) * int(l[2]) * 128 for l in own)
        h = ctypes.c_void_p()
        c = lib.sqn_create_caches(ctypes.byref(d), a[0], a[1], a[2], None, ctypes.byref(h))
        lib.sqn_destroy(h)
        out.append([nt, nph, n_p, s, c, len(own), nodes])
        free(a)
print(json.dumps(out))
""", data=grids)
    for nt, nph, n_p, s, c, own, nodes in got:
        assert s == 0 and c == 0, (nt, nph, n_p, s, c)
        assert own == (1 if nt * nph > 49152 else 0), (nt, nph, n_p, own)
        assert own == 0 or nodes >= nt * nph
