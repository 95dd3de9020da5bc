"""Accuracy of the binary32 opacity 1 - exp(-q) the render kernels weigh a
sample with (csrc/opacity.h), built for the host with hipcc and compared with
binary64."""
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2204_02585_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

PROGRAM = r"""
#include <stdio.h>
#include "opacity.h"
int main(int argc, char** argv)
{
    FILE* in = fopen(argv[1], "rb");
    FILE* out = fopen(argv[2], "wb");
    float q;
    while (fread(&q, sizeof(float), 1, in) == 1) {
        const float r = sqn::opacity(q);
        fwrite(&r, sizeof(float), 1, out);
    }
    fclose(in);
    fclose(out);
    return 0;
}
"""


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc missing")
def test_opacity_accuracy(tmp_path):
    src = tmp_path / "opacity_check.hip"
    src.write_text(PROGRAM)
    exe = tmp_path / "opacity_check"
    subprocess.run([HIPCC, "--offload-arch=gfx950", "-O2", "-ffp-contract=off", "-I", CSRC, "-o", str(exe),
                    str(src)], check=True, capture_output=True)
    rng = np.random.Generator(np.random.PCG64(3))
    ln2 = np.log(2.0)
    # all magnitudes, the reduction's boundaries (k + 1/2) ln 2, its centres
    q = np.concatenate([10.0 ** rng.uniform(-9, 2.1, 400_000), rng.uniform(0.0, 4.0, 400_000),
                        ((np.arange(48)[:, None] + 0.5) * ln2 * (1.0 + rng.uniform(-1e-5, 1e-5, 400))).ravel(),
                        ((np.arange(1, 48)[:, None]) * ln2 * (1.0 + rng.uniform(-1e-5, 1e-5, 400))).ravel()])
    special = np.array([0.0, 2.0 ** -149, 2.0 ** -126, 63.9, 64.0, 65.0, 3e38, np.inf, np.nan])
    q = np.concatenate([q, special]).astype(np.float32)
    (tmp_path / "in.bin").write_bytes(q.tobytes())
    subprocess.run([str(exe), str(tmp_path / "in.bin"), str(tmp_path / "out.bin")], check=True)
    got = np.fromfile(tmp_path / "out.bin", dtype=np.float32)
    assert got.size == q.size
    n = q.size - special.size
    ref = -np.expm1(-q[:n].astype(np.float64))
    ulp = np.exp2(np.floor(np.log2(ref)) - 23.0)
    err = np.abs(got[:n].astype(np.float64) - ref) / ulp
    # half a unit for the last rounding, and what the two roundings of r and
    # the one of e, 2^-24 of r each, leave where 2^n e is largest
    # against the result
    assert err.max() < 0.9, f"{err.max():.3f} units at q = {q[np.argmax(err)]!r}"
    assert np.sqrt(np.mean(err ** 2)) < 0.32
    tail = got[n:]
    np.testing.assert_array_equal(tail[:3], special[:3].astype(np.float32))
    assert np.all(tail[3:8] == 1.0)
    assert np.isnan(tail[8])
