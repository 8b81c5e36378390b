"""Locality blocks of the assembly (CPU): the mesh tables never cut more
blocks from a mesh than runs along the Morton curve give, since the tiles are
the pairs of blocks.  The driver calls mesh_prepare of the built library."""
import os
import subprocess

import numpy as np
import pytest

import synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2206_00708_amd")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
BT, SMAX = 16, 24

DRIVER = r"""
#include <cstdio>
#include "internal.h"
int main(int argc, char **argv)
{
    for (int a = 1; a < argc; ++a) {
        FILE *f = std::fopen(argv[a], "rb");
        bemtx::MeshData m;
        if (!f || std::fread(&m.nv, 8, 1, f) != 1 || std::fread(&m.nt, 8, 1, f) != 1) return 1;
        m.xyz_user.resize(3 * m.nv);
        m.tri_user.resize(3 * m.nt);
        if (std::fread(m.xyz_user.data(), 24, m.nv, f) != (size_t)m.nv) return 1;
        if (std::fread(m.tri_user.data(), 12, m.nt, f) != (size_t)m.nt) return 1;
        std::fclose(f);
        if (bemtx::mesh_prepare(m) != BEM_OK) return 2;
        std::printf("%d\n", m.nb);
    }
}
"""


def _meshes():
    x, t = synth.fibonacci_sphere(2002)
    az = np.arctan2(x[:, 1], x[:, 0])
    rng = np.random.default_rng(1)
    return [(x, t), (x * [1.0, 0.02, 0.02], t), (x * [1.0, 1.0, 0.002], t),
            (x * (1 + 0.6 * np.sin(9 * az) * (1 - x[:, 2] ** 2))[:, None], t),
            (x * np.abs(1 + 0.15 * rng.standard_normal(len(x)))[:, None], t), synth.icosphere(0), synth.icosphere(3)]


def _morton_blocks(xyz, tri):
    c = xyz[tri].mean(axis=1)
    lo = xyz.min(axis=0)
    q = np.clip((c - lo) / (xyz.max(axis=0) - lo).max() * 2097151.0, 0, 2097151).astype(np.uint64)
    code = np.zeros(len(tri), dtype=np.uint64)
    for b in range(21):
        for d in range(3):
            code |= ((q[:, d] >> np.uint64(b)) & np.uint64(1)) << np.uint64(3 * b + d)
    nb, count, seen = 0, BT, set()
    for t in np.argsort(code, kind="stable"):
        new = seen | set(tri[t])
        if count == BT or len(new) > SMAX:
            nb, count, new = nb + 1, 0, set(tri[t])
        seen, count = new, count + 1
    return nb


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not found")
def test_no_more_blocks_than_along_the_morton_curve(tmp_path):
    from paper_2206_00708_amd import build
    if not os.path.exists(build.LIB):
        build.build()
    src = tmp_path / "driver.cpp"
    src.write_text(DRIVER)
    exe = str(tmp_path / "driver")
    subprocess.check_call([HIPCC, "-O1", "-std=c++17", "--offload-arch=gfx950", "--offload-host-only", "-x", "hip",
                           "-I", os.path.join(PKG, "csrc"), "-c", str(src), "-o", exe + ".o"])
    subprocess.check_call([HIPCC, exe + ".o", build.LIB, "-Wl,-rpath," + PKG, "-o", exe])
    files = []
    meshes = _meshes()
    for i, (x, t) in enumerate(meshes):
        files.append(str(tmp_path / f"{i}.bin"))
        with open(files[-1], "wb") as f:
            f.write(np.array([len(x), len(t)], dtype=np.int64).tobytes())
            f.write(np.ascontiguousarray(x, dtype=np.float64).tobytes())
            f.write(np.ascontiguousarray(t, dtype=np.int32).tobytes())
    got = [int(v) for v in subprocess.check_output([exe, *files], text=True).split()]
    want = [_morton_blocks(x, t) for x, t in meshes]
    assert all(g <= w for g, w in zip(got, want)), (got, want)
