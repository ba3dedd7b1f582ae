"""Objective partials of a solve: as many as the prox's final pass has blocks,
for every size, depth, inner solver, dual storage, share of a batch and plane group (host code of the library, no GPU)."""
import itertools
import os
import subprocess

import pytest

from paper_1904_04884_amd import build_lib, rihvr

HERE = os.path.dirname(os.path.abspath(__file__))
TV2D, FGP, BF16, ROWS, LOW = 1, 2, 4, 8, 16


@pytest.fixture(scope="module")
def grids(tmp_path_factory):
    if not rihvr.LIB_PATH.exists():
        pytest.fail("librihvr.so is not built (run __graft_entry__.build())")
    exe = tmp_path_factory.mktemp("grids") / "prox_grids"
    lib = rihvr.LIB_PATH
    obj = str(exe) + ".o"
    hipcc = build_lib.hipcc()
    subprocess.run([hipcc, "-x", "hip", "--cuda-host-only", "-std=c++17", f"--offload-arch={build_lib.ARCH}",
                    "-I", str(build_lib.CSRC), "-c", os.path.join(HERE, "host_prox_grids.cpp"), "-o", obj], check=True)
    subprocess.run([hipcc, obj, str(lib), f"-Wl,-rpath,{lib.parent}", "-o", str(exe)], check=True)

    def run(rows, steps=7):
        text = "\n".join(" ".join(map(str, r)) for r in rows)
        out = subprocess.run([str(exe), str(steps)], input=text, capture_output=True, text=True, check=True).stdout
        return [tuple(map(int, line.split())) for line in out.splitlines()]
    return run


def test_partials_counted_are_those_written(grids):
    xy = [(16, 16), (32, 48), (48, 32), (64, 64), (128, 128), (512, 64), (96, 512), (512, 512), (768, 384), (1024, 1024)]
    kinds = [f | t for t in (0, TV2D) for f in (LOW, FGP | LOW, FGP | BF16, BF16, ROWS | LOW, LOW ^ LOW)]
    rows = [(nx, ny, nz, lv, tb, fill, fl, 0)
            for (nx, ny), nz, lv, (tb, fill), fl in itertools.product(
                xy, (1, 4, 8, 17, 32, 128), (2, 3, 4), ((1536, 256), (64, 256), (6144, 85), (1536, 1)), kinds)]
    rows += [(nx, ny, nz, lv, 1536, 256, TV2D | f, g)
             for (nx, ny), (nz, g), lv, f in itertools.product(xy, ((17, 4), (32, 1), (8, 7)), (2, 3, 4), (LOW, BF16))]
    out = grids(rows)
    assert len(out) == len(rows)
    for row, (counted, written, bound, _) in zip(rows, out):
        assert counted == written <= bound, row


@pytest.mark.parametrize("steps", (0, 1, 2, 3, 4, 5, 8))
def test_partials_of_short_proxes(grids, steps):
    """Proxes of one pass, and of a last pass with few steps, which choose cut, depth and form
    by rules of their own."""
    xy = [(16, 16), (48, 32), (64, 64), (128, 128), (512, 64), (512, 512), (768, 384), (768, 768), (1024, 384),
          (1024, 1024), (2048, 512), (2048, 2048)]
    kinds = [f | t for t in (0, TV2D) for f in (LOW, FGP | LOW, BF16 | LOW, ROWS | LOW, 0)]
    rows = [(nx, ny, nz, lv, tb, fill, fl, 0)
            for (nx, ny), nz, lv, (tb, fill), fl in itertools.product(
                xy, (1, 2, 8, 15, 16, 17, 24, 31, 64, 100, 256), (2, 3, 4),
                ((1536, 256), (64, 256), (65536, 256), (1536, 85), (1536, 1)), kinds)]
    rows += [(nx, ny, nz, lv, 1536, 256, TV2D | f, g)
             for (nx, ny), (nz, g), lv, f in itertools.product(xy, ((17, 4), (32, 1), (100, 33)), (2, 3, 4), (LOW, BF16))]
    for row, (counted, written, bound, _) in zip(rows, grids(rows, steps)):
        assert counted == written <= bound, row


# volume, depth and three tv_blocks whose dual passes are cut into different chunks, one of
# them ragged (tests/test_gpu_tv_forms.py compares their results)
CHUNKINGS = [((512, 512, 200), 2, (64, 512, 1536)), ((768, 768, 120), 3, (64, 512, 65536)),
             ((512, 512, 200), 4, (64, 512, 1536))]


@pytest.mark.parametrize("dims", (0, TV2D))
def test_chunkings_differ(grids, dims):
    cuts = [grids([(*shape, lv, b, 256, dims | LOW, 0) for b in blocks]) for shape, lv, blocks in CHUNKINGS]
    for (shape, _, _), out in zip(CHUNKINGS, cuts):
        chunks = {o[3] for o in out}
        assert len(chunks) == 3 and max(chunks) > min(chunks) >= 16, chunks
    assert any(shape[2] % o[3] for (shape, _, _), out in zip(CHUNKINGS, cuts) for o in out)
