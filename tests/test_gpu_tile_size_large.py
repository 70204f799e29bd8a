"""A build with 16384-element tiles, whose exact sums need more than 64 bits:
byte-identical state to the 2048-element build, on the iterations of the
tile-size child and on values near the upper end of the exact sum's range
(2^19), where 64 bits would overflow in such a tile."""
import os
import subprocess
import sys

import numpy as np
import pytest

from paper_2008_05823_amd import build as B

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _large_values(out):
    """One process: scales, sign words and errors of values just below 2^19."""
    import torch
    from paper_2008_05823_amd import saef as S
    n, K, res = [40000, 16384, 16385], 2, {}
    off, d_pad = [0, 40000, 56384], 72832
    lay = S.Layout(off, n, d_pad, K)
    res["n_tiles"] = np.array(lay.info()["n_tiles"])
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)
    g = 524200.0 + 80.0 * torch.rand((K, d_pad), generator=gen, device="cuda")
    g[1] *= torch.where(torch.rand(d_pad, generator=gen, device="cuda") < 0.3, -1.0, 1.0)
    e = torch.zeros((K, d_pad), device="cuda")
    signs = torch.zeros((K, d_pad // 64), dtype=torch.int64, device="cuda")
    scales = torch.zeros((K, 3), device="cuda")
    S.saef_compress(lay, K, 1.0, g, e, signs, scales)
    assert S.saef_status(lay) == S.OK
    for k in range(K):      # the exact mean, rounded to fp32
        for l in range(3):
            v = g[k, off[l]:off[l] + n[l]].double().abs().cpu().numpy()
            assert scales[k, l].item() == np.float32(v.sum() / n[l])
    res.update(scales=scales.cpu().numpy(), signs=signs.cpu().numpy(), e=e.cpu().numpy())
    np.savez(out, **res)


def _run(lib, module, out):
    print(f"[tile-size] {os.path.basename(lib)} {module}", flush=True)
    subprocess.run([sys.executable, "-m", module, str(out)], cwd=ROOT, check=True, timeout=300,
                   env=dict(os.environ, SAEF_LIBRARY=lib))
    return np.load(out)


@pytest.mark.timeout(700)
@pytest.mark.parametrize("module", ["tests.tile_size_child", "tests.test_gpu_tile_size_large"])
def test_large_tiles_do_not_change_any_byte(tmp_path, module):
    lib = B.tile_variant_lib(B.TILE_VARIANT_LARGE)
    assert os.path.exists(lib), f"{lib} is missing: run __graft_entry__.build()"
    ra, rb = _run(B.LIB, module, tmp_path / "a.npz"), _run(lib, module, tmp_path / "b.npz")
    assert sorted(ra.files) == sorted(rb.files) and len(ra.files) > 1
    for k in ra.files:
        if k.endswith("n_tiles"):
            assert int(ra[k]) > int(rb[k]), k
        else:
            assert np.array_equal(ra[k].view(np.uint8), rb[k].view(np.uint8)), k


if __name__ == "__main__":
    _large_values(sys.argv[1])
