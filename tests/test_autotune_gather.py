"""Tuned configurations and the direct gathers of small stacks: a cached
configuration is used for its shape, by cpi_refocus and cpi_refocus_noalloc,
although an untuned stack of that size is gathered; a later '#default' line
takes it back; the autotuner times the gathers and what it leaves is what
cpi_refocus then launches."""
import os
import subprocess
import sys

import pytest

from tests.test_abi_host import _tiles_with_cache

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_default_line_takes_back(tmp_path):
    key = "wa32_ha32_wb16_hb16_ow32_oh32_na5@dev?"
    default = _tiles_with_cache(tmp_path, [])
    tuned = f"{key} 8 8 2 1 3 123.0"
    assert _tiles_with_cache(tmp_path, [tuned, f"#default {key}"]) == default
    assert _tiles_with_cache(tmp_path, [tuned, "#default other", "# note"]) == (8, 8, 2, 1, 3)
    assert _tiles_with_cache(tmp_path, [tuned, f"#default {key}", tuned]) == (8, 8, 2, 1, 3)


_CHILD = """
import sys
sys.path.insert(0, {root!r})
import numpy as np, torch
import paper_2407_20692_amd as cpi
from tests.test_gpu_refocus_window_edges import _launched
geo = cpi.geometry_default(32, 32, 16, 16)
gen = torch.Generator(device="cuda")
gen.manual_seed(3)
gam = torch.randn(1024 * 256, generator=gen, device="cuda")
out = [torch.empty(5 * 1024, device="cuda") for _ in range(3)]
al = np.linspace(0.5, 1.5, 5)
names = _launched(lambda: cpi.refocus(gam, geo, al, out[0]))
assert ("k_ref_gather" in names) == (not {tiles!r}), names
cpi.refocus_noalloc(gam, geo, al, out[1])
if {tiles!r}:
    assert cpi.refocus_tiles(geo, 5) == {tiles!r}
    cpi.refocus_tiled(gam, geo, al, out[2], {tiles!r})
    assert torch.equal(out[0], out[2]) and "k_ref_sep" in names
assert torch.equal(out[0], out[1])
# tuning again: the gathers are among what is timed, and are not slower here
cpi.autotune_refocus(gam, geo, al, out[1])
names = _launched(lambda: cpi.refocus(gam, geo, al, out[0]))
assert torch.equal(out[0], out[1])
assert ("k_ref_gather" in names) == (cpi.refocus_tiles(geo, 5) == {default!r}), names
print("child ok", "k_ref_gather" in names and "k_ref_gather")
"""


@pytest.mark.gpu
def test_cached_configuration_over_gathers(tmp_path):
    import torch

    import paper_2407_20692_amd as cpi
    p = torch.cuda.get_device_properties(0)
    tag = p.gcnArchName.replace(":", "_").replace(" ", "_") + f"/cu{p.multi_processor_count}"
    key = f"wa32_ha32_wb16_hb16_ow32_oh32_na5@{tag}"
    default = tuple(cpi.refocus_tiles(cpi.geometry_default(32, 32, 16, 16), 5))
    for tiles in ((8, 8, 2, 1, 3), ()):
        cache = tmp_path / "cache.txt"
        cache.write_text(key + " " + " ".join(map(str, tiles)) + " 9.0\n" if tiles else "")
        env = dict(os.environ, CPI_AUTOTUNE_CACHE=str(cache))
        r = subprocess.run([sys.executable, "-c",
                            _CHILD.format(root=ROOT, tiles=tiles, default=default)],
                           env=env, capture_output=True, text=True, timeout=110)
        assert r.returncode == 0 and "child ok" in r.stdout, r.stdout + r.stderr
        # a fresh process reads what the tuning left
        lines = cache.read_text().splitlines()
        if "k_ref_gather" in r.stdout and tiles:
            assert lines[-1] == f"#default {key}", lines
