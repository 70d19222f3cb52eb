"""The sweep form that pamc_info reports: its place in the structure, which
older callers know without it, and the kernel names made from it."""
import ctypes
import os
import subprocess
from types import SimpleNamespace

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_info_keeps_its_layout(tmp_path):
    from paper_2606_25203_amd.pamc import pamc_info
    fields = [f[0] for f in pamc_info._fields_]
    src = tmp_path / "layout.c"
    src.write_text('#include "pamc.h"\n#include <stdio.h>\nint main(void) { printf("%zu", sizeof(pamc_info));\n' +
                   "".join(f'printf(" %zu", offsetof(pamc_info, {f}));\n' for f in fields) + "return 0; }\n")
    subprocess.run(["gcc", "-I", os.path.join(ROOT, "include"), str(src), "-o", str(tmp_path / "layout")], check=True)
    out = [int(x) for x in subprocess.run([str(tmp_path / "layout")], capture_output=True, text=True).stdout.split()]
    assert out == [ctypes.sizeof(pamc_info)] + [getattr(pamc_info, f).offset for f in fields]
    # the sweep form lies in what was padding
    assert out[0] == 80 and pamc_info.pull.offset == 16 and pamc_info.nnz.offset == 24


def info(**kw):
    base = dict(dense=0, replicas=256, potts_K=0, bit_sweeps=0, bit_tiles=0, tile_sweeps=0, pull=1, X=100, coupling_mode=2,
                tiles_per_wave=4, hubs=0)
    return SimpleNamespace(**{**base, **kw})


@pytest.mark.parametrize("kw,sweeps,rule,name", [
    (dict(bit_sweeps=3, bit_tiles=4), 10, 0, "k_sweep_bits_grid<4, false>"),
    (dict(bit_sweeps=3, bit_tiles=4), 2, 0, "k_sweep_pull<2, 4, false, false>"),
    (dict(bit_sweeps=1, bit_tiles=-2), 1, 1, "k_sweep_bits_quad<2, true>"),
    (dict(bit_sweeps=7, bit_tiles=-1, tile_sweeps=1), 6, 0, "k_sweep_tile<2>"),
    (dict(bit_sweeps=7, bit_tiles=-1, tile_sweeps=1), 7, 0, "k_sweep_bits_quad<1, false>"),
    (dict(), 10, 0, "k_sweep_pull<2, 4, false, false>"),   # a torus kept from packing
    (dict(tile_sweeps=2), 5, 0, "k_sweep_tmma_g<8>"),
    (dict(pull=0), 5, 0, "k_sweep_push"),
    (dict(potts_K=3), 5, 0, "k_sweep_potts<3>"),
    (dict(dense=1, replicas=64), 1, 1, "k_dense_step<1, 64>"),
    (dict(dense=1, replicas=128), 1, 0, "k_dense_step<0, 128>"),
    (dict(dense=1, replicas=192), 1, 0, "k_dense_step<0, 256>"),
])
def test_names(kw, sweeps, rule, name):
    from paper_2606_25203_amd.profile_kernels import kernel_source, sweep_kernel
    assert sweep_kernel(info(**kw), sweeps, rule) == name
    src = open(os.path.join(ROOT, "paper_2606_25203_amd", "csrc", kernel_source(name))).read()
    assert name.split("<")[0] + "(" in src
