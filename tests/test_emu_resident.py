"""The two state-resident kernels on the host SIMT stand-in: the library as it is (few windows: one
workgroup per window) against a host build in which every batch takes the one-wavefront-per-window
kernel, bit for bit, over every number of token blocks, both head sizes and both token sets; no
access outside any allocation in either."""
import os
import sys

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, os.path.join(HERE, "emu"))

import build_emu  # noqa: E402
import run_emu  # noqa: E402
from oracle import decoder as O  # noqa: E402
from paper_2601_09921_amd import synth  # noqa: E402
from test_emu_host import BF16_ATOL, emu  # noqa: E402,F401


@pytest.fixture(scope="module")
def waves(emu):  # noqa: F811
    out = os.path.join(build_emu.OUT, "waves")
    lib = os.path.join(out, "libpwdec_emu.so")
    if not os.path.exists(lib) or os.path.getmtime(lib) < os.path.getmtime(build_emu.LIB):
        lib = build_emu.build(out=out, lift=[("SPLIT_MAX_WINDOWS = 512", "SPLIT_MAX_WINDOWS = 0")],
                              base=build_emu.OUT)
    return run_emu.load(lib)


@pytest.mark.parametrize("d,W,B,H,L,grid", [(3, 3, 5, 8, 2, False), (5, 5, 1, 4, 1, False), (5, 5, 1, 8, 2, True),
                                            (7, 7, 1, 8, 1, True)])
def test_split_equals_one_wavefront(emu, waves, d, W, B, H, L, grid):  # noqa: F811
    wl = synth.Workload(f"s{d}", d, W, B, 0.05, 0.0, 128, L, H, 4, synth.DTYPE_BF16, grid=grid)
    w = synth.make_weights(wl, seed=d + 3)
    meas, types = synth.make_windows(wl, seed=d + 4, realistic_boundaries=False)
    a, abits, arc = run_emu.decode(emu, wl, w, meas, types)
    b, bbits, brc = run_emu.decode(waves, wl, w, meas, types)
    o, _ = O.forward_windows(meas, types, w, d, H, grid=grid)
    assert arc == 0 and brc == 0 and emu.emu_errors() == 0 and waves.emu_errors() == 0
    assert np.array_equal(a.view(np.uint32), b.view(np.uint32)) and np.array_equal(abits, bbits)
    assert np.abs(a - o).max() <= BF16_ATOL
