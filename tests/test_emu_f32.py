"""The fp32 kernel on the host SIMT stand-in, at the edges of its tiles, against the fp64 oracle."""
import os
import sys

import numpy as np
import pytest

from f32_shapes import IDS, OFF_IDS, OFF_SHAPES, SHAPES, case
from test_emu_host import emu  # noqa: F401

sys.path.insert(0, os.path.join(os.path.dirname(os.path.abspath(__file__)), "emu"))
import run_emu  # noqa: E402


@pytest.mark.parametrize("s", SHAPES, ids=IDS)
def test_matches_oracle(emu, s):  # noqa: F811
    wl, w, meas, types, o = case(s)
    logits, bits, rc = run_emu.decode(emu, wl, w, meas, types, recurrent=s[10])
    assert rc == 0 and emu.emu_errors() == 0
    # the fp32 workloads' tolerance: sums of up to 320 terms, 2^-24 each, over a dozen layers
    assert (np.abs(logits - o) <= 1e-4 * np.abs(o) + 1e-6).all(), np.abs(logits - o).max()


@pytest.mark.parametrize("s", OFF_SHAPES, ids=OFF_IDS)
def test_values_that_are_never_used_may_be_infinite(emu, s):  # noqa: F811
    wl, w, meas, types, o = case(s, off=True)
    logits, bits, rc = run_emu.decode(emu, wl, w, meas, types, recurrent=s[10])
    assert np.isfinite(o).all() and rc == 0 and emu.emu_errors() == 0
    assert (np.abs(logits - o) <= 1e-4 * np.abs(o) + 1e-6).all(), np.abs(logits - o).max()
