"""The fp32 kernel on the GPU at the edges of its tiles, against the fp64 oracle; every window of a
larger batch equals the same window decoded alone."""
import numpy as np
import pytest

from f32_shapes import IDS, OFF_IDS, OFF_SHAPES, SHAPES, case
from gpu_helpers import FP32_ATOL, FP32_RTOL, say, to_device
from paper_2601_09921_amd import pwdec

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("s,off", [(s, False) for s in SHAPES] + [(s, True) for s in OFF_SHAPES],
                         ids=IDS + [i + "_off" for i in OFF_IDS])
def test_matches_oracle(s, off):
    import torch
    wl, w, meas, types, o = case(s, off)
    reps = 67   # a ragged batch, the shape's windows repeated
    dec = pwdec.Decoder.from_workload(wl, w, max_windows=reps)
    idx = np.arange(reps) % wl.B
    mt, tt = to_device(meas[idx], types[idx])
    shape = (reps, wl.d) if s[10] else (reps,)
    logits = torch.full(shape, float("nan"), dtype=torch.float32, device="cuda")
    bits = torch.full(shape, 7, dtype=torch.uint8, device="cuda")
    (dec.decode_recurrent if s[10] else dec.decode)(mt, tt, logits, bits)
    assert dec.sync_status() == pwdec.PWD_OK
    g = logits.cpu().numpy()
    dec.close()
    err = np.abs(g[:wl.B] - o)
    say(f"  max |gpu - oracle| = {err.max():.2e}")
    assert (err <= FP32_RTOL * np.abs(o) + FP32_ATOL).all()
    assert np.array_equal(g, g[:wl.B][idx])
    assert np.array_equal(bits.cpu().numpy(), (g > 0).astype(np.uint8))
