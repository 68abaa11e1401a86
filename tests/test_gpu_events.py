"""The detection-event kernel at every remainder of its four words per thread, odd batches, and
buffers that start one word past a 16-byte boundary, against the oracle bit for bit."""
import numpy as np
import pytest

from gpu_helpers import say, to_device
from oracle import decoder as O
from paper_2601_09921_amd import pwdec, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,W,B", [(3, 3, 1), (3, 6, 333), (5, 13, 777), (7, 7, 259), (9, 9, 101), (13, 15, 67), (25, 50, 65)])
@pytest.mark.parametrize("offset", [0, 1])
def test_events_exact(d, W, B, offset):
    import torch
    say(f"events d={d} W={W} B={B} offset={offset}")
    D, H, dtype = (32, 2, synth.DTYPE_F32) if d <= 5 else (128, 8, synth.DTYPE_BF16)
    wl = synth.Workload("e", d, W, B, 0.05, 0.0, D, 1, H, 4, dtype)
    dec = pwdec.Decoder.from_workload(wl, synth.make_weights(wl, seed=1))
    meas, types = synth.make_windows(wl, seed=d + W, realistic_boundaries=False)
    mt, tt = to_device(meas, types)
    src = torch.empty(mt.numel() + offset, dtype=torch.int32, device="cuda")[offset:].view(mt.shape)
    src.copy_(mt)
    words = mt.shape[-1]
    ev = torch.full((B * W * words + offset,), -1, dtype=torch.int32, device="cuda")[offset:].view(B, W, words)
    dec.detection_events(src, tt, ev)
    assert dec.sync_status() == pwdec.PWD_OK
    expect = O.pack_bits(O.detection_events(meas, types, d)).view(np.int32).reshape(B, W, words)
    assert np.array_equal(ev.cpu().numpy(), expect)
    dec.close()
