"""The state-resident network at few windows runs with one workgroup per window: bit for bit the
results of the one-wavefront-per-window kernel, which takes more than 512. One to four token
blocks, heads of 16 and 32, one to four layers; batches on either side of a full pass over the
CUs and of the line between the kernels."""
import numpy as np
import pytest

from gpu_helpers import say, to_device
from paper_2601_09921_amd import pwdec, synth

pytestmark = pytest.mark.gpu

# (d, W, L, H, grid)
NETS = [(3, 3, 1, 4, False), (3, 6, 4, 8, False), (5, 5, 2, 8, False), (5, 10, 3, 4, True), (7, 14, 3, 8, False),
        (7, 7, 2, 4, False), (7, 8, 4, 8, True), (7, 7, 1, 4, True)]


@pytest.mark.parametrize("d,W,L,H,grid", NETS, ids=[f"d{c[0]}_L{c[2]}_H{c[3]}{'_grid' if c[4] else ''}" for c in NETS])
def test_split_equals_one_wavefront(d, W, L, H, grid):
    import torch
    n = 515
    wl = synth.Workload("x", d, W, n, 0.05, 0.0, 128, L, H, 4, synth.DTYPE_BF16, grid=grid)
    dec = pwdec.Decoder.from_workload(wl, synth.make_weights(wl, seed=5))
    dec.schedule(pwdec.SCHEDULE_RESIDENT)
    meas, types = synth.make_windows(wl, seed=6, realistic_boundaries=False)
    mt, tt = to_device(meas, types)

    def run(lo, hi):
        logits = torch.full((hi - lo,), float("nan"), dtype=torch.float32, device="cuda")
        bits = torch.full((hi - lo,), 7, dtype=torch.uint8, device="cuda")
        dec.decode(mt[lo:hi].contiguous(), tt[lo:hi].contiguous(), logits, bits)
        assert dec.sync_status() == pwdec.PWD_OK
        return logits.cpu().numpy(), bits.cpu().numpy()

    full, fbits = run(0, n)
    assert np.isfinite(full).all()
    for k in (1, 2, 255, 257, 512):
        for lo in (0, n - k):
            say(f"  {k} windows from {lo}")
            g, b = run(lo, lo + k)
            assert np.array_equal(g, full[lo:lo + k]) and np.array_equal(b, fbits[lo:lo + k])
    dec.close()
