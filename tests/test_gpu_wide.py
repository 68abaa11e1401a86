"""Few windows run on kernels that split the work the other way (features over a workgroup's
wavefronts, an item's query blocks over workgroups): bit for bit the results of the large-batch
kernels. One batch beyond the sizes of every rule (more than 1024 token blocks; more than 512
windows for the state-resident network) against the same windows in batches on either side of
each line, odd sizes among them; its first and last window against the oracle."""
import numpy as np
import pytest

from gpu_helpers import BF16_ATOL, say, to_device
from oracle import decoder as O
from paper_2601_09921_amd import pwdec, synth

pytestmark = pytest.mark.gpu
BF16 = synth.DTYPE_BF16

# (d, W, D, L, H, mlp, grid, resnet, dilations, schedule), windows of the large batch, small batches
CASES = [
    ((11, 11, 256, 2, 8, 4, False, False, (), 0), 131, (1, 2, 31, 33, 65, 128)),    # 8 blocks a window
    ((9, 10, 256, 2, 4, 5, False, False, (), 0), 207, (1, 51, 52, 204)),            # 5 blocks, heads of 64
    ((25, 26, 256, 1, 8, 4, False, False, (), 0), 28, (1, 6, 7, 13, 26)),           # 39 blocks
    ((7, 8, 128, 2, 8, 5, True, True, (1, 2, 4), 0), 259, (1, 3, 64, 65, 256)),     # split around convolutions
    ((13, 13, 128, 1, 8, 4, False, True, (), 0), 95, (1, 23, 24, 93)),              # heads of 16, 11 blocks
    ((25, 25, 128, 1, 8, 5, True, False, (), 0), 25, (1, 3, 7, 23)),                # tile of a whole CU's LDS
    ((7, 8, 128, 2, 8, 4, False, False, (), pwdec.SCHEDULE_LAYERS), 345, (1, 85, 86, 341)),
    # on either side of the attention's line (168 and 176 items; 168 and 172)
    ((19, 19, 256, 1, 8, 4, False, False, (), 0), 45, (1, 21, 22, 32, 44)),         # 23 blocks, heads of 32
    ((17, 17, 256, 1, 4, 4, False, False, (), 0), 57, (1, 32, 42, 43, 56)),         # 18 blocks, heads of 64
    # d_model 256, 9 blocks a window: the embedder block and the parts around the convolutions
    ((11, 11, 256, 2, 8, 4, True, True, (1, 2, 4), 0), 115, (1, 2, 57, 113)),
    ((11, 11, 256, 1, 4, 5, True, True, (2, 1, 3), 0), 114, (1, 29, 113)),
    ((9, 9, 256, 2, 8, 4, False, True, (), 0), 205, (1, 51, 204)),                  # the embedder block alone
    ((9, 9, 256, 1, 8, 5, True, True, (), 0), 147, (1, 37, 146)),                   # 7 blocks a window
    ((5, 6, 128, 2, 8, 4, True, False, (1, 2, 1), 0), 342, (1, 85, 341)),           # 3 blocks a window
]


@pytest.mark.parametrize("net,n,parts", CASES, ids=[f"d{c[0][0]}_D{c[0][2]}_H{c[0][4]}_r{c[0][5]}_n{c[1]}" for c in CASES])
@pytest.mark.parametrize("recurrent", [False, True], ids=["decode", "recurrent"])
def test_small_batches_equal_large(net, n, parts, recurrent):
    import torch
    d, W, D, L, H, r, grid, res, dil, sched = net
    wl = synth.Workload("x", d, W, n, 0.05, 0.0, D, L, H, r, BF16, grid=grid, resnet=res, dil=dil)
    w = synth.make_weights(wl, seed=5)
    dec = pwdec.Decoder.from_workload(wl, w)
    dec.schedule(sched)
    meas, types = synth.make_windows(wl, seed=6, realistic_boundaries=False)
    mt, tt = to_device(meas, types)

    def run(lo, hi):
        shape = (hi - lo, d) if recurrent else (hi - lo,)
        logits = torch.full(shape, float("nan"), dtype=torch.float32, device="cuda")
        bits = torch.full(shape, 7, dtype=torch.uint8, device="cuda")
        (dec.decode_recurrent if recurrent else dec.decode)(mt[lo:hi].contiguous(), tt[lo:hi].contiguous(), logits, bits)
        assert dec.sync_status() == pwdec.PWD_OK
        return logits.cpu().numpy(), bits.cpu().numpy()

    full, fbits = run(0, n)
    ends = [0, n - 1]
    o = (O.forward_windows_recurrent if recurrent else O.forward_windows)(meas[ends], types[ends], w, d, H, grid=grid)[0]
    assert np.isfinite(full).all() and np.abs(full[ends] - o).max() <= BF16_ATOL
    for k in parts:
        for lo in {0, n - k}:
            say(f"  {k} windows from {lo}")
            g, b = run(lo, lo + k)
            assert np.array_equal(g, full[lo:lo + k]) and np.array_equal(b, fbits[lo:lo + k])
    dec.close()
