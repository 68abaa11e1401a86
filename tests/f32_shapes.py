"""fp32 configurations at the edges of the fp32 kernel's tiles: per d_model 64 / 32 / 16 a matrix-core
step takes 4 / 8 / 16 tokens, so 8, 16, 24, 36, 48 and 64 tokens are whole or ragged tiles of
different counts; heads of 4 to 64; feed-forward 4x and 5x (whose fifth column group is shared
out); dilated convolutions and the embedder block; recurrent readouts."""

# (d, W, B, D, L, H, mlp, grid, resnet, dilations, recurrent)
SHAPES = [
    (3, 4, 3, 64, 2, 4, 4, False, False, (), False),
    (3, 4, 2, 64, 1, 1, 5, True, False, (), False),
    (5, 6, 2, 64, 1, 1, 4, False, False, (), False),
    (3, 3, 1, 64, 1, 16, 4, True, False, (1, 2, 1), True),
    (3, 5, 3, 32, 2, 8, 4, False, False, (), True),
    (3, 3, 3, 32, 1, 2, 5, True, True, (), False),
    (5, 7, 2, 32, 2, 4, 4, False, False, (), False),
    (5, 5, 2, 32, 1, 2, 4, True, False, (1, 2, 3), False),
    (5, 5, 1, 32, 1, 4, 5, False, False, (), False),
    (3, 4, 2, 16, 2, 4, 4, False, False, (), False),
    (3, 4, 2, 16, 1, 2, 5, True, False, (1, 1, 2), True),
    (5, 5, 2, 16, 1, 4, 4, False, True, (), False),
    (5, 5, 2, 16, 1, 2, 5, True, False, (), False),
    (7, 7, 2, 16, 1, 2, 4, False, False, (), False),
    (7, 7, 1, 16, 1, 1, 5, True, False, (), False),
]
IDS = [f"d{s[0]}_D{s[3]}_H{s[5]}_r{s[6]}" + ("_grid" if s[7] else "") + ("_res" if s[8] else "") +
       ("_dil" if s[9] else "") + ("_rec" if s[10] else "") for s in SHAPES]


# Token counts that end inside a block of 16 keys, every even hidden unit switched off by a bias of
# -inf: a value that the network never uses, but that sits in LDS beside what it does use.
OFF_SHAPES = [(3, 4, 2, 64, 2, 4, 4, False, False, (), False), (5, 5, 1, 64, 2, 1, 4, False, False, (), False),
              (3, 4, 2, 32, 2, 4, 5, False, False, (), False), (5, 5, 2, 32, 2, 4, 4, False, False, (), True),
              (5, 5, 1, 32, 2, 2, 4, True, False, (), False)]
OFF_IDS = [f"d{s[0]}_D{s[3]}_H{s[5]}_r{s[6]}" + ("_grid" if s[7] else "") for s in OFF_SHAPES]


def case(s, off=False):
    """(workload, weights, measurement bits, types, oracle logits) of a shape; `off`: with every even
    hidden unit of every layer switched off."""
    from oracle import decoder as O
    from paper_2601_09921_amd import synth
    d, W, B, D, L, H, r, grid, res, dil, rec = s
    wl = synth.Workload("x", d, W, B, 0.1, 0.0, D, L, H, r, synth.DTYPE_F32, grid=grid, resnet=res, dil=dil)
    w = synth.make_weights(wl, seed=3)
    if off:
        for lw in w["layers"]:
            lw["b1"][::2] = -float("inf")
    meas, types = synth.make_windows(wl, seed=4, realistic_boundaries=False)
    o = (O.forward_windows_recurrent if rec else O.forward_windows)(meas, types, w, d, H, grid=grid)[0]
    return wl, w, meas, types, o
