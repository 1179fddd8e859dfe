"""Which bands of widths sum together and in which form: the choice of choose_bands (csrc/spcfg_api.hip) and band_grid
(csrc/kernels_elem.hip) once more, so that a test can assert which kernels its case reaches."""
W = 4                                         # widths of a band, starts of a tile
TABLES, BYTES, BYTES_MANY, MANY_WAVES = 3072, 100e6, 50e6, 16384
CHAIN, FEW_WAVES, MIN_WAVES = 48, 768, 1536


def choose(N, lens):
    """({first width: wavefronts that share 64 nonterminals (1 or 16)} of the forward bands, the same of the reverse ones)"""
    blocks, n_long = (N + 63) // 64, max(lens)
    fwd, bwd = {}, {}
    for w0 in range(0, n_long, W):
        rows, steps, tiles = [0, 0], [0, 0], 0
        for n in lens:
            if n < w0:
                continue
            t = (n - w0 + W) // W
            tiles += t
            steps[0] += t * (w0 + 2)
            steps[1] += t * (n - w0)
            for w in range(max(w0, 1), min(w0 + W - 1, n) + 1):
                spans = n - w + 1
                rows[0] += spans * (2 * (w - 1) - 4 * (w - w0) - 2)
                rows[1] += spans * (2 * (n - w) - 4 * min(w0 + W - 1 - w, n - w) - 4)
        for side, out, chain in ((0, fwd, w0 >= CHAIN), (1, bwd, n_long - w0 >= CHAIN)):
            waves = (side + 1) * tiles * blocks
            saved = 4 * 64 * blocks * (rows[side] - (2 * W + 3) * steps[side]) - TABLES * steps[side]
            if side == 0 and w0 < 2 * W:
                continue
            if saved >= (BYTES_MANY if waves >= MANY_WAVES else BYTES) or (chain and waves < FEW_WAVES):
                out[w0] = 16 if waves < MIN_WAVES else 1
    return fwd, bwd
