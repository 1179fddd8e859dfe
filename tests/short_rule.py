"""Which kernel a projection launch takes, and with which tile: the choice of pick_shape (csrc/gemm_short.hip) with the tile
heights of csrc/gemm_nt_common.h once more, so that a test can assert what its case reaches (fp32, split products)."""
# tiles of 16 mi rows x 16 ni columns: (mi, ni, us a round, us a round and 1024 values of K)
SHAPES = [(1, 1, 0.2, 1.95), (2, 1, 0.6, 2.6), (2, 2, 0.7, 3.9), (4, 2, 1.4, 6.2), (4, 4, 3.0, 9.55)]


def tile_height(rows, work, wide):
    if rows <= 32 or work <= 1.6e9:
        return 32
    return 64 if rows <= 64 or work <= (3.2e9 if wide else 4.3e9) else 128


def pick(rows, cols, K, parts=None, groups=None):
    """(rows, columns) of the tile, or None where gemm_nt.hip runs.  parts: (rows, 32-value steps of K); groups: rows a sentence."""
    most = max(groups) if groups else rows
    work = sum(r * cols * kt * 32 for r, kt in parts) if parts else most * cols * K
    if tile_height(most, work, (parts is not None and len(parts) == 2) or cols > K) == 128:
        return None
    best, limit = None, 0.9 * (15.0 + 12.5e-9 * work * (len(groups) if groups else 1))
    for mi, ni, fixed, slope in SHAPES:
        bm = 16 * mi
        if groups:
            tiles = sum(-(-c // max(bm, 32)) for c in groups) * (2 if bm == 16 else 1)
        else:
            tiles = sum(-(-r // bm) for r, _ in parts) if parts else -(-rows // bm)
        rounds = -(-tiles * -(-cols // (16 * ni)) // 256)
        t = 2.0 + rounds * (fixed + slope * K / 1024.0)
        if t < limit:
            best, limit = (16 * mi, 16 * ni), t
    return best


def tiles(N, P, lens, per_sentence=False):
    """The launches of a batch, forward and reverse: sets of "RxC" (rows x columns of the tile; "gemm_nt" where that kernel runs),
    with a "p" behind it where the launch is cut into parts."""
    Np, Pp, kt = -(-N // 64) * 64, -(-P // 64) * 64, -(-N // 64) * 2
    fwd, bwd = set(), set()
    name = lambda tile, parts=False: "gemm_nt" if tile is None else "%dx%d" % tile + ("p" if parts else "")
    for w in range(1, max(lens)):
        c = [n - w + 1 for n in lens if n >= w]
        rows, groups = sum(c), c if per_sentence else None
        if w == 1:
            fwd.add(name(pick(rows, 2 * Np, Pp, groups=groups)))
            bwd.add(name(pick(rows, P, 2 * Np, groups=groups)))
            continue
        n_pre, n_suf, n_mid = len(c), sum(x >= 2 for x in c), sum(max(0, x - 2) for x in c)
        if per_sentence or Np % 128:
            fwd.add(name(pick(rows, 2 * Np, Np, groups=groups)))
        else:
            fwd.add(name(pick(rows, Np, Np, parts=[(n_pre + n_mid, kt), (n_mid + n_suf, kt)]), True))
        if per_sentence:
            bwd.add(name(pick(rows, Np, 2 * Np, groups=groups)))
            continue
        parts = [(n_pre, kt), (n_mid, 2 * kt), (n_suf, kt)]
        bm = tile_height(rows, sum(r * Np * k * 32 for r, k in parts), False)
        keep = -(-rows // bm) * 2 * kt > sum(-(-r // bm) * k for r, k in parts)
        bwd.add(name(pick(rows, Np, 2 * Np, parts=parts if keep else None), keep))
    return fwd, bwd
