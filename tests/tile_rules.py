"""The rules of csrc/tile_rules.h once more, for GPU tests that have to know which kernel a launch takes
(test_tile_rules.py holds the two together)."""
import math

TILE_256x256, TILE_256x128, TILE_128x128, TILE_64x128, TILE_128x64, TILE_64x64, TILE_32x64 = range(7)
F32_128x128, F32_64x64, F32_32x64_STEP4, F32_32x64, F32_32x32_STEP4, F32_32x32 = range(6)


def tiles(n_probs, rows, cols, bm, bn):
    return -(-rows // bm) * -(-cols // bn) * n_probs


def rounds(*launch):
    return -(-tiles(*launch) // 256)


def f32_tile(n_probs, rows, cols, k):
    launch = (n_probs, rows, cols)
    if tiles(*launch, 64, 64) >= 512:
        large = k >= 512 and tiles(*launch, 128, 128) > 256 and 3.9 * rounds(*launch, 128, 128) <= 0.5 * (rounds(*launch, 64, 64) + tiles(*launch, 64, 64) / 256)
        return F32_128x128 if large else F32_64x64
    fours = k // 32 % 4 == 0 or k // 32 > 12
    if tiles(*launch, 32, 32) <= 256:
        return F32_32x32_STEP4 if fours else F32_32x32
    if tiles(*launch, 32, 64) <= 256:
        return F32_32x64_STEP4 if fours else F32_32x32
    return F32_32x32 if 1.1 * rounds(*launch, 32, 32) < 2 * rounds(*launch, 32, 64) else F32_32x64


def wide_ok(rows, cols, k, row_stride):
    """gemm8_wide_ok for the plain products of the path (k: bytes of a row)."""
    return rows >= 256 and cols >= 256 and k >= 256 and cols % 4 == 0 and row_stride % 32 == 0


def exact_tile(n_probs, rows, cols, k, b16=False, kl=False, wide=False, residual=False):
    def per_cu(bm, bn):
        return float(rounds(n_probs, rows, cols, bm, bn))
    narrow = cols <= 64 and not kl
    best, r = (TILE_128x64, per_cu(128, 64)) if narrow else (TILE_128x128, per_cu(128, 128))
    cost = 0.37 + 0.48 * r if narrow else 0.5 + 0.85 * r
    large = False
    if not narrow and not b16 and not kl and rows >= 8192 and cols >= 128:
        rp = per_cu(256, 128)
        if rp >= 5 or 0.1 + 1.8 * rp <= cost:
            best, r, cost, large = TILE_256x128, rp, 0.1 + 1.8 * rp, rp >= 5
    if not large:
        if r > 1 and k > 1024:
            cost *= 0.94
        others = [] if narrow else [(TILE_64x128, 0.37 + 0.48 * per_cu(64, 128))]
        if not kl:
            others += [(TILE_64x64, 0.3 + 0.26 * per_cu(64, 64)), (TILE_32x64, 0.27 + 0.17 * per_cu(32, 64))]
        for tile, c in others:
            if c < cost:
                best, cost = tile, c
    if wide:
        t = tiles(n_probs, rows, cols, 256, 256) / 256
        per_round = 1.2 + 40.0 / k if b16 else 1.25 + (300.0 if residual else 120.0) / k
        short_rows = b16 and residual and k <= 1024 and t < 2
        if not short_rows and 0.6 + per_round * (math.ceil(t) + t) <= 0.94 * cost:
            best = TILE_256x256
    return best
