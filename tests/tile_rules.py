"""The rules of csrc/tile_rules.h once more, for GPU tests that have to know which kernel a launch takes
(test_tile_rules.py holds the two together)."""
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
