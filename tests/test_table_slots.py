"""The arithmetic by which kernels find a table's slot (csrc/nm_device.h, slot_offset), on the CPU: for every position the slot
holds the segment that the normative rule (subtract, multiply, clamp, floor in fp32) gives, around every break point, at both
ends and beyond them, for segment widths that are and are not a power of two."""
import numpy as np
import pytest

F = np.float32


def segments(x, lo, inv_w, nseg):
    with np.errstate(over="ignore", invalid="ignore"):
        u = (x - F(lo)) * F(inv_w)
        return np.floor(np.fmin(np.fmax(u, F(0)), F(nseg - 1))).astype(np.int64)


def slot_segments(x, lo, inv_w, nseg, pow2):
    """slot_offset on 1/256 of the position, then the entry that write_slots puts there.  The products by powers of two are exact in
    binary64, and rounding a sum of such numbers there first can only turn a position just off an integer into that integer."""
    iw = F(F(inv_w) / F(256))
    with np.errstate(over="ignore", invalid="ignore"):
        if pow2:
            u = (x.astype(np.float64) * np.float64(iw) + np.float64(F(F(-F(lo) * F(inv_w)) / F(256)))).astype(F)
        else:
            u = (x - F(lo)) * iw
    u = np.where(np.isnan(u), F(0), np.clip(u, F(0), F(1)))
    s = (u.astype(np.float64) * 2048.0 + 8388607.5).astype(F)
    slot = (s.view(np.uint32) & np.uint32(0xff8)) >> 3
    table = np.full(512, -1)
    table[:256] = np.minimum(np.arange(256), nseg - 1)
    table[256], table[511] = nseg - 1, 0
    return table[slot]


@pytest.mark.parametrize("lo,hi,nseg", [(-8.0, 8.0, 128), (-16.0, 0.0, 256), (-16.0, 0.0, 16), (-8.0, 8.0, 100), (1e-3, 64.0, 255),
                                        (1.0, 512.0, 37), (0.0, 3.0, 3), (-1.0, 1.0, 2), (-4.0, 4.0, 1), (0.0, 1e-20, 64), (-1e20, 1e20, 256)])
def test_slots_hold_the_rules_segments(lo, hi, nseg):
    inv_w = F(nseg / (float(F(hi)) - float(F(lo))))
    pow2 = np.frexp(inv_w)[0] == 0.5
    edges = (np.float64(lo) + np.arange(-2, nseg + 3) * (np.float64(hi) - lo) / nseg).astype(F)
    steps = np.arange(-300, 301)
    key = edges.view(np.int32)
    key = np.where(key < 0, np.int32(-2147483648) - key, key).astype(np.int64)   # neighbours in value are neighbours in key
    key = np.clip(key[:, None] + steps[None, :], -0x7f7fffff, 0x7f7fffff)
    bits = np.where(key < 0, -2147483648 - key, key).astype(np.int64).astype(np.uint32)
    g = np.random.default_rng(nseg)
    span = float(hi) - float(lo)
    x = np.concatenate([bits.astype(np.uint32).view(F).ravel(), g.uniform(lo - span, hi + span, 200000).astype(F),
                        np.array([0.0, -0.0, 1e38, -1e38, np.inf, -np.inf, 1e-45, -1e-45, 1e-38, lo, hi], F)])
    want = segments(x, lo, inv_w, nseg)
    assert (slot_segments(x, lo, inv_w, nseg, False) == want).all()
    if pow2:
        assert (slot_segments(x, lo, inv_w, nseg, True) == want).all()
