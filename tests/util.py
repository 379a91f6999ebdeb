"""Shared helpers of the GPU parity tests (no arithmetic of the method lives here)."""
import numpy as np

TOL = 1e-2  # elementwise bound |gpu - oracle| <= TOL * (1 + |oracle|)


def dev(a):
    import torch
    return None if a is None else torch.from_numpy(np.ascontiguousarray(a)).cuda()


def host(t):
    return t.detach().cpu().numpy()


def assert_close(gpu, ref, what=""):
    g = np.asarray(gpu, dtype=np.float64)
    r = np.asarray(ref, dtype=np.float64)
    assert g.shape == r.shape, (what, g.shape, r.shape)
    assert np.all(np.isfinite(g)), what + ": non-finite GPU output"
    err = np.abs(g - r)
    bound = TOL * (1.0 + np.abs(r))
    bad = err > bound
    if bad.any():
        i = np.unravel_index(np.argmax(err - bound), err.shape)
        raise AssertionError("%s: %d of %d outside tolerance; worst at %s gpu=%r oracle=%r" %
                             (what, int(bad.sum()), bad.size, i, g[i], r[i]))


def assert_bit_equal(gpu, ref, what=""):
    g = np.ascontiguousarray(gpu).view(np.uint16)
    r = np.ascontiguousarray(ref).view(np.uint16)
    assert g.shape == r.shape, (what, g.shape, r.shape)
    # +0 and -0 compare equal as values; integer-valued cases never produce -0 after ReLU / sums
    if not np.array_equal(g, r):
        diff = np.argwhere(g != r)
        i = tuple(diff[0])
        raise AssertionError("%s: %d elements differ; first at %s gpu=%r oracle=%r" %
                             (what, len(diff), i, np.asarray(gpu)[i], np.asarray(ref)[i]))


def patch_share(N, P, Q, K1):
    """Waves per unit behind the last whole round of a pair with a residual, from the rule of conv_patch_kernel: units of 4 x (6 to 8) pixels
    for 256 workgroups of four waves, 128 waves on each of eight XCDs, and the columns of op1 in chunks of 64."""
    units_of = lambda tq: N * -(-P // 4) * -(-Q // tq)
    units = units_of(min((8, 7, 6), key=lambda tq: (-(-units_of(tq) // 1024) * (8 + tq), -tq)))
    left, chunks = -(-units // 8) % 128, -(-K1 // 64)
    if units < 1024 or left == 0 or left * 2 > 128 or chunks < 2:
        return 1
    return 4 if left * 4 <= 128 and chunks > 3 else 3 if left * 3 <= 128 and chunks > 2 else 2


# 1029 to 2100 units of 8 columns for 1024 waves; and images of 56 columns, whose units have 6 or 7: 1470 to 2016
# Case: N H W C K0 R stride pad K1 of a pair, and the waves that share a unit behind the last whole round.
PATCH_SHARES = [
    ((147, 28, 8, 8, 24, 3, 1, 1, 256), 4), ((192, 28, 8, 8, 24, 3, 1, 1, 256), 3), ((175, 28, 8, 8, 24, 3, 1, 1, 136), 3), ((217, 28, 8, 8, 24, 3, 1, 1, 200), 2),
    ((175, 28, 8, 40, 24, 3, 1, 1, 72), 2), ((252, 28, 8, 8, 24, 3, 1, 1, 256), 1), ((300, 28, 8, 8, 24, 3, 1, 1, 256), 4), ((175, 55, 15, 8, 24, 3, 2, 1, 136), 3),
    ((147, 55, 15, 8, 24, 3, 2, 1, 256), 4), ((217, 28, 8, 16, 40, 1, 1, 0, 136), 2), ((192, 28, 8, 16, 40, 1, 1, 0, 256), 3), ((300, 28, 8, 72, 24, 1, 1, 0, 200), 4),
    ((21, 28, 56, 8, 24, 3, 1, 1, 256), 2), ((25, 28, 56, 16, 40, 1, 1, 0, 136), 1), ((36, 28, 56, 8, 24, 1, 1, 0, 256), 1), ((25, 55, 111, 8, 24, 3, 2, 1, 72), 1)]
