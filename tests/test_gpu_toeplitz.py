"""GPU tests of the one-kernel Toeplitz product (csrc/toeplitz.hip): every transform length up to
8192 with full, ragged and odd sizes, odd channel counts (a pair with one channel), several units
per work-group and a last work-group that is not full, channels of one pair whose sizes differ by
2^40, and the sizes on both sides of the choice at 8192.

Tolerance: the library's model of the transform's rounding, at every output i
|dy_i| <= 8 u log2(2 N) (||h||_2 ||x||_2 s / sqrt(2 N) + |y_i|), u = 2^-24, h the circulant kernel, x
the packed pair of channels, each over its scale s (the power of two of its largest entry; 1 for a
zero channel, which so receives the pair's rounding).
"""
import numpy as np
import pytest

import oracle
from parity_util import to_gpu

pytestmark = pytest.mark.gpu


def _check(lib, b, a, noalloc=False):
    B, H, C, n = a.shape
    f = lib.toeplitz_conv_noalloc if noalloc else lib.toeplitz_conv
    y = f(to_gpu(b), to_gpu(a)).cpu().numpy().astype(np.float64)
    N = 1 << max(0, (n - 1).bit_length())
    lg = np.log2(2 * N)
    rows = np.unique(np.concatenate([[0, n - 1, n // 2], np.random.default_rng(n).integers(0, n, 40)]))
    for h in range(H):
        c = np.exp(b[h].astype(np.float64))
        hn = np.linalg.norm(c)
        ah = a[:, h].astype(np.float64)                                     # [B, C, n]
        mx = np.max(np.abs(ah), axis=-1)
        s = np.where(mx > 0, 2.0 ** np.ceil(np.log2(np.where(mx > 0, mx, 1.0))), 1.0)
        sq = np.sum((ah / s[..., None]) ** 2, axis=-1)
        sq = np.concatenate([sq, np.zeros((B, C % 2))], axis=1).reshape(B, -1, 2).sum(-1)
        x = np.sqrt(np.repeat(sq, 2, axis=1)[:, :C])                        # norm of each channel's pair
        for i in rows:
            ref = ah @ c[n - 1 - i:2 * n - 1 - i]
            bound = 8 * 2.0 ** -24 * lg * (hn * x * s / np.sqrt(2 * N) + np.abs(ref))
            assert np.all(np.abs(y[:, h, :, i] - ref) <= bound), (n, h, i)


@pytest.mark.parametrize("B,H,C,n", [
    (1, 1, 1, 1), (2, 1, 3, 2), (1, 3, 5, 3), (2, 2, 4, 7), (1, 2, 33, 16), (3, 1, 7, 31), (1, 2, 18, 64), (2, 3, 11, 100),
    (1, 1, 37, 256), (5, 2, 3, 300), (1, 3, 6, 1000), (2, 2, 5, 2047), (1, 2, 4, 4096), (1, 1, 3, 5000), (2, 8, 64, 4500),
])
@pytest.mark.parametrize("causal", [False, True])
def test_toeplitz_sizes(gpu_lib, B, H, C, n, causal):
    print(f"toeplitz B={B} H={H} C={C} n={n} causal={causal}", flush=True)
    rng = np.random.default_rng([77, n, C])
    b = (0.5 * rng.standard_normal((H, 2 * n - 1))).astype(np.float32)
    if causal:
        b[:, n:] = -np.inf
    _check(gpu_lib, b, rng.standard_normal((B, H, C, n)).astype(np.float32))


@pytest.mark.parametrize("n", [50, 4096, 8192])
def test_toeplitz_channels_of_different_size(gpu_lib, n):
    """Channels 2^40 apart in one pair, a zero channel, and the call without a workspace."""
    rng = np.random.default_rng(n)
    b = (0.5 * rng.standard_normal((1, 2 * n - 1))).astype(np.float32)
    a = rng.standard_normal((1, 1, 4, n)).astype(np.float32)
    a[0, 0, 1] *= 2.0 ** 40
    a[0, 0, 2] = 0.0
    _check(gpu_lib, b, a)
    _check(gpu_lib, b, a, noalloc=True)
