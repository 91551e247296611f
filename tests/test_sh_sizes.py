"""Which Shack-Hartmann sizes are admitted (host only): the rule of the unfolded
tables, and every admitted size's folded tables fit the 160 KiB of LDS."""

import pytest

from paper_2602_06688_amd import pwfs as P


def _unfolded(b, M, k):
    wide, tall = (b + 1 if b % 2 == 0 else b), (257 if M <= 256 else M)
    return 8 * (M * wide + b * tall + b * b) + 4 * (k * k + 256)


def _folded(b, M, k):
    h, hm = (b + 1) // 2, (M + 1) // 2
    return 16 * (h * M + 2 * h * h) + 8 * (hm * (h | 1) + b * b) + 4 * (k * k + 1 + 512)


def _validate(b, M, r):
    import ctypes
    d = P.sh_desc(4 * b, 4, M, r, 0.0, 750.0)
    return P.lib().pwfs_sh_validate(ctypes.byref(d))


@pytest.mark.parametrize("b", range(1, 33))
def test_admitted_sizes(b):
    for M in range(2, 513):
        for r in (1, 2, 3, 4, 7, 16, M // 2, M):
            if r < 1 or M % r:
                continue
            k = M // r
            want = 0 if _unfolded(b, M, k) <= 150 * 1024 else P.PWFS_EUNSUPPORTED
            assert _validate(b, M, r) == want, (b, M, r)
            assert want or _folded(b, M, k) <= 160 * 1024
