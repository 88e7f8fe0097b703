"""CPU model of the interpolation on the geometric nodes 2^i (interp_geo.hip):
the divided differences and the expansion of the Newton form as one triangular
convolution each, and the cut of that convolution into column tiles and
windows with the kernel's index arithmetic and bounds."""

import random

import pytest

import paper_1201_1548_amd as br

MAX_POINTS = 8192


def tables(p, n):
    inv = lambda z: pow(z, p - 2, p)  # noqa: E731
    u = [1]
    for m in range(1, n):
        u.append(u[-1] * (pow(2, m, p) - 1) % p)
    iu = [inv(x) for x in u]
    b = [(-1) ** j * pow(2, j * (j - 1) // 2, p) * iu[j] % p for j in range(n)]
    w = [u[k] * inv(pow(2, k * (k - 1) // 2, p)) % p for k in range(n)]
    return iu, b, w


def windowed(x, b, D, nwin, p):
    """The tiled convolution: every output of the nt tiles, window by window."""
    nt = (D + 255) // 256
    plane = list(x)
    out = []
    for R in range(nt):
        nw = min(4 * (R + 1), nwin)
        assert nw <= 4 * nt
        for col in range(16):
            c = 16 * R + col
            for s in range(16):
                acc = 0
                for win in range(nw):
                    for kk in range(64):
                        j, i = 16 * c - 48 - 64 * win + kk, s + 48 + 64 * win - kk
                        assert -256 <= j < 256 * nt and i < 256 * nt  # LDS planes and table
                        if i >= 0 and j >= 0:
                            acc += b[i] * plane[j]
                out.append(acc % p)
    return out


def interpolate(v, p):
    D = len(v)
    Dr = (D + 255) // 256 * 256
    iu, b, w = tables(p, Dr)
    x = [v[i] * iu[i] % p if i < D else 0 for i in range(Dr)]
    y = windowed(x, b, D, (D - 1) // 64 + 1, p)
    e = [0] * Dr
    for k in range(Dr):
        e[Dr - 1 - k] = y[k] * w[k] % p if k < D else 0
    z = windowed(e, b, D, (D + 14) // 64 + 1, p)
    return [z[Dr - 1 - j] * iu[j] % p for j in range(D)]


@pytest.mark.parametrize("D", [1, 2, 17, 63, 65, 130, 256, 257, 300])
def test_two_windowed_convolutions_interpolate(D):
    p = br.primes(1)[0]
    rnd = random.Random(D)
    f = [rnd.randrange(p) for _ in range(D)]
    v = [sum(c * pow(pow(2, i, p), j, p) for j, c in enumerate(f)) % p for i in range(D)]
    assert interpolate(v, p) == f


def test_two_has_order_above_max_points_for_every_table_prime():
    for p in br.primes(2048):
        m = p - 1
        assert all(m % d or pow(2, d, p) != 1 for d in range(1, MAX_POINTS + 1))
