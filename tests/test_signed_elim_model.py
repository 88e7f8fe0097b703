"""CPU model of the signed Montgomery arithmetic of ee.hip: the reduction's
identity and bound, the balanced representative, the invariant |x| <= 1.126 p of
a chain of remainder steps without corrections, and the widths of the sums that
join the digit products of the evaluation."""

import random

import pytest

import paper_1201_1548_amd as br

W = 1 << 32


def s32(x):
    return (x + (1 << 31)) % W - (1 << 31)


def redc(t, p):
    assert -(1 << 63) <= t < 1 << 63
    m = s32(t * pow(p, -1, W))
    r = (t >> 32) - (m * p >> 32)
    assert (t - m * p) % W == 0 and r == (t - m * p) // W
    assert abs(r) <= abs(t) / W + p / 2 and -(1 << 31) <= r < 1 << 31
    return r


def balance(x, p):
    h = (p - 1) >> 1
    v = (x + h) % W
    v = min(v, (v + p) % W)
    v = min(v, (v - p) % W)
    v = s32((v - h) % W)
    assert (v - x) % p == 0 and abs(v) <= h
    return v


@pytest.fixture(scope="module", params=[0, -1])
def prime(request):
    return br.primes(64)[request.param]


def test_reduction_and_balance(prime):
    p = prime
    rng = random.Random(p)
    lim = 3 * p // 2 - 1
    for x in [0, 1, -1, p, -p, p // 2, -(p // 2), p // 2 + 1, lim, -lim] + [rng.randint(-lim, lim) for _ in range(2000)]:
        balance(x, p)
        y = rng.choice([lim, -lim, rng.randint(-lim, lim)])
        assert (redc(x * y, p) * W - x * y) % p == 0


def test_remainder_chain_keeps_the_bound(prime):
    p = prime
    rng = random.Random(p + 1)
    B = 9 * p // 8
    one = W % p
    for ext in (False, True):
        pick = (lambda: rng.choice([B, -B])) if ext else (lambda: rng.randint(-B, B))
        n = 24
        X, Y = [pick() for _ in range(n)], [pick() for _ in range(n - 1)]
        a0 = balance(X[0], p)
        while len(Y) > 1:
            lb = balance(Y[0], p)
            if lb == 0 or a0 == 0:
                break
            Xp, Yp = X + [0, 0], Y + [0, 0, 0]
            n2 = balance(redc(a0 * Yp[1] - lb * Xp[1], p), p)
            l2, l1 = redc(lb * lb, p), redc(-lb * a0, p)
            assert max(abs(l2), abs(l1)) <= 0.584 * p
            R = [redc(l2 * Xp[k + 2] + l1 * Yp[k + 2] + n2 * Yp[k + 1], p) for k in range(len(Y) - 1)]
            assert max(abs(r) for r in R) <= 1.126 * p
            # against lb^2 A mod B with the Montgomery factors taken out
            ri = pow(W, -1, p)
            A = [x * lb * lb * ri * ri for x in X]
            q1 = lb * a0 * ri * ri
            T = [A[i] - q1 * Yp[i] for i in range(len(X))]
            assert T[0] % p == 0
            q0 = (lb * X[1] - a0 * Yp[1]) * ri * ri
            assert [(T[k + 2] - q0 * Yp[k + 1] - r) % p for k, r in enumerate(R)] == [0] * len(R)
            X, Y, a0 = Y, R, lb
    assert abs(balance(one, p)) <= p // 2


def test_paired_division_steps_keep_their_bound(prime):
    # A[j] <- A[j+2] + y1 B[j+2] + y0 B[j+1] with 1 / lc(B) balanced: |A| <= 1.3 p throughout
    p = prime
    rng = random.Random(p + 2)
    one, ri = balance(W % p, p), pow(W, -1, p)
    for ext in (False, True):
        pick = (lambda: rng.choice([9 * p // 8, -(9 * p // 8)])) if ext else (lambda: rng.randint(-p, p))
        m, n = 31, 6
        A, B = [pick() for _ in range(m + 1)], [pick() for _ in range(n + 1)]
        lb = balance(B[0], p)
        ninv = redc(-pow(lb, -1, p) * pow(W, 2, p) % p * W, p)  # any representative up to 0.6 p
        ninv = balance(ninv, p) if abs(ninv) > 0.6 * p else ninv
        ref = [a % p for a in A]
        Bp = B + [0] * (m + 3)
        ap = m
        while ap > n:
            y1 = redc(A[0] * ninv, p)
            y0 = redc(redc(one * A[1] + y1 * Bp[1], p) * ninv, p)
            assert max(abs(y1), abs(y0)) <= 0.76 * p
            A = A + [0, 0]
            A = [redc(one * A[j + 2] + y1 * Bp[j + 2] + y0 * Bp[j + 1], p) if j < n else A[j + 2]
                 for j in range(len(A) - 2)][: ap - 1]
            assert max(abs(a) for a in A) <= 1.3 * p
            for _ in range(2):
                q = ref[0] * pow(B[0], -1, p) % p
                ref = [(ref[j + 1] - q * Bp[j + 1]) % p for j in range(len(ref) - 1)]
            assert [a % p for a in A] == ref
            ap -= 2
    assert ri * W % p == 1


@pytest.mark.parametrize("kw", [32, 64])
def test_digit_products_join_in_the_given_widths(prime, kw):
    p = prime
    h = (p - 1) // 2
    top = ((h + 0x808080) >> 24) + 1
    G = [0] * 7
    for s in range(4):
        for r in range(4):
            G[s + r] += kw * (top if s == 3 else 128) * (top if r == 3 else 128)
    assert top <= 65
    for c in (0, 2, 4):
        assert G[c] + 256 * G[c + 1] < 1 << 31
    S = (G[0] + 256 * G[1]) + (G[2] + 256 * G[3]) * 65536 + (G[4] + 256 * G[5]) * h + G[6] * h
    assert S / W + p / 2 <= 9 * p / 8  # the values enter the chain within its bound
    for v in (h, -h, 0, 1, -1, 12345678, -87654321):
        w = ((v + 0x808080) % W) ^ 0x808080
        d = [((w >> (8 * s) & 255) + 128) % 256 - 128 for s in range(4)]
        assert sum(x << (8 * s) for s, x in enumerate(d)) == v


def test_tile_rows_and_transposed_points():
    # row slot rho holds row 4 (rho % 4) + rho / 4: register j of lane group g is row 4 j + g
    assert sorted(4 * (rho & 3) + (rho >> 2) for rho in range(16)) == list(range(16))
    # u[t][j] of lane (g, x): row slot 4 g + j at point 16 t + x; after the swaps lane (g, x)
    # holds rows 4 j + r of point 16 g + x
    for j in range(4):
        u = [[(4 * g + j, 16 * t + x) for g in range(4) for x in range(16)] for t in range(4)]

        def swap32(a, b):  # upper half of a with the lower half of b
            return a[:32] + b[:32], a[32:] + b[32:]

        def swap16(a, b):  # odd rows of 16 of a with the even rows of b
            return a[:16] + b[:16] + a[32:48] + b[32:48], a[16:32] + b[16:32] + a[48:] + b[48:]

        s0, s2 = swap32(u[0], u[2])
        s1, s3 = swap32(u[1], u[3])
        v = swap16(s0, s1) + swap16(s2, s3)
        for lane in range(64):
            for r in range(4):
                slot, point = v[r][lane]
                assert point == lane and 4 * (slot & 3) + (slot >> 2) == 4 * j + r
