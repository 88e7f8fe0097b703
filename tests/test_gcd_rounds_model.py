"""CPU model of the rounds of the block gcd over F_p (gcd_kernels.hip): 31 normal
Euclid steps on the top 64 coefficients, the matrix they produce applied to
the whole pair with the kernel's index ranges, and the division rounds of 32
quotient coefficients."""

import random

import pytest

P = 1431655751
W, TAPS, PAD = 64, 32, 36


def step(A, B):
    """(constants) of the double elimination of top-aligned A by B, deg A = deg B + 1."""
    lb, a0, a1, b1 = B[0], A[0], A[1], B[1]
    n1 = -a0
    return lb * lb % P, lb * n1 % P, -(lb * a1 + n1 * b1) % P


def window_steps(A, B):
    """Steps on windows of W lanes; lanes past what a step can know hold None."""
    MA, MB = [[1], []], [[], [1]]
    s = 0
    while s < TAPS - 1:
        l2, l1, n2 = step(A, B)
        R = []
        for i in range(W):
            v = (A[i + 2] if i + 2 < W else None, B[i + 2] if i + 2 < W else None, B[i + 1] if i + 1 < W else None)
            R.append(None if None in v else (l2 * v[0] + l1 * v[1] + n2 * v[2]) % P)
        assert R[0] is not None and R[1] is not None  # what the next step's constants read
        if R[0] == 0:
            break
        MR = []
        for h in range(2):
            n = max(len(MA[h]), len(MB[h]) + 1)
            at = lambda p, i: p[i] if 0 <= i < len(p) else 0  # noqa: E731
            MR.append([(l2 * at(MA[h], i) + l1 * at(MB[h], i - 1) + n2 * at(MB[h], i)) % P for i in range(n)])
        A, B, MA, MB = B, R, MB, MR
        s += 1
    # the entries fit the lane halves, and the shift never crosses them
    assert all(len(MB[h]) <= TAPS for h in range(2)) and len(MB[0]) <= TAPS - 1
    return s, MA, MB


def apply(M, X, Y, top):
    """sum_i M0[i] X[t - i] + M1[i] Y[t - i] for t <= top."""
    out = []
    for t in range(top + 1):
        v = 0
        for h, Z in ((0, X), (1, Y)):
            for i, m in enumerate(M[h]):
                assert t - i >= -PAD and t - i < len(Z)
                if t >= i:
                    v += m * Z[t - i]
        out.append(v % P)
    return out


def mod_rounds(X, Y):
    """X mod Y in rounds of TAPS quotient coefficients from windows of 64."""
    X, a, b = list(X), len(X) - 1, len(Y) - 1
    inv = pow(Y[b], P - 2, P)
    while a >= b:
        n, s = min(TAPS, a - b + 1), a - b
        x = [X[a - l] if a >= l else 0 for l in range(W)]
        y = [Y[b - l] if b >= l else 0 for l in range(W)][1:] + [0]
        q = []
        for _ in range(n):
            c = x[0] * inv % P
            q.append(c)
            x = [((x[i + 1] if i + 1 < W else 0) - c * y[i]) % P for i in range(W)]
        for t in range(max(0, s - n + 1) & ~3, a - n + 1):
            for j in range(n):
                i = t - s + j
                assert i <= b - 1
                if i >= 0:
                    X[t] = (X[t] - q[j] * Y[i]) % P
        a -= n
    X = X[:b]
    while X and X[-1] == 0:
        X.pop()
    return X


def mod_plain(X, Y):
    X, inv = list(X), pow(Y[-1], P - 2, P)
    while len(X) >= len(Y):
        c = X[-1] * inv % P
        for i in range(len(Y)):
            X[len(X) - len(Y) + i] = (X[len(X) - len(Y) + i] - c * Y[i]) % P
        X.pop()
    while X and X[-1] == 0:
        X.pop()
    return X


def proportional(u, v):
    return len(u) == len(v) and all((u[-1] * y - v[-1] * x) % P == 0 for x, y in zip(u, v))


@pytest.mark.parametrize("b", [63, 64, 95, 150])
def test_a_round_equals_thirty_one_divisions(b):
    rnd = random.Random(b)
    X = [rnd.randrange(1, P) for _ in range(b + 2)]
    Y = [rnd.randrange(1, P) for _ in range(b + 1)]
    s, MA, MB = window_steps(X[::-1][:W], Y[::-1][:W])
    assert s == 31
    A, B = X, Y
    for _ in range(s):
        A, B = B, mod_plain(A, B)
    a = b + 1 - s
    assert proportional(apply(MA, X, Y, a), A) and proportional(apply(MB, X, Y, a - 1), B)


def test_a_round_stops_before_a_vanishing_leading_coefficient():
    rnd = random.Random(1)
    Y = [rnd.randrange(1, P) for _ in range(80)]
    R = [rnd.randrange(1, P) for _ in range(78)]  # degree gap of two after one step
    quo = [rnd.randrange(1, P), rnd.randrange(1, P)]
    X = [0] * 81
    for i, c in enumerate(quo):
        for j, y in enumerate(Y):
            X[i + j] = (X[i + j] + c * y) % P
    for j, r in enumerate(R):
        X[j] = (X[j] + r) % P
    s, MA, MB = window_steps(X[::-1][:W], Y[::-1][:W])
    assert s == 0 and MA == [[1], []] and MB == [[], [1]]


@pytest.mark.parametrize("a,b", [(5, 5), (40, 7), (100, 99), (100, 1), (131, 67), (64, 32), (95, 64)])
def test_division_rounds(a, b):
    rnd = random.Random(a * 1000 + b)
    X = [rnd.randrange(1, P) for _ in range(a + 1)]
    Y = [rnd.randrange(1, P) for _ in range(b + 1)]
    assert mod_rounds(X, Y) == mod_plain(X, Y)
