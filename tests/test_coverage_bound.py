"""The forward finds a pixel's candidate entries from the sign of a polynomial
q(X, Y) - q_cut - slack whose coefficients enter a matrix product as two or
three bf16 pieces.  Checked here with that arithmetic in numpy: no pixel that
the exact FP32 test (q <= q_cut) accepts may be missed, for the view-tied
range of conics, strongly anisotropic, very large and very small ones, and
few others may be let through (they cost a step each)."""
import numpy as np
import pytest

F = np.float32
Q_CUT = F(11.0826)


def bf16(x):
    u = np.asarray(x, F).view(np.uint32).astype(np.uint64)
    return ((((u + 0x7fff + ((u >> 16) & 1)) >> 16) << 16).astype(np.uint32)).view(F)


def pieces(x, n):
    out = []
    for _ in range(n):
        out.append(bf16(x))
        x = (x - out[-1]).astype(F)
    return out


def conics(kind, rng, n):
    if kind == "view":
        s1 = rng.uniform(0.3, 5, n); s2 = s1 * rng.uniform(0.2, 1, n)
    elif kind == "aniso":
        s1 = 10 ** rng.uniform(-0.5, 6, n); s2 = np.maximum(0.3, s1 * 10 ** rng.uniform(-6, 0, n))
    elif kind == "large":
        s1 = 10 ** rng.uniform(2, 8, n); s2 = s1 * rng.uniform(0.01, 1, n)
    else:
        s1 = 10 ** rng.uniform(-6, 0, n); s2 = s1 * rng.uniform(0.01, 1, n)
    th = rng.uniform(0, np.pi, n)
    c, s = np.cos(th), np.sin(th)
    a, b, d = c * c * s1 + s * s * s2, c * s * (s1 - s2), s * s * s1 + c * c * s2
    det = a * d - b * b
    return (d / det).astype(F), (-b / det).astype(F), (a / det).astype(F), np.sqrt(Q_CUT * s1)


@pytest.mark.parametrize("tile", [8, 16, 32])
@pytest.mark.parametrize("kind", ["view", "aniso", "large", "small"])
def test_no_accepted_pixel_is_missed(tile, kind):
    rng = np.random.default_rng(tile)
    n = 4000
    qa, qb, qc, ext = conics(kind, rng, n)
    ox, h = F(592), F(tile // 2)
    cx = ox + h
    reach = np.minimum(ext, 1e4) + tile / 2
    mx = (cx + rng.uniform(-1, 1, n) * reach).astype(F)
    my = (cx + rng.uniform(-1, 1, n) * reach).astype(F)
    A, B, C, ux, uy = qa, F(2) * qb, qc, mx - cx, my - cx
    D, E = -(F(2) * A * ux + B * uy), -(F(2) * C * uy + B * ux)
    S, M = abs(A) + abs(B) + abs(C), np.maximum(abs(ux), abs(uy)) + h
    slack = S * (M * M * F(2 ** -18) + h * h * F(2 ** -16)) + F(1e-5) * Q_CUT
    Fc = F(-0.5) * (D * ux + E * uy) - (Q_CUT + slack)
    rows = [pieces(A, 2), pieces(B, 2), pieces(C, 2), pieces(D, 3), pieces(E, 3), pieces(Fc, 3)]
    missed = accepted = 0
    for X in range(-tile // 2, tile // 2):
        for Y in range(-tile // 2, tile // 2):
            p = np.zeros(n, F)
            for pc, m in zip(rows, (X * X, X * Y, Y * Y, X, Y, 1)):
                assert bf16(F(m)) == F(m)  # the monomials are exact in bf16
                for v in pc:
                    p = (p + v * F(m)).astype(F)
            dx, dy = (F(X) + cx - mx).astype(F), (F(Y) + cx - my).astype(F)
            fma = lambda x, y, z: (x.astype(np.float64) * y + z).astype(F)
            q = fma(qc * dy, dy, fma(B * dx, dy, (qa * dx) * dx))
            acc, bit = q <= Q_CUT, np.signbit(p)
            missed += int((acc & ~bit).sum())
            assert np.all(q[bit] <= Q_CUT + F(2) * slack[bit])
            accepted += int(acc.sum())
    assert missed == 0
    assert accepted > 0
