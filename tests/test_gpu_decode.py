"""Decryption's lift and transform on the device against extended precision on the CPU."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _slots(m, N):
    """m(zeta^(5^j)) of long double coefficients."""
    i = np.arange(N, dtype=np.longdouble)
    pi = np.longdouble(4) * np.arctan(np.longdouble(1))
    w = m * (np.cos(pi * i / N) + 1j * np.sin(pi * i / N))
    f = np.fft.ifft(w) * N
    assert f.dtype == np.clongdouble
    e, x = np.empty(N // 2, dtype=np.int64), 1
    for j in range(N // 2):
        e[j], x = (x - 1) // 2, x * 5 % (2 * N)
    return f[e]


@pytest.mark.parametrize("log_n,n_q,n_p,q_bits,level,bits", [
    (10, 1, 1, 50, 0, 40),      # one limb
    (11, 2, 1, 61, 1, 60),      # an odd split of the transform; words beyond 2^53
    (12, 3, 2, 50, 2, 20),
    (12, 4, 1, 45, 3, 170),     # every digit in use
    (13, 18, 2, 50, 17, 300),
    (16, 8, 2, 50, 1, 62),
])
def test_slots_of_a_known_polynomial(log_n, n_q, n_p, q_bits, level, bits):
    from paper_2506_10399_amd import ficgcn as fg
    ctx = fg.Context(log_n, n_q, q_bits, n_p, 61)
    N, q = ctx.N, ctx.ckks_ctx_moduli()[: level + 1]
    cl, _ = ctx.ckks_keygen(5, [], with_relin=False)
    Q = int(np.prod(np.array(q, dtype=object)))
    rng = np.random.default_rng(log_n)
    words = [int.from_bytes(rng.bytes(bits // 8 + 1), "little") % (1 << bits) for _ in range(N)]
    m = [v if rng.random() < 0.5 else -v for v in words]
    m[:6] = [0, 1, -1, 2, -2, 3]
    if bits + 4 > sum(x.bit_length() for x in q):
        m[6:8] = [(Q - 1) // 2, -((Q - 1) // 2)]
    scale = 2.0 ** 40
    res = np.zeros((2, level + 1, N), dtype=np.uint64)      # the second polynomial is zero: it decrypts to the first
    for i, p in enumerate(q):
        res[0, i] = np.array([v % p for v in m], dtype=np.uint64)
    ct = ctx.ckks_ct_load(res, level)
    ld = np.array([np.ldexp(np.longdouble(abs(v) >> max(0, v.bit_length() - 63)), max(0, v.bit_length() - 63))
                   * (1 if v >= 0 else -1) for v in m])
    want = _slots(ld / np.longdouble(scale), N)
    # each of log N steps rounds by a few 2^-53 of the values' size, which is about the polynomial's 2-norm
    tol = 16 * log_n * 2.0 ** -53 * float(np.sqrt(np.sum((ld / np.longdouble(scale)) ** 2)))
    for n in (1, 130, N // 2):
        got = ctx.ckks_decrypt(cl, ct, level, scale, n)
        assert got.shape == (n,)
        assert np.max(np.abs(got - want[:n].astype(complex))) <= tol
