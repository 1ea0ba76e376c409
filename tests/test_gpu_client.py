"""Encoding and encryption, whose transforms' column passes make their own input, at the edges of their tiles."""
import numpy as np
import pytest

from oracle import ckks
from oracle.params import Params

pytestmark = pytest.mark.gpu

RINGS = [   # log_n, n_q, q_bits, n_p, p_bits, log2 of the column pass (0: log_n / 2)
    (9, 1, 30, 1, 31, 0),      # 16-point columns and 32-point rows
    (10, 4, 45, 1, 50, 0),     # primes below the fp64 range
    (11, 3, 50, 2, 60, 0),
    (12, 3, 61, 1, 61, 8),     # the widest primes; 256-point columns and 16-point rows
    (13, 5, 50, 1, 60, 9),     # a split beyond the fused passes' 256 points
    (13, 2, 52, 1, 60, 5),
    (17, 2, 50, 2, 60, 0),     # 512-point rows
]


@pytest.mark.parametrize("ring", RINGS, ids=lambda r: "-".join(map(str, r)))
def test_encoding_and_encryption(ring):
    from paper_2506_10399_amd import ficgcn as fg
    log_n, n_q, q_bits, n_p, p_bits, split = ring
    d = dict(log_n=log_n, n_q=n_q, q_bits=q_bits, n_p=n_p, p_bits=p_bits, log_scale=20)
    prm, ctx = Params.from_dict(d), fg.Context.from_dict(d)
    if split:
        ctx.ckks_ntt_config(split, 16, 4)
    N, level, q = prm.N, n_q - 1, prm.q_level(n_q - 1)
    keys = ckks.keygen(prm, 5, [], relin=False)
    cl, _ = ctx.ckks_keygen(5, [], with_relin=False)
    rng = np.random.default_rng(log_n)
    # the library's plaintexts: one polynomial's residues on every limb, each coefficient the exact one rounded
    rows, scale = rng.uniform(-1, 1, (3, N // 2 - 7)), 2.0 ** (min(62, sum(x.bit_length() for x in q) - 2) - 4)
    pts = ctx.ckks_encode_batch(rows, scale, level)
    coefs = [ctx.ckks_poly_store(pts[i], level, 1)[0] for i in range(3)]
    pi, i = np.longdouble(4) * np.arctan(np.longdouble(1)), np.arange(N, dtype=np.longdouble)
    for z, m in zip(rows, coefs):
        v = np.zeros(N, dtype=np.clongdouble)
        e = 1
        for x in z:
            v[(e - 1) // 2] = v[(2 * N - e - 1) // 2] = x
            e = e * 5 % (2 * N)
        exact = (np.fft.fft(v) * (np.cos(pi * i / N) - 1j * np.sin(pi * i / N))).real / N * np.longdouble(scale)
        # centred on as many limbs as hold it
        k = next(j for j in range(1, n_q + 1) if sum(x.bit_length() - 1 for x in q[:j]) > np.log2(scale) + 3)
        Q = int(np.prod(np.array(q[:k], dtype=object)))
        r = sum(m[j].astype(object) * (Q // q[j] * pow(Q // q[j], -1, q[j])) for j in range(k)) % Q
        r = np.array([int(x) - Q if x > Q // 2 else int(x) for x in r], dtype=object)
        for j in range(n_q):
            assert np.array_equal((r % q[j]).astype(np.uint64), m[j])
        # each of log N steps rounds by a few 2^-53 of the values' size (at most scale times the slots' rms)
        err = np.abs(np.array([np.longdouble(int(x)) for x in r]) - exact)
        assert err.max() <= 0.5 + 16 * log_n * 2.0 ** -53 * scale
    # encryption: the oracle's words
    for ct_id, m in ((0, coefs[0]), (2 ** 32 - 1, coefs[1])):
        want = ckks.encrypt(prm, 7, ct_id, keys.s, type("Pt", (), {"m": m, "level": level, "scale": scale})())
        ct = ctx.ckks_encrypt(cl, ctx.ckks_pt_load(m, level), level, 7, ct_id)
        assert np.array_equal(ctx.ckks_poly_store(ct, level, 2), np.stack([want.c0, want.c1]))
        seeded = ctx.ckks_encrypt_seeded(cl, ctx.ckks_pt_load(m, level), level, 8, 9, ct_id)
        want = ckks.encrypt(prm, 8, ct_id, keys.s, type("Pt", (), {"m": m, "level": level, "scale": scale})(), a_seed=9)
        assert np.array_equal(ctx.ckks_poly_store(seeded, level, 2), np.stack([want.c0, want.c1]))
