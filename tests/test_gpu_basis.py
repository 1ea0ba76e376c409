"""The transforms fused with base conversion (ModUp, ModDown, rescale) against the oracle, word for
word, at the edges of their dispatch: every column-pass size, one to three special primes (three take
the separate passes), primes inside and outside the fp64 range, the largest prime size, last digits
that are short, and small batches, whose destination limbs are split over blocks."""
import numpy as np
import pytest

from oracle import ckks, encoding as enc
from oracle.params import Params

pytestmark = pytest.mark.gpu

# log_n, n_q, q_bits, n_p, p_bits, NTT split (0: half)
RINGS = [
    (9, 3, 50, 1, 60, 0),     # 16-point column pass
    (10, 5, 50, 2, 60, 4),
    (11, 4, 50, 2, 50, 5),    # special primes in the fp64 range
    (11, 5, 50, 3, 60, 0),    # longer digits: the separate passes
    (12, 4, 45, 2, 60, 6),    # integer residues throughout
    (12, 3, 52, 1, 61, 8),    # 256-point column pass, 16-point rows; the widest primes
    (13, 5, 61, 2, 61, 9),    # a split beyond the fused passes' 256 points
    (14, 6, 50, 2, 60, 7),
    (17, 2, 50, 2, 60, 0),
]


@pytest.mark.parametrize("ring", RINGS, ids=lambda r: "-".join(map(str, r)))
def test_fused_conversions_match_oracle(ring):
    from paper_2506_10399_amd import ficgcn as fg
    log_n, n_q, q_bits, n_p, p_bits, split = ring
    d = dict(log_n=log_n, n_q=n_q, q_bits=q_bits, n_p=n_p, p_bits=p_bits, log_scale=40)
    prm, ctx = Params.from_dict(d), fg.Context.from_dict(d)
    if split:
        ctx.ckks_ntt_config(split, 16, 4)
    steps = [1, -3]
    keys = ckks.keygen(prm, 5, steps, relin=True)
    _, ev = ctx.ckks_keygen(5, steps, with_relin=True)
    rng = np.random.default_rng(log_n)
    for level in sorted({n_q - 1, (n_q - 1) // 2, 0}):
        cts, dev = [], []
        for i in range(2):
            z = rng.uniform(-1, 1, prm.M)
            cts.append(ckks.encrypt(prm, 6, 10 * level + i, keys.s, enc.encode(prm, z, prm.scale, level)))
            dev.append(ctx.ckks_ct_load(np.stack([cts[i].c0, cts[i].c1]), level))

        def check(got, want):
            lv = len(want.c0) - 1
            assert np.array_equal(ctx.ckks_poly_store(got, lv, 2), np.stack([want.c0, want.c1]))

        for out, s in zip(ctx.ckks_rotate_hoisted(ev, dev[0], level, steps), steps):
            check(out, ckks.rotate(prm, keys, cts[0], s))
        for i, out in enumerate(ctx.ckks_rotate_batch(ev, dev, level, steps)):
            check(out, ckks.rotate(prm, keys, cts[i], steps[i]))
        check(ctx.ckks_mul_relin(ev, dev[0], dev[1], level), ckks.ct_mul_relin(prm, keys, cts[0], cts[1]))
        if level:
            ctx.ckks_rescale(dev[1], level)
            check(dev[1], ckks.rescale(prm, cts[1]))
