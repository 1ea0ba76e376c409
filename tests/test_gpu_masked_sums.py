"""The batched form's masked sums under shared masks against the per-operation form, word for word, on
layers with enough terms for the sums that hold the ciphertexts in LDS: two and three packed ciphertexts
(which take that form) and the other numbers, primes in and below the fp64 range and above the halves'
50 bits (the other sums)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("f_out,q_bits", [(1, 50), (2, 50), (3, 50), (5, 50), (3, 45), (4, 49), (3, 52)])
def test_baby_step_giant_step_sums_equal_plain_form(f_out, q_bits):
    import torch
    from paper_2506_10399_amd import ficgcn as fg, graph
    ctx = fg.Context(14, 3, q_bits, 1, 60)
    n = 7000
    rng = np.random.default_rng(f_out)
    # two neighbours anywhere and a local one: giant steps of very different lengths, some of one term
    nbrs = [np.unique(np.append(rng.integers(0, n, 2 if v % 3 else 0), (v + 1 + v % 7) % n)) for v in range(n)]
    csr = graph.normalize(n, nbrs, "mean")
    plan = fg.Plan(ctx, *csr, n, [2, f_out], [rng.normal(0, 0.1, (2, f_out))], first_mode=1, use_noo=False, family=2,
                   t=1)
    d = plan.ficgcn_plan_info()[0]
    assert d["n_shifts"] >= 3000
    _, ev = ctx.ckks_keygen(3, plan.ficgcn_plan_rot_steps(), with_relin=False)
    plan.ficgcn_plan_fill_operands(4)
    x = torch.empty((2, 2, d["level_in"] + 1, ctx.N), dtype=torch.int64, device="cuda")
    for i, q in enumerate(ctx.ckks_ctx_moduli()[: d["level_in"] + 1]):
        x[:, :, i].random_(0, q, generator=torch.Generator(device="cuda").manual_seed(9 + i))
    outs = [[ctx.ct_buffer(d["level_in"]) for _ in range(d["n_out_cts"])] for _ in range(2)]
    for mode in range(2):
        plan.ficgcn_gcn_layer(ev, 0, list(x), outs[mode], mode=mode)
    words = 2 * (d["level_out"] + 1) * ctx.N
    for a, b in zip(*outs):
        assert torch.equal(a.reshape(-1)[:words], b.reshape(-1)[:words])
