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


@pytest.mark.parametrize("family,f_out,n_q,n_p,q_bits,p_bits", [
    (4, 5, 4, 2, 50, 60),      # one output a wave
    (4, 30, 4, 1, 50, 60),     # two outputs a wave, an odd number of waves at work
    (4, 25, 9, 1, 50, 60),     # eight digits, rotations in several launches
    (4, 24, 4, 2, 45, 50),     # primes below the fp64 range
    (4, 7, 4, 2, 52, 61),      # 128-bit sums on every limb
    (2, 6, 4, 2, 50, 60),      # giant steps: a source of its own for every rotation
])
def test_rotations_and_masks_shared_by_many_outputs(family, f_out, n_q, n_p, q_bits, p_bits):
    import torch
    from paper_2506_10399_amd import ficgcn as fg, graph
    ctx = fg.Context(11, n_q, q_bits, n_p, p_bits)
    n = 300
    rng = np.random.default_rng(f_out)
    nbrs = [np.unique([(v + 1) % n, (v + 3) % n, (v + 17) % n, (v * 7) % 40 if v % 5 == 0 else v]) for v in range(n)]
    plan = fg.Plan(ctx, *graph.normalize(n, nbrs, "mean"), n, [2, f_out], [rng.normal(0, 0.1, (2, f_out))], first_mode=1,
                   use_noo=False, family=family, t=1)
    d = plan.ficgcn_plan_info()[0]
    _, ev = ctx.ckks_keygen(3, plan.ficgcn_plan_rot_steps(), with_relin=False)
    plan.ficgcn_plan_fill_operands(4)
    x = torch.empty((2, 2, d["level_in"] + 1, ctx.N), dtype=torch.int64, device="cuda")
    for i, q in enumerate(ctx.ckks_ctx_moduli()[: d["level_in"] + 1]):
        x[:, :, i].random_(0, q, generator=torch.Generator(device="cuda").manual_seed(9 + i))
    outs = [[ctx.ct_buffer(d["level_in"]) for _ in range(d["n_out_cts"])] for _ in range(3)]
    for mode in range(3):
        plan.ficgcn_gcn_layer(ev, 0, list(x), outs[mode], mode=mode)
    words = 2 * (d["level_out"] + 1) * ctx.N
    for a, b, c in zip(*outs):
        assert torch.equal(a.reshape(-1)[:words], b.reshape(-1)[:words])
        assert torch.equal(a.reshape(-1)[:words], c.reshape(-1)[:words])


# on both sides of the lines between the list's products made once for all outputs and made for each
@pytest.mark.parametrize("log_n,family,f_out,n_q,n_p,q_bits", [
    (13, 4, 11, 8, 2, 50),     # eleven outputs
    (13, 4, 12, 8, 2, 50),     # twelve: shared
    (12, 4, 5, 8, 2, 50),      # five, the products of seven limbs in 2304 rounds: shared
    (12, 4, 5, 9, 2, 50),      # of eight limbs in 2560
    (13, 2, 12, 8, 2, 50),     # a source for each rotation
    (12, 2, 12, 8, 2, 50),     # in a ring of 2^12: shared
    (12, 4, 6, 9, 2, 52),      # 128-bit sums output by output
    (11, 4, 6, 7, 3, 50),      # three special primes
])
def test_lines_between_shared_and_separate_products(log_n, family, f_out, n_q, n_p, q_bits):
    import torch
    from paper_2506_10399_amd import ficgcn as fg, graph
    ctx = fg.Context(log_n, n_q, q_bits, n_p, 60)
    n = 300
    rng = np.random.default_rng(f_out)
    nbrs = [np.unique([(v + 1) % n, (v + 3) % n, (v + 17) % n, (v * 7) % 40 if v % 5 == 0 else v]) for v in range(n)]
    plan = fg.Plan(ctx, *graph.normalize(n, nbrs, "mean"), n, [2, f_out], [rng.normal(0, 0.1, (2, f_out))], first_mode=1,
                   use_noo=False, family=family, t=1)
    d = plan.ficgcn_plan_info()[0]
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
