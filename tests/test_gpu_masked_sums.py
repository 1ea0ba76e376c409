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


def _shift_layer(fg, graph, log_n, f_out, shifts, n_q=3, q_bits=50):
    """A baby-step/giant-step layer whose nodes' neighbours are exactly the given shifts away, uniform masks and inputs,
    and its outputs by the per-operation form."""
    import torch
    ctx = fg.Context(log_n, n_q, q_bits, 1, 60)
    rng = np.random.default_rng(1)
    nbrs = [[] for _ in range(ctx.M)]
    for v, s in zip(rng.integers(0, ctx.M, len(shifts)), shifts):
        nbrs[v].append((v + int(s)) % ctx.M)
    plan = fg.Plan(ctx, *graph.normalize(ctx.M, [np.unique(x).astype(int) for x in nbrs], "mean"), ctx.M, [2, f_out],
                   [rng.normal(0, 0.1, (2, f_out))], first_mode=1, use_noo=False, family=2, t=1)
    d = plan.ficgcn_plan_info()[0]
    _, ev = ctx.ckks_keygen(3, plan.ficgcn_plan_rot_steps(), with_relin=False)
    plan.ficgcn_plan_fill_operands(4)
    x = torch.empty((2, 2, d["level_in"] + 1, ctx.N), dtype=torch.int64, device="cuda")
    for i, q in enumerate(ctx.ckks_ctx_moduli()[: d["level_in"] + 1]):
        x[:, :, i].random_(0, q, generator=torch.Generator(device="cuda").manual_seed(9 + i))
    words = 2 * (d["level_out"] + 1) * ctx.N

    def run(mode):
        outs = [ctx.ct_buffer(d["level_in"]) for _ in range(f_out)]
        plan.ficgcn_gcn_layer(ev, 0, list(x), outs, mode=mode)
        return [o.reshape(-1)[:words] for o in outs]
    return ctx, d, run, run(0)


@pytest.mark.parametrize("case", ["two lists of terms", "a short rest", "more ciphertexts than the table"])
def test_sums_over_several_launches(case):
    """Three ciphertexts: the term list holds 12288 terms and the ciphertext table 128 places a launch.  What is left
    goes to a second launch, or, below 3000 terms, to the sums that read ciphertexts from memory."""
    import torch
    from paper_2506_10399_amd import ficgcn as fg, graph
    rng = np.random.default_rng(7)
    if case == "more ciphertexts than the table":
        # giant steps of 256; the first forty of them share 128 baby steps, the others take any
        log_n, n_shifts, G = 17, 4649, 256   # the identity is not among those drawn
        shifts = np.concatenate([256 * g + (rng.permutation(128)[:100] if 128 <= g < 168 else rng.permutation(256)[:3])
                                 for g in range(256)])
    else:
        log_n, G, n_shifts = 15, 128, 15800 if case == "two lists of terms" else 13000
        shifts = rng.permutation(1 << 14)[:n_shifts]
    ctx, d, run, want = _shift_layer(fg, graph, log_n, 3, shifts)
    assert (d["G"], d["n_shifts"]) == (G, n_shifts)
    ctx.ficgcn_profile_enable(True)
    got = run(1)
    assert ctx.ficgcn_profile_read("bsgs_inner")[1] == 2
    ctx.ficgcn_profile_enable(False)
    for a, b in zip(want, got):
        assert torch.equal(a, b)
