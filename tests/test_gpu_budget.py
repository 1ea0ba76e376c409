"""Masked sums whose sources exceed a launch group's memory: every rotation of an output reads a source of its own
(giant steps), and one output's extended digits take several times the 3 GiB a group may hold.  A served request's
scratch has to stay within what it was admitted with, and the words are those of the per-operation form."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

PARAMS = dict(log_n=16, n_q=17, q_bits=50, n_p=2, p_bits=60, log_scale=40)


def test_giant_steps_beyond_a_chunk_stay_within_the_admitted_scratch():
    import torch
    from paper_2506_10399_amd import ficgcn as fg, graph
    ctx = fg.Context.from_dict(PARAMS)
    n = ctx.M
    rng = np.random.default_rng(1)
    offs = rng.choice(np.arange(1, n), 140, replace=False)   # scattered: the cheapest split is giant steps alone
    csr = graph.normalize(n, [np.unique([(v + offs[v % 140]) % n]) for v in range(n)], "mean")
    plan = fg.Plan(ctx, *csr, n, [2, 5], [rng.normal(0, 0.1, (2, 5))], first_mode=1, use_noo=False, family=2, t=1)
    d = plan.ficgcn_plan_info()[0]
    l1 = d["level_out"] + 2                                  # limbs of the aggregation
    giants = {s // d["G"] for s in plan.ficgcn_plan_shifts(0)} - {0}
    per_source = ((l1 + 1) // 2 * (l1 + 2) + l1) * ctx.N * 8
    assert l1 == 16 and len(giants) * per_source > 3 * (3 << 30)
    _, ev = ctx.ckks_keygen(3, plan.ficgcn_plan_rot_steps(), with_relin=False)
    plan.ficgcn_plan_encode()
    x = torch.empty((2, 2, d["level_in"] + 1, ctx.N), dtype=torch.int64, device="cuda")
    for i, q in enumerate(ctx.ckks_ctx_moduli()[: d["level_in"] + 1]):
        x[:, :, i].random_(0, q, generator=torch.Generator(device="cuda").manual_seed(9 + i))
    outs = [ctx.ct_buffer(d["level_in"]) for _ in range(5)]
    plan.ficgcn_gcn_layer(ev, 0, list(x), outs, mode=0)
    words = 2 * (d["level_out"] + 1) * ctx.N
    want = torch.stack([o.reshape(-1)[:words] for o in outs]).cpu().numpy()
    got = np.zeros((5, words), dtype=np.uint64)
    srv = fg.Server(PARAMS, 1, 1 << 40)
    rid = srv.ficgcn_server_submit(plan, ev, x.cpu(), 2, got, 5)
    srv.ficgcn_server_wait(rid)
    st = srv.ficgcn_server_stats()
    srv.close()
    assert np.array_equal(got, want.view(np.uint64))
    assert st["scratch_overruns"] == 0
