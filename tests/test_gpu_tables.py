"""Tables on their way to the device: many small calls (the staging ring's laps) and one that takes large tables."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,calls", [
    (40, 900),      # about 4 KB a call: several laps of 2 MB
    (3400, 6),      # just below and above a quarter megabyte of jobs alone: a third of a lap, or past the ring
    (5200, 3),
])
def test_rotations_through_many_and_large_tables(n, calls):
    import torch
    from paper_2506_10399_amd import ficgcn as fg
    ctx = fg.Context(9, 1, 50, 1, 60)
    steps = [1, 5, -3]
    _, ev = ctx.ckks_keygen(3, steps, with_relin=False)
    gen = torch.Generator(device="cuda").manual_seed(4)
    q = ctx.ckks_ctx_moduli()[0]
    cts = torch.empty((7, 2, 1, ctx.N), dtype=torch.int64, device="cuda").random_(0, q, generator=gen)
    want = torch.stack([torch.stack([o.clone() for o in ctx.ckks_rotate_hoisted(ev, c, 0, steps)]) for c in cts])
    out = torch.empty((2, n) + want.shape[2:], dtype=torch.int64, device="cuda")
    rng = np.random.default_rng(n)
    for k in range(calls):
        i, j = rng.integers(0, 7, n), rng.integers(0, 3, n)
        ctx.ckks_rotate_batch(ev, [cts[x] for x in i], 0, [steps[x] for x in j], list(out[k % 2]))
        ix = torch.as_tensor(i, device="cuda"), torch.as_tensor(j, device="cuda")
        assert torch.equal(out[k % 2], want[ix[0], ix[1]]), (n, k)


@pytest.mark.parametrize("n,calls", [(1000, 40), (2250, 30)])   # 116 and 259 KB a call: the largest that take the ring
def test_rotations_through_ring_sized_tables(n, calls):
    test_rotations_through_many_and_large_tables(n, calls)


def test_a_lap_of_the_ring_waits_for_the_stream():
    """One layer uploads tables of 200 and 90 KB (its 40 ciphertexts' baby steps) and ten of 250 KB (their sums, four
    ciphertexts at a time) with no wait between them, more than the ring holds, while the stream is still at work on
    what was queued before: the first table's words must not go before the device took them."""
    import torch
    from paper_2506_10399_amd import ficgcn as fg, graph
    from test_gpu_masked_sums import _shift_layer
    rng = np.random.default_rng(3)
    ctx, d, run, want = _shift_layer(fg, graph, 14, 40, rng.permutation(1 << 13)[:6200], n_q=4)
    assert (d["G"], d["n_shifts"], d["level_out"]) == (64, 6200, 1)
    run(1)                                     # scratch grown: the next call waits for nothing else
    a = torch.ones((8192, 8192), device="cuda")
    b = torch.empty_like(a)
    torch.mm(a, a, out=b)
    torch.cuda.synchronize()
    for _ in range(10):                        # about 100 ms
        torch.mm(a, a, out=b)
    for g, w in zip(run(1), want):
        assert torch.equal(g, w)
