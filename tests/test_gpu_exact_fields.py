"""The fields of every row's record that rounding does not touch (the maximum, its lowest
index, the -inf flag, the count of logits above the drafted one) compared exactly, over whole
batches whose rows start in every 16-byte phase, with torch on the device as the reference.
(The whole-batch parity tests compare them on the workloads, whose rows are aligned but for
one.)"""
import pytest
import torch

pytestmark = pytest.mark.gpu

CASES = [  # batch, k_max, vocab, dtype, padding of the row stride, share of -inf logits
    (64, 8, 152064, torch.bfloat16, 0, 0.0),
    (64, 8, 50257, torch.bfloat16, 6, 0.0),
    (32, 8, 100003, torch.float32, 2, 0.03),
    (300, 16, 32003, torch.bfloat16, 0, 0.03),
    (400, 12, 16001, torch.float32, 0, 0.0),
    (600, 8, 1003, torch.bfloat16, 0, 0.5),
    (600, 8, 1003, torch.float32, 1, 0.5),
]


def _first(rows, m):
    i = torch.arange(rows.shape[1], device=rows.device, dtype=torch.int32)
    return torch.where(rows == m[:, None], i, torch.full_like(i, rows.shape[1])).amin(1)


def _by_chunks(rows, f):
    step = max(1, (1 << 25) // rows.shape[1])
    parts = [f(slice(r, r + step), rows[r:r + step]) for r in range(0, rows.shape[0], step)]
    return [torch.cat(p) for p in zip(*parts)]


@pytest.mark.parametrize("B,K,V,dtype,pad,masked", CASES)
def test_exact_fields(B, K, V, dtype, pad, masked):
    from paper_2508_15371_amd import cmsd
    dev = torch.device("cuda:0")
    g = torch.Generator(device=dev).manual_seed(V + B)
    beta = 5

    def rows(n):
        x = torch.empty(n, V + pad, dtype=dtype, device=dev)
        step = max(1, (1 << 25) // V)
        for r in range(0, n, step):
            z = 2.0 * torch.randn(min(step, n - r), V + pad, generator=g, device=dev)
            if masked:
                z[torch.rand(z.shape, generator=g, device=dev) < masked] = float("-inf")
                z[:, 0] = 0.0                              # a finite logit in every row
            x[r:r + step] = z
        return x[:, :V]

    draft, target = rows(B * K), rows(B * (K + 1))
    # a drafted token near the target's top, so that counts end on either side of beta
    near, = _by_chunks(target, lambda s, z: (torch.topk(z.float(), 8, 1).indices,))
    top = near.view(B, K + 1, 8)[:, :K].reshape(B * K, 8)
    drafted = top.gather(1, torch.randint(0, 8, (B * K, 1), generator=g, device=dev))[:, 0].int()
    unif = torch.rand(B * (K + 1), generator=g, device=dev)
    m, first, inf = _by_chunks(draft, lambda s, z: (z.amax(1).float(), _first(z, z.amax(1)), torch.isinf(z).any(1).int()))
    y = torch.zeros(B, K + 1, dtype=torch.long, device=dev)
    y[:, :K] = drafted.view(B, K).long()
    y = y.view(-1)
    tm, tfirst, above = _by_chunks(target, lambda s, z: (z.amax(1).float(), _first(z, z.amax(1)),
                                                        (z > z.gather(1, y[s][:, None])).sum(1).int()))
    want = above.clamp(max=beta).view(B, K + 1)
    want[:, K] = -1
    for mode in (cmsd.CMSD_MODE_CM, cmsd.CMSD_MODE_GREEDY):
        o = cmsd.cmsd_logit_pass(draft, target, drafted, unif, batch=B, k_max=K, mode=mode, top_beta=beta)
        off = torch.arange(B + 1, dtype=torch.int32, device=dev) * (K + 1)
        k = torch.full((B,), K, dtype=torch.int32, device=dev)
        st = cmsd.cmsd_confidence(draft)
        ts = cmsd.cmsd_verify(draft, st, target, off, k, drafted, unif, batch=B, k_max=K, mode=mode, top_beta=beta)[2]
        var = cmsd.cmsd_confidence_var(draft)[0]
        torch.cuda.synchronize()
        for s in (o["draft_stats"], st, var):
            assert torch.equal(s[:, 0], m)
            assert torch.equal(s.view(torch.int32)[:, 6], first)
            assert torch.equal(s.view(torch.int32)[:, 7] & 1, inf)
        for t in (o["target_stats"], ts):
            i = t.view(torch.int32)
            assert torch.equal(t[:, 0], tm)
            assert torch.equal(i[:, 2].view(B, K + 1), want)
            if mode == cmsd.CMSD_MODE_GREEDY:
                assert torch.equal(i[:, 4], tfirst)
