"""Packed calls without row counts (dense, or sparse without them) that run with two waves per row issue their rows longest
first, as calls of one length do by themselves.  Results do not depend on the order, and neither does the time on how
sequences of one length are handed over."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sale():
    from paper_2505_24179_amd import sale as mod
    return mod


def _qkv(tokens, q_heads, kv_heads, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    return tuple(torch.randn(1, h, tokens, 128, generator=gen, device="cuda").bfloat16() for h in (q_heads, kv_heads, kv_heads))


# 528 and 1040 rows: just above the 512 that all start at once; 640: one head per KV head, 20 sequences, one of them long
@pytest.mark.parametrize("lengths,q_heads,kv_heads", [((64, 2048, 704, 1408), 8, 2), ((4096, 64, 64, 2432), 10, 5),
                                                      ((64,) * 9 + (6784,) + (2624,) * 10 + (576,), 1, 1)])
@pytest.mark.parametrize("block_k", [64, 32])
def test_packed_rows_longest_first_give_the_bits_of_each_sequence_alone(sale, lengths, q_heads, kv_heads, block_k):
    total = sum(lengths)
    assert 512 < total // 64 * q_heads <= 1152
    q, k, v = _qkv(total, q_heads, kv_heads, total)
    cu = [0]
    for n in lengths:
        cu.append(cu[-1] + n)
    p = sale.Params(1, q_heads, kv_heads, total, block_k=block_k, cu_seqlens=tuple(cu))
    gen = torch.Generator(device="cuda").manual_seed(5)
    mask = torch.randint(-2 ** 62, 2 ** 62, (1, q_heads, p.n_q, p.words), generator=gen, dtype=torch.int64, device="cuda") | 1
    bits = (mask[..., None] >> torch.arange(64, device="cuda")) & 1
    starts = torch.repeat_interleave(torch.tensor(cu[:-1]), torch.tensor(lengths) // 64) // 64
    last = ((torch.arange(p.n_q) - starts + 1) * (64 // block_k) - 1).cuda()      # last visible block of a row
    counts = (bits.flatten(-2) * (torch.arange(64 * p.words, device="cuda") <= last[:, None])).sum(-1).to(torch.int32)
    full = sale.workspace_bytes(p, sale.WS_DENSE_ATTN)
    order = total // 64 * q_heads * 4
    for size in (full, full - order):      # without the order's bytes the rows are issued as they come, one wave each
        ws = torch.empty(size, dtype=torch.uint8, device="cuda")
        o, lse = sale.sparse_attn(p, q, k, v, mask, want_lse=True, out=torch.full_like(q, float("nan")))
        oc, lsec = sale.sparse_attn(p, q, k, v, mask, counts, want_lse=True, out=torch.full_like(q, float("nan")))
        assert torch.equal(oc, o) and torch.equal(lsec, lse)
        od, lsed = sale.dense_attn(p, q, k, v, want_lse=True, out=torch.full_like(q, float("nan")), ws=ws)
        for a, b in zip(cu[:-1], cu[1:]):
            one = sale.Params(1, q_heads, kv_heads, b - a, block_k=block_k)
            qs, ks, vs = (t[:, :, a:b].contiguous() for t in (q, k, v))
            m = mask[:, :, a // 64:b // 64, :one.words].contiguous()
            oa, lsea = sale.sparse_attn(one, qs, ks, vs, m, want_lse=True)
            oda, lseda = sale.dense_attn(one, qs, ks, vs, want_lse=True)
            assert torch.equal(o[:, :, a:b], oa) and torch.equal(lse[:, :, a:b], lsea), (a, b)
            assert torch.equal(od[:, :, a:b], oda) and torch.equal(lsed[:, :, a:b], lseda), (a, b)
    with pytest.raises(sale.SaleError):
        sale.dense_attn(p, q, k, v, ws=torch.empty(full - order - 64, dtype=torch.uint8, device="cuda"))


def test_packing_equal_sequences_takes_no_longer_than_a_batch_of_them(sale):
    """64 sequences of 1024 tokens, one head: packed, the rows of the last sequences came first and the long rows of the
    first ones last, 65 us where the batch took 43.  (Packed calls have one small launch more, for the sequence table.)"""
    n, tokens = 64, 1024
    q, k, v = _qkv(n * tokens, 1, 1, 1)
    packed = sale.Params(1, 1, 1, n * tokens, cu_seqlens=tuple(range(0, (n + 1) * tokens, tokens)))
    batch = sale.Params(n, 1, 1, tokens)
    qb, kb, vb = (t.view(n, 1, tokens, 128) for t in (q, k, v))
    out = torch.empty_like(q)

    def time_of(p, a, b, c, o):
        ws = torch.empty(sale.workspace_bytes(p, sale.WS_DENSE_ATTN), dtype=torch.uint8, device="cuda")
        best = float("inf")
        for _ in range(8):
            t0, t1 = torch.cuda.Event(True), torch.cuda.Event(True)
            t0.record()
            for _ in range(20):
                sale.dense_attn(p, a, b, c, out=o, ws=ws)
            t1.record()
            torch.cuda.synchronize()
            best = min(best, t0.elapsed_time(t1) * 50)
        return best

    time_of(packed, q, k, v, out)
    us = time_of(packed, q, k, v, out), time_of(batch, qb, kb, vb, out.view_as(qb))
    assert us[0] < 1.25 * us[1] + 5, us
