"""The reference of a row's exponents in the attention kernels (bf16 and 8-bit first product): the running maximum of its
kept keys.  Rows whose scores rise far above those of their first kept half-tile, against 64-bit attention over the same
operands; rows that take no part in their last window; and the largest probability, which is 1 and is not rounded.

Tolerance: the probabilities and the output are rounded to bf16 (2^-9 of the largest |v| each), the logits carry the rounding
of fp32 sums and of the scaling FMA, up to 2^-20 of 1000 in the exponent; together below 2^-7 of the largest |v|.
"""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu

D = 128


@pytest.fixture(scope="module")
def sale():
    from paper_2505_24179_amd import sale as s
    return s


def _inputs(n, heads, rise, seed):
    """Query r and key t have a common component whose size grows from the first keys to the last by `rise` (natural
    logarithm) in total for half of the heads, and falls for the others."""
    g = torch.Generator().manual_seed(seed)
    q = torch.randn(1, heads, n, D, generator=g)
    k = torch.randn(1, heads, n, D, generator=g)
    v = torch.randn(1, heads, n, D, generator=g)
    ramp = torch.linspace(-0.5, 0.5, n)[None, :] * torch.where(torch.arange(heads) % 2 == 0, 1.0, -1.0)[:, None]
    q[..., 0] = 16.0
    k[..., 0] = ramp * rise * math.sqrt(D) / 16.0
    return q.bfloat16(), k.bfloat16(), v.bfloat16()


def _attend(q, k, v, keep):
    n = q.shape[-2]
    s = (q.double() @ k.double().transpose(1, 2)) / math.sqrt(D)
    hide = torch.triu(torch.ones(n, n, dtype=torch.bool), 1) | ~keep
    s.masked_fill_(hide, -math.inf)
    return torch.softmax(s, -1) @ v.double(), torch.logsumexp(s, -1)


def _check(o, lse, ref, ref_lse, v):
    seen = torch.isfinite(ref_lse)
    err = (o.double() - ref).abs()[seen]
    assert err.max() <= 2.0 ** -7 * v.abs().max(), err.max()
    # (lse of sums of bf16-rounded probabilities: 2^-8; fp32 at the size of the logits)
    lim = 4e-3 + 2.0 ** -21 * ref_lse[seen].abs()
    assert ((lse.double() - ref_lse).abs()[seen] <= lim).all()


@pytest.mark.parametrize("rise", [60.0, 160.0, 2000.0])      # beyond fp32 from about 88 on, if nothing were rescaled
@pytest.mark.parametrize("block_k", [64, 32])
@pytest.mark.parametrize("n,heads", [(640, 2), (64, 2), (1088, 96)])      # two waves per row; one block; one wave per row
def test_rows_that_rise_above_their_first_keys(sale, rise, block_k, n, heads):
    q, k, v = _inputs(n, heads, rise, 5)
    p = sale.Params(1, heads, heads, n, block_k=block_k)
    n_q, n_k, f = n // 64, n // block_k, 64 // block_k
    g = torch.Generator().manual_seed(9)
    bits = torch.rand(heads, n_q, n_k, generator=g) < 0.4
    bits[:, torch.arange(n_q), torch.arange(n_q) * f] = True      # (every query sees a key of its own diagonal block)
    words = torch.zeros(heads, n_q, p.words, dtype=torch.int64)
    for j in range(n_k):
        words[:, :, j // 64] |= torch.where(bits[:, :, j], torch.tensor(1, dtype=torch.int64) << (j % 64), 0)
    qd, kd, vd = q.cuda(), k.cuda(), v.cuda()
    o, lse = sale.sparse_attn(p, qd, kd, vd, words.cuda()[None], want_lse=True)
    od, lsed = sale.dense_attn(p, qd, kd, vd, want_lse=True)
    torch.cuda.synchronize()
    some = range(heads) if heads <= 4 else (0, 1, heads - 1)
    for h in some:
        keep = bits[h].repeat_interleave(64, 0).repeat_interleave(block_k, 1)
        _check(o[0, h].cpu(), lse[0, h].cpu(), *(x[0] for x in _attend(q[0, h:h + 1], k[0, h:h + 1], v[0, h:h + 1], keep)), v[0, h])
        _check(od[0, h].cpu(), lsed[0, h].cpu(),
               *(x[0] for x in _attend(q[0, h:h + 1], k[0, h:h + 1], v[0, h:h + 1], torch.ones_like(keep))), v[0, h])


def test_rows_that_rise_in_the_window_launches(sale):
    """A row that is parked between windows keeps its maximum: the bits of the one-sweep call."""
    n, heads = 20480, 2
    q, k, v = _inputs(n, heads, 400.0, 6)
    p = sale.Params(1, heads, heads, n)
    mask = torch.full((1, heads, p.n_q, p.words), -1, dtype=torch.int64, device="cuda")
    counts = (torch.arange(p.n_q, dtype=torch.int32, device="cuda") + 1).expand(1, heads, -1).contiguous()
    qd, kd, vd = q.cuda(), k.cuda(), v.cuda()
    o, lse = sale.sparse_attn(p, qd, kd, vd, mask, counts, want_lse=True)      # rows above 192 blocks in windows
    o1, lse1 = sale.sparse_attn(p, qd, kd, vd, mask, None, want_lse=True)      # one sweep per row
    torch.cuda.synchronize()
    assert torch.isfinite(o).all() and torch.equal(o, o1) and torch.equal(lse, lse1)
    rows = slice(n - 64, n)
    for h in range(heads):
        s = (q[0, h, rows].double() @ k[0, h].double().T) / math.sqrt(D)
        s.masked_fill_(torch.arange(n)[None, :] > torch.arange(n)[rows][:, None], -math.inf)
        _check(o[0, h, rows].cpu(), lse[0, h, rows].cpu(), torch.softmax(s, -1) @ v[0, h].double(), torch.logsumexp(s, -1), v[0, h])


@pytest.mark.parametrize("block_k,int8", [(64, False), (32, False), (64, True), (32, True)])
def test_rows_that_keep_nothing_in_their_last_window(sale, block_k, int8):
    """A row that rises in its parked windows and has no key in the last one: what was parked goes out as it is."""
    n, heads, clear_from = 20480, 2, 16384
    q, k, v = _inputs(n, heads, 400.0, 6)
    p = sale.Params(1, heads, heads, n, block_k=block_k, flags=sale.FLAG_ATTN_INT8_QK if int8 else 0)
    mask = torch.full((1, heads, p.n_q, p.words), -1, dtype=torch.int64, device="cuda")
    mask[..., clear_from // block_k // 64:] = 0
    counts = (torch.arange(1, p.n_q + 1, device="cuda").clamp(max=clear_from // 64) * (64 // block_k)).int()
    counts = counts.expand(1, heads, -1).contiguous()
    qd, kd, vd = q.cuda(), k.cuda(), v.cuda()
    o, lse = sale.sparse_attn(p, qd, kd, vd, mask, counts, want_lse=True)      # rows above 192 blocks in windows
    o1, lse1 = sale.sparse_attn(p, qd, kd, vd, mask, None, want_lse=True)      # one sweep per row
    torch.cuda.synchronize()
    assert torch.isfinite(o).all() and torch.isfinite(lse).all()
    assert torch.equal(o, o1) and torch.equal(lse, lse1)
    if not int8:      # (8-bit logits of this size are not those of the bf16 operands)
        rows = slice(n - 64, n)
        for h in range(heads):
            s = (q[0, h, rows].double() @ k[0, h, :clear_from].double().T) / math.sqrt(D)
            _check(o[0, h, rows].cpu(), lse[0, h, rows].cpu(), torch.softmax(s, -1) @ v[0, h, :clear_from].double(),
                   torch.logsumexp(s, -1), v[0, h])


@pytest.mark.parametrize("block_k", [64, 32])
@pytest.mark.parametrize("n,heads", [(640, 2), (1088, 96), (20480, 2)])      # two waves per row; one; windows
def test_the_largest_probability_is_exact(sale, block_k, n, heads):
    """Rows dominated by one late key: the log-sum-exp is its logit, to the rounding of fp32 (2^-20 of a logit of up to 32).
    A largest probability that is rounded to bf16 is off by up to 2^-8."""
    g = torch.Generator().manual_seed(11)
    q, k, v = (torch.randn(1, heads, n, D, generator=g) for _ in range(3))
    at = n - n // 8
    q[..., 0] = 16.0
    k[..., 0] = 0.0
    k[:, :, at, 0] = 20.0
    q, k, v = q.bfloat16(), k.bfloat16(), v.bfloat16()
    p = sale.Params(1, heads, heads, n, block_k=block_k)
    mask = torch.full((1, heads, p.n_q, p.words), -1, dtype=torch.int64, device="cuda")
    counts = ((torch.arange(p.n_q, device="cuda") + 1) * (64 // block_k)).int().expand(1, heads, -1).contiguous()
    o, lse = sale.sparse_attn(p, q.cuda(), k.cuda(), v.cuda(), mask, counts, want_lse=True)
    od, lsed = sale.dense_attn(p, q.cuda(), k.cuda(), v.cuda(), want_lse=True)
    for h in (0, heads - 1):
        s = q[0, h, at:].double() @ k[0, h].double().T / math.sqrt(D)
        s.masked_fill_(torch.arange(n)[None, :] > torch.arange(at, n)[:, None], -math.inf)
        want = torch.logsumexp(s, -1)
        assert (s[:, at] - want).min() > -1e-5 and want.max() < 32
        for got in (lse, lsed):
            assert (got[0, h, at:].cpu().double() - want).abs().max() <= 2.0 ** -15
        for got in (o, od):
            err = (got[0, h, at:].cpu().double() - torch.softmax(s, -1) @ v[0, h].double()).abs()
            assert err.max() <= 2.0 ** -8 * v[0, h].abs().max()


@pytest.mark.parametrize("rise", [60.0, 400.0])
def test_rows_that_rise_with_the_8_bit_first_product(sale, rise):
    n, heads = 640, 2
    q, k, v = _inputs(n, heads, rise, 7)
    p = sale.Params(1, heads, heads, n, flags=sale.FLAG_ATTN_INT8_QK)
    qd, kd, vd = q.cuda(), k.cuda(), v.cuda()
    q8, k8, qs, ks, mean = sale.attn_int8_operands(p, qd, kd)
    o, lse = sale.dense_attn(p, qd, kd, vd, want_lse=True)
    torch.cuda.synchronize()
    for h in range(heads):
        qh = q8[0, h].cpu().double() * qs[0, h].cpu().double().repeat_interleave(64)[:, None]
        kh = k8[0, h].cpu().double() * ks[0, h].cpu().double().repeat_interleave(64)[:, None]
        s = qh @ kh.T / math.sqrt(D)
        s.masked_fill_(torch.triu(torch.ones(n, n, dtype=torch.bool), 1), -math.inf)
        shift = q[0, h].double() @ mean[0, h].cpu().double() / math.sqrt(D)
        err = (o[0, h].cpu().double() - torch.softmax(s, -1) @ v[0, h].double()).abs()
        # (the accumulators' offset of 1.5 * 2^23 leaves with the scaling FMA: two roundings at its size in logits)
        off = 1.5 * (qs[0, h].max() * ks[0, h].max()).item() / math.sqrt(D) * 1.4427
        assert err.max() <= (2.0 ** -7 + off) * v[0, h].abs().max()
        got = lse[0, h].cpu().double() - shift
        ref = torch.logsumexp(s, -1)
        assert ((got - ref).abs() <= 4e-3 + off + 2.0 ** -18 * (ref.abs() + shift.abs())).all()


@pytest.mark.parametrize("value", [float("nan"), float("inf")])
@pytest.mark.parametrize("n,heads", [(640, 2), (1088, 96)])      # two waves per row; one
def test_nan_and_infinity_stay_with_their_queries(sale, value, n, heads):
    """Rows of other queries are the bits they are without the value."""
    q, k, v = _inputs(n, heads, 0.0, 7)
    p = sale.Params(1, heads, heads, n)
    want, want_lse = sale.dense_attn(p, q.cuda(), k.cuda(), v.cuda(), want_lse=True)
    q[0, 0, 70, 5] = value
    k[0, 1, 300, 9] = value
    o, lse = sale.dense_attn(p, q.cuda(), k.cuda(), v.cuda(), want_lse=True)
    other = torch.ones(1, heads, n, dtype=torch.bool)
    other[0, 0, 70] = False
    other[0, 1, 300:] = False
    assert torch.equal(o.cpu()[other], want.cpu()[other]) and torch.equal(lse.cpu()[other], want_lse.cpu()[other])


def test_values_near_the_largest(sale):
    """A sum of probabilities above 1 times V near the largest float is not within reach: the mean of V, not infinity."""
    n, heads = 640, 2
    q, k, v = _inputs(n, heads, 0.0, 8)
    v[0, :, 70] = 3.0e38
    p = sale.Params(1, heads, heads, n)
    o, _ = sale.dense_attn(p, q.cuda(), k.cuda(), v.cuda())
    assert torch.isfinite(o).all()
