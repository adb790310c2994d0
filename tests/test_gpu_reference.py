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


def _flags(sale, attn):
    return {"bf16": 0, "int8": sale.FLAG_ATTN_INT8_QK, "fp8": sale.FLAG_ATTN_INT8_QK | sale.FLAG_ATTN_FP8_PV}[attn]


@pytest.mark.parametrize("block_k,attn", [(64, "bf16"), (32, "bf16"), (64, "int8"), (32, "int8"), (64, "fp8")])
def test_rows_that_rise_in_the_window_launches(sale, block_k, attn):
    """A row that is parked between windows keeps its maximum: the bits of the one-sweep call."""
    n, heads = 20480, 2
    q, k, v = _inputs(n, heads, 400.0, 6)
    p = sale.Params(1, heads, heads, n, block_k=block_k, flags=_flags(sale, attn))
    mask = torch.full((1, heads, p.n_q, p.words), -1, dtype=torch.int64, device="cuda")
    counts = ((torch.arange(p.n_q, device="cuda") + 1) * (64 // block_k)).int().expand(1, heads, -1).contiguous()
    qd, kd, vd = q.cuda(), k.cuda(), v.cuda()
    o, lse = sale.sparse_attn(p, qd, kd, vd, mask, counts, want_lse=True)      # rows above 192 blocks in windows
    o1, lse1 = sale.sparse_attn(p, qd, kd, vd, mask, None, want_lse=True)      # one sweep per row
    torch.cuda.synchronize()
    assert torch.isfinite(o).all() and torch.equal(o, o1) and torch.equal(lse, lse1)
    if attn != "bf16":      # (8-bit logits of this size are not those of the bf16 operands)
        return
    rows = slice(n - 64, n)
    for h in range(heads):
        s = (q[0, h, rows].double() @ k[0, h].double().T) / math.sqrt(D)
        s.masked_fill_(torch.arange(n)[None, :] > torch.arange(n)[rows][:, None], -math.inf)
        _check(o[0, h, rows].cpu(), lse[0, h, rows].cpu(), torch.softmax(s, -1) @ v[0, h].double(), torch.logsumexp(s, -1), v[0, h])


@pytest.mark.parametrize("rise", [60.0, 400.0])
@pytest.mark.parametrize("block_k", [64, 32])
def test_rows_that_rise_in_packed_calls(sale, block_k, rise):
    """Three sequences packed: the bits of each alone."""
    lengths, heads = (1088, 64, 640), 24
    parts = [_inputs(n, heads, rise, 20 + i) for i, n in enumerate(lengths)]
    offsets = (0, 1088, 1152, 1792)
    p = sale.Params(1, heads, heads, 1792, block_k=block_k, cu_seqlens=offsets)
    q, k, v = (torch.cat([x[i] for x in parts], dim=2).cuda() for i in range(3))
    mask = torch.full((1, heads, p.n_q, p.words), -1, dtype=torch.int64, device="cuda")
    calls = sale.sparse_attn(p, q, k, v, mask, want_lse=True), sale.dense_attn(p, q, k, v, want_lse=True)
    for (qs, ks, vs), n, t in zip(parts, lengths, offsets):
        ps = sale.Params(1, heads, heads, n, block_k=block_k)
        o, lse = sale.dense_attn(ps, qs.cuda(), ks.cuda(), vs.cuda(), want_lse=True)
        assert torch.isfinite(o).all()
        for od, lsed in calls:
            assert torch.equal(od[:, :, t:t + n], o) and torch.equal(lsed[:, :, t:t + n], lse)


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
@pytest.mark.parametrize("n,heads", [(640, 2), (1088, 96)])      # two waves per row; one
def test_rows_that_rise_with_the_8_bit_first_product(sale, n, heads, rise):
    q, k, v = _inputs(n, heads, rise, 7)
    p = sale.Params(1, heads, heads, n, flags=sale.FLAG_ATTN_INT8_QK)
    qd, kd, vd = q.cuda(), k.cuda(), v.cuda()
    q8, k8, qs, ks, mean = sale.attn_int8_operands(p, qd, kd)
    calls = [sale.dense_attn(p, qd, kd, vd, want_lse=True)]
    for block_k in (64, 32):      # (everything kept)
        ps = sale.Params(1, heads, heads, n, block_k=block_k, flags=sale.FLAG_ATTN_INT8_QK)
        mask = torch.full((1, heads, ps.n_q, ps.words), -1, dtype=torch.int64, device="cuda")
        calls.append(sale.sparse_attn(ps, qd, kd, vd, mask, want_lse=True))
    torch.cuda.synchronize()
    for h in range(heads) if heads <= 4 else (0, 1, heads - 1):
        qh = q8[0, h].cpu().double() * qs[0, h].cpu().double().repeat_interleave(64)[:, None]
        kh = k8[0, h].cpu().double() * ks[0, h].cpu().double().repeat_interleave(64)[:, None]
        s = qh @ kh.T / math.sqrt(D)
        s.masked_fill_(torch.triu(torch.ones(n, n, dtype=torch.bool), 1), -math.inf)
        shift = q[0, h].double() @ mean[0, h].cpu().double() / math.sqrt(D)
        want, ref = torch.softmax(s, -1) @ v[0, h].double(), torch.logsumexp(s, -1)
        # (the accumulators' offset of 1.5 * 2^23 leaves with the scaling FMA: two roundings at its size in logits)
        off = 1.5 * (qs[0, h].max() * ks[0, h].max()).item() / math.sqrt(D) * 1.4427
        for o, lse in calls:
            assert (o[0, h].cpu().double() - want).abs().max() <= (2.0 ** -7 + off) * v[0, h].abs().max()
            got = lse[0, h].cpu().double() - shift
            assert ((got - ref).abs() <= 4e-3 + off + 2.0 ** -18 * (ref.abs() + shift.abs())).all()


def _with(value, q, k):
    q, k = q.clone(), k.clone()
    q[0, 0, 70, 5] = value
    k[0, 1, 300, 9] = value
    return q, k


@pytest.mark.parametrize("value", [float("nan"), float("inf")])
@pytest.mark.parametrize("n,heads", [(640, 2), (1088, 96)])      # two waves per row; one
@pytest.mark.parametrize("block_k,attn", [(64, "bf16"), (32, "bf16"), (64, "int8"), (32, "int8"), (64, "fp8")])
def test_nan_and_infinity_stay_with_their_queries(sale, value, n, heads, block_k, attn):
    """Rows of other queries are the bits they are without the value.  (8-bit operands: an infinity is the scale of its 64
    queries, and the mean key takes what a key holds to its whole head.)"""
    q, k, v = _inputs(n, heads, 0.0, 7)
    qv, kv = _with(value, q, k)
    p = sale.Params(1, heads, heads, n, block_k=block_k, flags=_flags(sale, attn))
    mask = torch.full((1, heads, p.n_q, p.words), -1, dtype=torch.int64, device="cuda")
    other = torch.ones(1, heads, n, dtype=torch.bool)
    if attn == "bf16":
        other[0, 0, 70] = False
        other[0, 1, 300:] = False
    else:
        other[0, 0, 70 if math.isnan(value) else slice(64, 128)] = False
        other[0, 1] = False
    for call in (sale.dense_attn, lambda *x, **y: sale.sparse_attn(*x, mask, **y)):
        want, want_lse = call(p, q.cuda(), k.cuda(), v.cuda(), want_lse=True)
        o, lse = call(p, qv.cuda(), kv.cuda(), v.cuda(), want_lse=True)
        assert torch.isfinite(want).all()
        assert torch.equal(o.cpu()[other], want.cpu()[other]) and torch.equal(lse.cpu()[other], want_lse.cpu()[other])


@pytest.mark.parametrize("value", [float("nan"), float("inf")])
@pytest.mark.parametrize("block_k", [64, 32])
def test_nan_and_infinity_in_the_window_launches(sale, value, block_k):
    n, heads = 20480, 2
    q, k, v = _inputs(n, heads, 0.0, 7)
    qv, kv = _with(value, q, k)
    qv[0, 0, n - 20, 5] = value      # (a row that is parked)
    kv[0, 1, 300, 9] = k[0, 1, 300, 9]
    kv[0, 1, 17000, 9] = value      # (in the last window)
    p = sale.Params(1, heads, heads, n, block_k=block_k)
    mask = torch.full((1, heads, p.n_q, p.words), -1, dtype=torch.int64, device="cuda")
    counts = ((torch.arange(p.n_q, device="cuda") + 1) * (64 // block_k)).int().expand(1, heads, -1).contiguous()
    want, want_lse = sale.sparse_attn(p, q.cuda(), k.cuda(), v.cuda(), mask, counts, want_lse=True)
    o, lse = sale.sparse_attn(p, qv.cuda(), kv.cuda(), v.cuda(), mask, counts, want_lse=True)
    other = torch.ones(1, heads, n, dtype=torch.bool)
    other[0, 0, 70] = other[0, 0, n - 20] = False
    other[0, 1, 17000:] = False
    assert torch.equal(o.cpu()[other], want.cpu()[other]) and torch.equal(lse.cpu()[other], want_lse.cpu()[other])


def test_values_near_the_largest(sale):
    """One V near the largest float: the probabilities are at most 1, so that their products with it stay finite.  (The sum of
    several such products need not: O is divided by the sum of the probabilities at the end.)  Rounded: the probability, O and
    the sum of the probabilities, 2^-9 each."""
    n, heads = 640, 2
    q, k, v = _inputs(n, heads, 0.0, 8)
    v[0, :, 70] = 3.0e38
    p = sale.Params(1, heads, heads, n)
    o, _ = sale.dense_attn(p, q.cuda(), k.cuda(), v.cuda())
    for h in range(heads):
        want, _ = _attend(q[0, h:h + 1], k[0, h:h + 1], v[0, h:h + 1], torch.ones(n, n, dtype=torch.bool))
        got = o[0, h, 70:].cpu().double()
        assert torch.isfinite(o[0, h]).all() and ((got - want[0, 70:]).abs() <= 2.0 ** -7 * want[0, 70:].abs()).all()
