"""Calls of few rows split them over more waves than calls of many rows do.  The rule goes by the whole call, so the same
sequence alone and repeated along the batch takes different splits, and its results must not differ by a bit (the
element-by-element comparison of the single calls with the oracle is in the parity tests)."""
import pytest
import torch

from paper_2505_24179_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sale():
    from paper_2505_24179_amd import sale as mod
    return mod


def _qkv(tokens, q_heads, kv_heads):
    w = inputs.scaled(inputs.LLAMA_32K, tokens, q_heads, kv_heads, f"small-{tokens}-{q_heads}")
    return w, [t.unsqueeze(0).cuda() for t in inputs.make_inputs(w)]


def _blocks_per_wave(p):
    """Key blocks of a row that one wave scores (0: the whole row): the cut of the library."""
    group = p.n_q_heads // p.n_kv_heads
    long = p.words >= 8 and p.batch * p.n_q_heads * p.n_q * p.words >= 40960
    heads = 4 if p.block_k == 64 and group % 4 == 0 and long else 2 if group % 2 == 0 else 1
    waves, blocks, chunk = p.n_q * (p.n_q_heads // heads) * p.batch, p.words * 64, 8
    while chunk * 16384 < blocks * waves:
        chunk *= 2
    return chunk if chunk < blocks else 0


# Every batch takes another cut than the single call (asserted).  In 64-key blocks: 65 blocks, 16 / 4 heads: 8, 16, 32, 64, whole
# rows, 32 / 8 heads: from 16 on; 198 blocks: 64, 128, whole rows.  6 / 2 heads: one head per wave; otherwise two.
@pytest.mark.parametrize("tokens,q_heads,kv_heads,batches", [(4160, 32, 8, (2, 4, 8, 16)), (4160, 16, 4, (2, 4, 8, 16)), (12672, 32, 8, (2, 4, 8)),
                                                             (4160, 6, 2, (4, 11, 22)), (4160, 4, 2, (33, 64)), (64, 4, 1, (2400,))])
@pytest.mark.parametrize("block_k,segments", [(64, False), (32, True)])
def test_selection_does_not_depend_on_how_rows_are_cut(sale, tokens, q_heads, kv_heads, batches, block_k, segments):
    w, (q, k, _) = _qkv(tokens, q_heads, kv_heads)
    tau = torch.tensor([w.tau], dtype=torch.float32, device="cuda")
    flags = sale.FLAG_SEGMENT_LOCAL if segments else 0

    def choose(n):
        p = sale.Params(n, q_heads, kv_heads, tokens, block_k=block_k, flags=flags)
        qn, kn = q.expand(n, -1, -1, -1).contiguous(), k.expand(n, -1, -1, -1).contiguous()
        codes = sale.quantize_qk(p, qn, kn)
        out = (torch.full((n, q_heads, p.n_q, p.words), -1, dtype=torch.int64, device="cuda"),
               torch.full((n, q_heads, p.n_q), -1, dtype=torch.int32, device="cuda"))
        mask, counts, _, _ = sale.select(p, qn, kn, *codes, tau, out=out)
        return mask, counts, _blocks_per_wave(p)

    mask, counts, alone = choose(1)
    for n in batches:
        mask_n, counts_n, cut = choose(n)
        assert cut != alone, (n, cut)
        assert torch.equal(mask_n, mask.expand_as(mask_n)) and torch.equal(counts_n, counts.expand_as(counts_n)), n


# Four heads per wave: the masks of the same heads one by one (one per wave).  833 blocks, 14 words, rows whole and cut; packed: a
# sequence of 577 blocks among short ones.
@pytest.mark.parametrize("tokens,q_heads,kv_heads,offsets", [(53312, 4, 1, ()), (36928, 16, 2, ()),
                                                             (65536, 4, 1, (0, 64, 36992, 36992 + 1024, 65536))])
def test_selection_does_not_depend_on_heads_per_wave(sale, tokens, q_heads, kv_heads, offsets):
    gen = torch.Generator(device="cuda").manual_seed(tokens)
    q, k = (torch.randn(1, h, tokens, 128, generator=gen, device="cuda") for h in (q_heads, kv_heads))
    q += 0.5 * k.repeat_interleave(q_heads // kv_heads, 1)      # (a query's own key is its largest: few other blocks are kept)
    q, k, tau = q.bfloat16(), k.bfloat16(), torch.tensor([0.1], device="cuda")

    def choose(qs, ks):
        p = sale.Params(1, qs.shape[1], ks.shape[1], tokens, cu_seqlens=offsets)
        return p, *sale.select(p, qs, ks, *sale.quantize_qk(p, qs, ks), tau)[:2]

    p, mask, counts = choose(q, k)
    assert p.words >= 8 and q_heads * p.n_q * p.words >= 40960      # (four heads)
    assert 0.05 < counts.float().mean() / (p.n_q / 2) < 0.95      # (some of the blocks that they see)
    for h in range(q_heads):
        kv = h * kv_heads // q_heads
        _, alone, alone_counts = choose(q[:, h:h + 1].contiguous(), k[:, kv:kv + 1].contiguous())
        assert torch.equal(mask[:, h:h + 1], alone) and torch.equal(counts[:, h:h + 1], alone_counts)


# 1024 tokens, 8 / 2 heads: 128 rows alone (two waves per row), 2176 rows seventeen times (one).  704 tokens: an odd
# number of blocks, one head per KV head; 64: nothing but the diagonal block.
@pytest.mark.parametrize("attn", ["bf16", "int8", "fp8"])
@pytest.mark.parametrize("block_k", [64, 32])
@pytest.mark.parametrize("tokens,q_heads,kv_heads,n", [(1024, 8, 2, 17), (704, 3, 3, 64), (64, 4, 1, 600)])
def test_attention_does_not_depend_on_waves_per_row(sale, attn, block_k, tokens, q_heads, kv_heads, n):
    if attn == "fp8" and block_k == 32:
        pytest.skip("the FP8 second product takes 64-key blocks only")
    _, (q, k, v) = _qkv(tokens, q_heads, kv_heads)
    flags = {"bf16": 0, "int8": sale.FLAG_ATTN_INT8_QK, "fp8": sale.FLAG_ATTN_INT8_QK | sale.FLAG_ATTN_FP8_PV}[attn]
    gen = torch.Generator(device="cuda").manual_seed(tokens + block_k)
    p1 = sale.Params(1, q_heads, kv_heads, tokens, block_k=block_k, flags=flags)
    # random masks: odd counts, rows that keep only early blocks
    mask = torch.randint(-2 ** 62, 2 ** 62, (1, q_heads, p1.n_q, p1.words), generator=gen, dtype=torch.int64, device="cuda") | 1
    bits = (mask[..., None] >> torch.arange(64, device="cuda")) & 1
    last = (torch.arange(p1.n_q, device="cuda") + 1) * (64 // block_k) - 1      # last visible block of a row
    counts = (bits.flatten(-2) * (torch.arange(64 * p1.words, device="cuda") <= last[:, None])).sum(-1).to(torch.int32)

    def attend(m):
        p = sale.Params(m, q_heads, kv_heads, tokens, block_k=block_k, flags=flags)
        qm, km, vm = (t.expand(m, -1, -1, -1).contiguous() for t in (q, k, v))
        out = [torch.full_like(qm, float("nan")) for _ in range(3)]
        masks = mask.expand(m, -1, -1, -1).contiguous()
        o, lse = sale.sparse_attn(p, qm, km, vm, masks, want_lse=True, out=out[0])
        # with counts the rows are sorted: another order of the same work
        oc, lsec = sale.sparse_attn(p, qm, km, vm, masks, counts.expand(m, -1, -1).contiguous(), want_lse=True, out=out[2])
        assert torch.equal(oc, o) and torch.equal(lsec, lse)
        od, lsed = sale.dense_attn(p, qm, km, vm, want_lse=True, out=out[1])
        return o, lse, od, lsed

    for alone, many in zip(attend(1), attend(n)):
        assert torch.isfinite(alone.float()).all() and torch.equal(many, alone.expand_as(many))
