"""Sparse calls whose shorter rows are issued from queues (one per KV head; row counts, one wave per row, no window launches)
give the bits of the same call issued by position (without row counts): a row's arithmetic does not depend on when and where
it runs, and every row runs once.  Heads keep very different numbers of blocks, so that rows move between the XCDs.
"""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sale():
    from paper_2505_24179_amd import sale as s
    return s


@pytest.mark.parametrize("n,batch,q_heads,kv_heads,block_k,attn,offsets", [
    (2112, 1, 64, 2, 64, "fp8", ()),           # shortest rows, many rows per head, fewer KV heads than XCDs
    (2112, 3, 36, 18, 64, "fp8", ()),          # more KV heads than XCDs, not a multiple of them
    (10240, 1, 26, 13, 64, "bf16", ()),        # 16-bit operands: the shortest rows that are issued so
    (10240, 1, 26, 13, 64, "int8", ()),        # 8-bit first product: the same
    (16384, 1, 16, 4, 32, "bf16", ()),         # 32-key blocks
    (16384, 1, 16, 4, 32, "int8", ()),
    (12352, 1, 32, 8, 64, "bf16", (0, 64, 10304, 11328, 12352)),      # packed (bf16 only): the queues hold rows of all sequences
    (18496, 1, 32, 8, 32, "bf16", (0, 16384, 16448, 18496)),
])
def test_rows_from_queues_are_those_issued_by_position(sale, n, batch, q_heads, kv_heads, block_k, attn, offsets):
    g = torch.Generator(device="cuda").manual_seed(3)
    flags = {"bf16": 0, "int8": sale.FLAG_ATTN_INT8_QK, "fp8": sale.FLAG_ATTN_INT8_QK | sale.FLAG_ATTN_FP8_PV}[attn]
    p = sale.Params(batch=batch, n_q_heads=q_heads, n_kv_heads=kv_heads, seq_len=n, block_k=block_k, flags=flags, cu_seqlens=offsets)
    q = torch.randn(batch, q_heads, n, 128, generator=g, device="cuda").bfloat16()
    k, v = (torch.randn(batch, kv_heads, n, 128, generator=g, device="cuda").bfloat16() for _ in range(2))
    share = torch.rand(batch, q_heads, 1, 1, generator=g, device="cuda") ** 4      # of the blocks that a head keeps
    keep = torch.rand(batch, q_heads, n // 64, p.words * 64, generator=g, device="cuda") < share
    ends = list(offsets or (0, n))
    row = torch.cat([torch.arange((b - a) // 64) for a, b in zip(ends, ends[1:])]).cuda()[:, None]      # (within its sequence)
    col = torch.arange(p.words * 64, device="cuda")[None, :] * block_k // 64
    keep = (keep | (col == row)) & (col <= row)
    mask = (keep.view(batch, q_heads, n // 64, p.words, 64).long() << torch.arange(64, device="cuda")).sum(-1)
    counts = keep.sum(-1).int()
    want, want_lse = sale.sparse_attn(p, q, k, v, mask, None, want_lse=True)
    for _ in range(3):
        o, lse = sale.sparse_attn(p, q, k, v, mask, counts, want_lse=True)
        assert torch.equal(o, want) and torch.equal(lse, want_lse)
