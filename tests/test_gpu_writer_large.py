"""The writer's two-piece launch (protected appends of 49 152 tokens or more)
against one-piece launches of the same tokens, byte for byte (GPU): cache pages
and protection buffers, at an odd token count whose last thread has one piece,
with skipped slots, sequences outside the batch and protection buffers outside
the range.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

N = 49153


@pytest.mark.parametrize("c_bits", [4, 2])
@pytest.mark.parametrize("paper", [False, True])
def test_two_piece_append_equals_one_piece(c_bits, paper):
    import torch

    from paper_2609_36760_amd import _binding as mb
    fmt = mb.cache_format(c_bits=c_bits, meta=mb.MLA_META_PAPER if paper else mb.MLA_META_FP16)
    pol = mb.protect_policy(4, 128)
    g = torch.Generator(device="cuda")
    g.manual_seed(7 + c_bits)
    c = torch.randn((N, 512), generator=g, device="cuda").bfloat16()
    k = torch.randn((N, 64), generator=g, device="cuda").bfloat16()
    pages = (N + 63) // 64
    slots = torch.randperm(pages * 64, generator=g, device="cuda")[:N].contiguous()
    slots[5::997] = -1
    slots[11::1499] = pages * 64
    B, per = 3, (N + 2) // 3
    seq = (torch.arange(N, device="cuda") // per).to(torch.int32)
    pos = (torch.arange(N, device="cuda") % per).to(torch.int32)
    seq[100:110], seq[200:210] = -1, B
    lens = torch.tensor([per, per, N - 2 * per], dtype=torch.int32, device="cuda")
    prot_slot = torch.tensor([1, 0, 5], dtype=torch.int32, device="cuda")      # the last one out of range
    got = []
    for chunk in (N, 20011):
        cache = torch.zeros(pages * mb.mla_lowbit_page_bytes(fmt), dtype=torch.uint8, device="cuda")
        prot = torch.zeros(2 * mb.mla_protect_buffer_bytes(fmt, pol), dtype=torch.uint8, device="cuda")
        for i in range(0, N, chunk):
            s = slice(i, min(N, i + chunk))
            mb.mla_lowbit_quant_append_protected(fmt, pol, c[s], k[s], slots[s], cache, pages, seq[s], pos[s], lens,
                                                 prot_slot, prot, 2)
        torch.cuda.synchronize()
        got.append((cache.cpu().numpy(), prot.cpu().numpy()))
    assert np.array_equal(got[0][0], got[1][0]) and np.array_equal(got[0][1], got[1][1])
    assert got[0][0].any() and got[0][1].any()
