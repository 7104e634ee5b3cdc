"""GPU parity where the decode kernels change shape with the number of query
rows and of work items.

A wave of the few-row kernel owns 16 or 32 rows, over tiles of 32 or 16 tokens;
with few workgroups a work item's keys are shared by four or two waves that
merge their parts.  It serves up to 32 rows, and any number while the work
items are few; enough of them run in 64-row workgroups (33 to 64 rows) whose
waves split each tile's tokens in two halves, or in 128-row ones.  The lengths sit on the edges of those tiles and
parts (one key, one token short of and past a 16- or 32-token tile, parts with
no key at all), the work-item counts on both sides of 256 and 512, and single
ranges run past the 64 page ids that a wave holds at a time.  Each case names
the shape it runs in, by the library's own rule.  Every output of
every compared row against the oracle, with the bounds of ``gpu_support``, the
closer ones from the kernels' own rounding among them.
"""
import numpy as np
import pytest

from gpu_support import (FP16_LIMITED, AttnStats, check_fp16_limited, check_modelled, check_sequence,
                         check_sequence_protected)
from launch_shape import of_run
from paper_2609_36760_amd import synthetic as syn

pytestmark = pytest.mark.gpu

EDGES = [2, 15, 16, 17, 31, 32, 33, 47, 48, 49, 63, 64, 65, 97, 129, 160]
SHORT = [33, 2, 40, 17]
FULL = SHORT * 60                # with EDGES: 256 sequences
CASES = [
    # (name, H, s_q, lens, cache, split, page, (sink, recent) or None, sequences compared: None all,
    #  the shape it runs in: rows and waves per workgroup)
    ("r16_four_waves", 16, 1, EDGES, "c4", 0, 64, None, None, (16, 4)),
    ("r16_four_waves_split96_paper", 16, 1, EDGES, "c2paper", 96, 64, None, None, (16, 4)),
    ("r16_four_waves_bf16", 16, 1, EDGES, "bf16", 0, 64, None, None, (16, 4)),
    # (32 rows of few work items: two row blocks of 16)
    ("r32_few_items", 16, 2, EDGES, "c4", 0, 64, None, None, (16, 4)),
    ("r32_few_items_prot", 32, 1, EDGES + [300], "c4", 128, 64, (4, 128), None, (16, 4)),
    ("r32_few_items_bf16", 32, 1, EDGES, "bf16", 96, 64, None, None, (16, 4)),
    # 257 to 512 workgroups: two waves per work item
    ("r16_two_waves_prot", 16, 1, EDGES + SHORT * 70, "c2", 0, 64, (3, 20), list(range(18)), (16, 2)),
    ("r32_two_waves_paper", 32, 1, EDGES + SHORT * 70, "c4paper", 0, 64, None, list(range(18)), (32, 2)),
    # more than 512: one wave per work item
    ("r16_one_wave", 16, 1, EDGES + SHORT * 130, "c4", 0, 64, None, list(range(18)), (16, 1)),
    ("r16_one_wave_paper_split64", 16, 1, EDGES + SHORT * 130, "c2paper", 64, 64, None, list(range(18)), (16, 1)),
    ("r32_one_wave", 16, 2, EDGES + SHORT * 130, "c2", 0, 64, None, list(range(18)), (32, 1)),
    ("r32_one_wave_prot", 16, 2, EDGES + SHORT * 130, "c4paper", 0, 64, (3, 20), list(range(18)), (32, 1)),
    ("r32_one_wave_bf16", 32, 1, EDGES + SHORT * 130, "bf16", 0, 64, None, list(range(18)), (32, 1)),
    # more than 64 pages in one wave's range
    ("r16_pages", 16, 1, [2200] + SHORT * 130, "c4", 0, 32, None, [0, 1], (16, 1)),
    ("r32_pages", 16, 2, [2200] + SHORT * 130, "c4", 0, 32, None, [0, 1], (32, 1)),
    ("r16_pages_four_waves", 16, 1, [8400, 33], "c4", 0, 32, None, None, (16, 4)),
    # many row blocks of 16 or 32 rows: few work items at 64 to 256 rows
    ("r64_few_items", 64, 1, EDGES, "c4", 0, 64, None, None, (16, 4)),
    ("r256_few_items_prot", 128, 2, [2, 33, 300], "c4", 64, 64, (4, 128), None, (16, 4)),
    ("r80_few_items_bf16", 80, 1, EDGES, "bf16", 96, 64, None, None, (16, 4)),
    ("r128_mid_items_paper", 128, 1, EDGES + SHORT * 12, "c2paper", 0, 64, None, list(range(18)), (32, 4)),
    # 256 work items of up to 192 tokens fill the chip with 64-row workgroups,
    # whose waves split each tile's tokens
    ("r64_nosplit", 64, 1, EDGES + FULL, "c4", 0, 64, None, list(range(18)), (64, 4)),
    ("r64_split160_sq2", 32, 2, EDGES + FULL, "c2", 160, 64, None, list(range(18)), (64, 4)),
    ("r48_paper", 48, 1, EDGES + FULL, "c4paper", 0, 32, None, list(range(18)), (64, 4)),
    ("r64_prot", 64, 1, EDGES + FULL, "c4", 0, 64, (3, 20), list(range(18)), (64, 4)),
    ("r64_bf16_sq2", 32, 2, EDGES + FULL, "bf16", 0, 64, None, list(range(18)), (64, 4)),
    ("r48_bf16", 48, 1, EDGES + FULL, "bf16", 0, 64, None, list(range(18)), (64, 4)),
    # and with 128-row ones
    ("r128_nosplit", 128, 1, EDGES + FULL, "c4", 0, 64, None, list(range(18)), (128, 4)),
    ("r128_split96_paper", 128, 1, EDGES + FULL, "c2paper", 96, 64, None, list(range(18)), (128, 4)),
    ("r256_sq2", 128, 2, EDGES + FULL, "c2", 0, 64, None, list(range(18)), (128, 4)),
    ("r128_prot_split96", 128, 1, EDGES + FULL, "c4", 96, 64, (3, 20), list(range(18)), (128, 4)),
    ("r160_bf16_sq2", 80, 2, EDGES + FULL, "bf16", 0, 64, None, list(range(18)), (128, 4)),
    # 32-row workgroups of four waves: 129 to 256 of them
    ("r32_four_waves", 16, 2, EDGES + SHORT * 30, "c4", 0, 64, None, list(range(18)), (32, 4)),
    ("r32_four_waves_prot", 32, 1, EDGES + [300] + SHORT * 30, "c2", 0, 64, (4, 128), list(range(18)), (32, 4)),
    ("r32_four_waves_bf16", 32, 1, EDGES + SHORT * 30, "bf16", 0, 64, None, list(range(18)), (32, 4)),
    ("r32_four_waves_paper_split384", 32, 1, EDGES + SHORT * 30 + [900], "c4paper", 384, 64, None,
     [*range(18), 136], (32, 4)),
    # and several row blocks of 32 rows
    ("r128_four_waves", 128, 1, EDGES + SHORT * 6, "c4", 0, 64, None, list(range(18)), (32, 4)),
    ("r128_four_waves_prot", 128, 1, EDGES + [300] + SHORT * 6, "c4paper", 0, 64, (3, 20), list(range(18)), (32, 4)),
    ("r160_four_waves_bf16", 80, 2, EDGES + SHORT * 6, "bf16", 0, 64, None, list(range(18)), (32, 4)),
    # two waves: 257 to 512 workgroups
    ("r32_two_waves_prot", 16, 2, EDGES + [300] + SHORT * 70, "c4", 0, 64, (4, 128), list(range(18)), (32, 2)),
    ("r32_two_waves_bf16", 32, 1, EDGES + SHORT * 70, "bf16", 0, 64, None, list(range(18)), (32, 2)),
    ("r32_two_waves_int2", 32, 1, EDGES + SHORT * 70, "c2", 0, 64, None, list(range(18)), (32, 2)),
    ("r128_two_waves", 128, 1, EDGES + SHORT * 14, "c4", 0, 64, None, list(range(18)), (32, 2)),
    ("r96_two_waves_prot", 48, 2, EDGES + [300] + SHORT * 18, "c2paper", 0, 64, (3, 20), list(range(18)), (32, 2)),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_row_regimes(case):
    import torch

    from paper_2609_36760_amd import _binding as mb
    from paper_2609_36760_amd.runner import DecodeRun
    name, H, s_q, lens, cache, split, page, prot, compared, shape = case
    w = syn.Workload(name, 900 + CASES.index(case), B=len(lens), H=H, s_q=s_q, context=None,
                     layers=((2 if cache.startswith("c2") else 4, 4),), split_tokens=split, ctx_range=(1, 2))
    policy = None if prot is None else mb.protect_policy(*prot)
    run = DecodeRun(w, kind="bf16" if cache == "bf16" else "lowbit", seq_lens=np.asarray(lens, np.int32),
                    page_size=page, protect=policy, meta="paper" if cache.endswith("paper") else "fp16")
    assert of_run(run) == shape
    run.fused_step()
    torch.cuda.synchronize()
    stats = AttnStats()
    check = check_sequence if policy is None else check_sequence_protected
    for b in range(len(lens)) if compared is None else compared:
        check(stats, run, b)
    print(f"  {name}: {len(lens)} sequences, {run.num_splits or len(lens)} work items", flush=True)
    # BF16 cache, one wave per work item or 64- and 128-row workgroups: the weights
    # are bf16 operands (relative error 2^-8), which alone moves an output of a
    # short sequence by up to 2^-7 of the magnitudes it averages -- past 2e-2 of the
    # batch's RMS where an outlier channel (10 x RMS) cancels.  The per-element
    # bound, which carries that term, applies instead.  Several waves carry each
    # weight to 16 bits, and the rule stands.
    pairs = shape[0] <= 32 and shape[1] > 1
    for b in range(len(lens)) if compared is None else compared:
        check_modelled(run, b, 2.0 ** -16 if pairs else 2.0 ** -8)
    if name in FP16_LIMITED:
        check_fp16_limited(stats, name)
    else:
        stats.check(name, max_rule=cache != "bf16" or pairs)
