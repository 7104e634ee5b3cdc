"""GPU parity of every compiled decode kernel.

The decode kernels are instances over the cache (INT4 and INT2 content with the
fp16 and the paper's metadata, BF16), with and without BF16 protection, and the
launch shape: 16 or 32 query rows with one, two or four waves that share a work
item's keys, 64 rows (token-split waves) and 128.  Here each of them runs, in a
shape set for the call, over key lists that end one short of, on and past a
16- or 32-token tile, that leave some of the waves without a key, and that reach
from packed into protected tiles; row blocks full, part-filled and several of
them; the step's new tokens written inside the launch.  Every output against the
oracle, with the bounds of ``gpu_support``: the mean, lse and per-element rules
against the exact attention, and the closer ones of ``check_modelled``, which a
product dropped or misplaced in one kernel does not pass.
"""
import numpy as np
import pytest

from gpu_support import AttnStats, check_modelled, check_sequence, check_sequence_protected
from launch_shape import NARROW
from paper_2609_36760_amd import synthetic as syn

pytestmark = pytest.mark.gpu

LENS = [2, 15, 17, 31, 32, 33, 49, 64, 65, 97, 129, 160, 261]
LOWBIT = ["c4", "c2", "c4paper", "c2paper"]
# (heads, query tokens) of few and many rows for each shape
ROWS = {16: [(16, 1), (48, 2)], 32: [(16, 2), (80, 1)], 64: [(48, 1), (32, 2)], 128: [(80, 1), (80, 2)]}
KERNELS = [(cache, prot, shape)
           for cache, prot in [(c, None) for c in [*LOWBIT, "bf16"]] + [(c, (3, 20)) for c in LOWBIT]
           for shape in [*NARROW, (64, 4), (128, 4)]]


@pytest.mark.parametrize("split", [0, 96])
@pytest.mark.parametrize("cache,prot,launch_shape", KERNELS, indirect=["launch_shape"],
                         ids=[f"{c}{'-prot' if p else ''}-{s[0]}x{s[1]}" for c, p, s in KERNELS])
def test_every_kernel(cache, prot, launch_shape, split):
    import torch

    from paper_2609_36760_amd import _binding as mb
    from paper_2609_36760_amd.runner import DecodeRun
    rows, waves = launch_shape
    H, s_q = ROWS[rows][split // 96]
    if cache == "bf16" and waves == 1:
        H, s_q = 16, rows // 16             # one wave: launches of at most 32 rows
    seed = 1000 + KERNELS.index((cache, prot, launch_shape))
    w = syn.Workload(f"kernel_{cache}_{rows}x{waves}", seed, B=len(LENS), H=H, s_q=s_q, context=None,
                     layers=((2 if cache.startswith("c2") else 4, 4),), split_tokens=split, ctx_range=(1, 2))
    policy = None if prot is None else mb.protect_policy(*prot)
    run = DecodeRun(w, kind="bf16" if cache == "bf16" else "lowbit", seq_lens=np.asarray(LENS, np.int32),
                    protect=policy, meta="paper" if cache.endswith("paper") else "fp16")
    run.fused_step()
    torch.cuda.synchronize()
    stats = AttnStats()
    for b in range(len(LENS)):
        (check_sequence if policy is None else check_sequence_protected)(stats, run, b)
    label = f"{cache} {prot} {launch_shape} split {split} {H} heads"
    # the max rule is a rule for a batch of many rows; here the far closer bound
    # from the kernels' own rounding stands in its place
    stats.check(label, max_rule=False)
    pairs = rows <= 32 and waves > 1
    worst = max(check_modelled(run, b, 2.0 ** -16 if pairs else 2.0 ** -8) for b in range(len(LENS)))
    print(f"  {label}: {worst:.3g} of the bound from the rounding model", flush=True)
