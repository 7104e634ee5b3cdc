"""The rule that shapes a decode launch (host only; no GPU): which kernels it
reaches, where its lines lie, and that a shape pinned for a call is checked."""
import itertools

import pytest

from launch_shape import NARROW, chosen, set_next


@pytest.fixture(scope="module", autouse=True)
def built():
    import os

    from paper_2609_36760_amd import _binding as mb
    if not os.path.exists(mb.LIB_PATH):
        pytest.skip("libmla_lowbit.so not built (run __graft_entry__.build())")


@pytest.mark.parametrize("lowbit", [True, False])
def test_every_shape_is_reached_and_no_other(lowbit):
    got = {}
    items = [*range(1, 70), *range(70, 700, 13), 1024, 5000, 1 << 20]
    for rows, n, split in itertools.product([16, 32, 48, 64, 80, 96, 128, 160, 256, 512], items, [0, 32, 64, 256, 512, 4096]):
        got.setdefault(chosen(lowbit, rows, n, split), set()).add(rows)
    assert set(got) == {*NARROW, (64, 4), (128, 4)}
    assert got[(64, 4)] == {48, 64}
    assert got[(128, 4)] == {80, 96, 128, 160, 256, 512}
    assert all(r <= 32 or r > 32 and lowbit for r in got[(16, 1)] | got[(32, 1)]), got
    assert 16 not in got[(32, 4)] | got[(32, 2)] | got[(32, 1)]


def test_lines_of_the_rule():
    # 16 rows: four waves up to 256 workgroups, two up to 512
    assert [chosen(True, 16, n, 64) for n in (1, 256, 257, 512, 513)] == [(16, 4), (16, 4), (16, 2), (16, 2), (16, 1)]
    # the measured points of the rule's comment, 128 and 64 rows
    assert chosen(True, 128, 16, 512) == (16, 4)
    assert chosen(True, 128, 64, 512) == (32, 4)
    assert chosen(True, 128, 64, 2048) == (32, 4)
    assert chosen(True, 128, 256, 512) == (128, 4)
    assert chosen(True, 64, 128, 512) == (32, 4)
    assert chosen(True, 64, 272, 2048) == (64, 4)
    # the largest launches that the host accepts keep a shape that fits one dispatch
    assert chosen(True, 16, (1 << 26) - 8, 0) == (16, 1)
    assert chosen(True, 32, (1 << 25) - 8, 0)[1] == 1
    assert chosen(True, 128, (1 << 24) - 8, 0) == (128, 4)


@pytest.mark.parametrize("rows,lowbit,shape", [(16, True, (32, 4)), (32, True, (64, 4)), (64, True, (128, 4)),
                                               (128, True, (64, 4)), (128, True, (16, 3)), (128, False, (16, 1)),
                                               (128, True, (48, 4)), (128, True, (128, 2)), (128, True, (-16, 4))])
def test_a_shape_that_is_not_one_for_the_rows_is_refused(rows, lowbit, shape):
    import ctypes

    from paper_2609_36760_amd import _binding as mb
    lib, fmt = mb.library(), mb.cache_format()
    fn = lib.mla_lowbit_decode_attn if lowbit else lib.mla_bf16_decode_attn
    set_next(shape)
    try:        # (addresses that a refused call never uses)
        assert fn(ctypes.byref(fmt), 16, 16, 256, 4, 16, 2, 16, 1, 1, rows, 0.07, 0, None, 0, 16, None, None, None,
                  None, None) == mb.MLA_EINVAL
    finally:
        set_next((0, 0))
