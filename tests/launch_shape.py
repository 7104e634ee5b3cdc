"""Launch shapes of the decode kernels for the tests: which one a call takes
(the library's own rule), and calls made in a given one.

A shape is (query rows per workgroup, waves per workgroup): 16 or 32 rows with
one, two or four waves that share a work item's keys (decode_narrow.hip), 64 or
128 rows with four waves on one tile (decode_attn.hip).
"""
from __future__ import annotations

import contextlib

NARROW = [(16, 1), (16, 2), (16, 4), (32, 1), (32, 2), (32, 4)]


def chosen(lowbit: bool, rows: int, num_work: int, split_tokens: int) -> tuple[int, int]:
    """The shape of a call of ``rows`` = s_q * H query rows over ``num_work``
    work items (``split_tokens`` = 0: unsplit)."""
    from paper_2609_36760_amd import _binding as mb
    v = mb.library().mla_internal_decode_shape(int(lowbit), rows, num_work, split_tokens)
    return v // 8, v % 8


def of_run(run) -> tuple[int, int]:
    """The shape that the library chooses for a DecodeRun's decode calls."""
    return chosen(run.kind != "bf16", run.s_q * run.H, run.num_splits or run.B, run.split_tokens or 0)


def wide(rows: int) -> tuple[int, int]:
    """The shape of large launches of ``rows`` > 32 query rows."""
    return (64, 4) if rows <= 64 else (128, 4)


def set_next(shape: tuple[int, int]) -> None:
    from paper_2609_36760_amd import _binding as mb
    mb.library().mla_internal_shape_next_decode(*shape)


@contextlib.contextmanager
def pinned(shape):
    """Every decode call of a DecodeRun inside the block runs in ``shape`` (None:
    in the shape the library chooses)."""
    from paper_2609_36760_amd.runner import DecodeRun
    if shape is None:
        yield
        return
    calls = {n: getattr(DecodeRun, n) for n in ("attend", "fused_step")}

    def wrapped(call):
        def run(self, *args, **kw):
            set_next(shape)
            return call(self, *args, **kw)
        return run

    for n, call in calls.items():
        setattr(DecodeRun, n, wrapped(call))
    try:
        yield
    finally:
        for n, call in calls.items():
            setattr(DecodeRun, n, call)
        set_next((0, 0))


def with_wide(cases, rows_of):
    """(case, shape) pairs: every case in the shape the library chooses for it
    (few work items: 16 or 32 rows), and those of more than 32 query rows in the
    64- or 128-row one of large launches too."""
    return [(c, None) for c in cases] + [(c, wide(rows_of(c))) for c in cases if rows_of(c) > 32]


def ids(pairs, name_of=lambda c: c[0]):
    return [name_of(c) + ("" if s is None else f"-rows{s[0]}") for c, s in pairs]
