"""Launch shapes of the decode kernels for the tests: which one a call takes
(the library's own rule), and calls made in a given one.

A shape is (query rows per workgroup, waves per workgroup): 16 or 32 rows with
one, two or four waves that share a work item's keys (decode_narrow.hip), 64 or
128 rows with four waves on one tile (decode_attn.hip).
"""
from __future__ import annotations

import contextlib
import inspect

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


DECODE_CALLS = ("mla_lowbit_decode_attn", "mla_bf16_decode_attn", "mla_lowbit_append_decode_attn",
                "mla_bf16_append_decode_attn", "mla_lowbit_decode_attn_protected",
                "mla_lowbit_append_decode_attn_protected", "mla_lowbit_decode_attn_noalloc")


@contextlib.contextmanager
def pinned(shape):
    """Every decode call of the binding inside the block runs in ``shape``: a
    pair, "wide" for :func:`wide` of the call's rows (calls of up to 32 rows run
    as they would), or None for the shape the library chooses."""
    from paper_2609_36760_amd import _binding as mb
    if shape is None:
        yield
        return
    calls = {n: getattr(mb, n) for n in DECODE_CALLS}

    def wrapped(call):
        sig = inspect.signature(call)

        def run(*args, **kw):
            given = sig.bind(*args, **kw).arguments
            rows = given["s_q"] * given["H"]
            if shape != "wide":
                set_next(shape)
            elif rows > 32:
                set_next(wide(rows))
            return call(*args, **kw)
        return run

    for n, call in calls.items():
        setattr(mb, n, wrapped(call))
    try:
        yield
    finally:
        for n, call in calls.items():
            setattr(mb, n, call)
        set_next((0, 0))


def with_wide(cases, rows_of):
    """Parameters (case, launch_shape): every case in the shape the library
    chooses for it -- small tests have few work items, which run in 16- or 32-row
    workgroups -- and those of more than 32 query rows (``rows_of(case)``) in the
    64- or 128-row workgroups of large launches as well."""
    import pytest
    return ([pytest.param(c, None, id=c[0]) for c in cases] +
            [pytest.param(c, "wide", id=f"{c[0]}-wide") for c in cases if rows_of(c) > 32])
