"""Candidate groups of 1, 2, 4 and 8 at the sizes where the plan changes
between them (GPU), against the oracle.

The plan groups candidates by the bytes of all of them together: groups of 1
up to 16 MiB (8 MiB fail-fast), of 2 up to 64 MiB (48 MiB for up to 31 16-bit
candidates, 16 MiB fail-fast), else of 4, or 8 for 32 or more 16-bit
candidates; lists of more than 128 candidates groups of 2 up to 24 MiB and 4 up
to 64 MiB.
"""
import sys

import numpy as np
import pytest
import torch

import oracle
import paper_2608_02611_amd as kb
from tests.helpers import (assert_records_match, check_partial, ensure_built, oracle_positions_host, oracle_records,
                           same_record, to_device)

pytestmark = pytest.mark.gpu

CODE = {"f32": kb.KB_F32, "f16": kb.KB_F16, "bf16": kb.KB_BF16}
MIB = 1 << 20


@pytest.fixture(scope="module")
def dev():
    ensure_built()
    return torch.device("cuda:0")


def tensors(dt, K, n):
    """Passing candidates with noise of 2^-12 relative, and every third one
    wrong in a few elements (the last among them), with a NaN."""
    rng = np.random.default_rng(n)
    r = rng.standard_normal(n).astype(np.float32) + np.float32(3.0)
    cands = []
    for k in range(K):
        c = r * (1 + np.float32(2.0 ** -12) * rng.uniform(-1, 1, n).astype(np.float32))
        if k % 3 == 1:
            c[rng.integers(0, n, 3)] += np.float32(1.0)
            c[n - 1] = np.nan if k % 2 else c[n - 1] * 2
        cands.append(c)
    conv = {"f32": lambda x: x.astype(np.float32), "f16": oracle.f32_to_f16_n, "bf16": oracle.f32_to_bf16_n}[dt]
    return conv(r), [conv(c) for c in cands]


@pytest.mark.parametrize("dt,K,limit,group", [("f32", 7, 8, 1), ("f32", 7, 16, 1), ("bf16", 5, 16, 1),
                                              ("f32", 11, 64, 2), ("f16", 35, 64, 2)])
@pytest.mark.parametrize("past", [0, 1])
def test_group_size_limits(dev, dt, K, limit, group, past):
    n = limit * MIB // (K * (4 if dt == "f32" else 2)) + past
    atol, rtol = (1e-5, 1e-3) if dt == "f32" else (1e-3, 1e-2)
    print("groups", dt, K, n, flush=True)
    sys.stdout.flush()
    size = kb.kb_screen_launch(K, n, CODE[dt])["group_size"]
    if limit > 8:
        nxt = 2 if group == 1 else 8 if dt == "f16" else 4
        assert size == (nxt if past else group)
    r, cs = tensors(dt, K, n)
    orc = oracle_records(r, cs, atol, rtol, dt=dt)
    locs = oracle_positions_host(r, cs, dt, atol, rtol, orc)
    ref, cands = to_device(r, dt, dev), [to_device(c, dt, dev) for c in cs]
    # one workspace for all modes, zero-filled once: their groups may differ
    ws = torch.empty(kb.kb_screen_positions_workspace_bytes(K, n, CODE[dt]), dtype=torch.uint8, device=dev)
    kb.kb_screen_workspace_init(ws)
    for _ in range(2):
        st, _ = kb.kb_screen(ref, cands, atol, rtol, 0, ws)
        full, _ = kb.kb_screen_stats(st, K)
        assert_records_match(full, orc, "plain")
        st, _ = kb.kb_screen(ref, cands, atol, rtol, kb.KB_FAIL_FAST, ws)
        fast, _ = kb.kb_screen_stats(st, K)
        for k, (g, f, o) in enumerate(zip(fast, full, orc)):
            if o["mismatches"] == 0:
                assert same_record(g, f), (k, g, f)
            else:
                check_partial(g, o, "fail-fast %d" % k)
        d_loc = kb.alloc_locate(K, dev)
        st, _ = kb.kb_screen(ref, cands, atol, rtol, 0, ws, d_loc=d_loc)
        recs, _ = kb.kb_screen_stats(st, K)
        assert_records_match(recs, orc, "positions")
        assert kb.read_locate(d_loc, K) == locs


@pytest.mark.parametrize("dt,K", [("f32", 3), ("f32", 9), ("bf16", 37)])
def test_one_workspace_for_all_sizes(dev, dt, K):
    """One workspace, sized for the largest tensor and zero-filled between
    sizes, through every group size of the plan (groups of 1, 2 and 4 or 8
    lay their tickets and sums in the same regions)."""
    es = 4 if dt == "f32" else 2
    atol, rtol = (1e-5, 1e-3) if dt == "f32" else (1e-3, 1e-2)
    sizes = [m * MIB // (K * es) for m in (65, 64, 17, 15, 9, 7, 1)]
    ws = torch.empty(kb.kb_screen_positions_workspace_bytes(K, sizes[0], CODE[dt]), dtype=torch.uint8, device=dev)
    r, cs = tensors(dt, K, sizes[0])
    seen = set()
    for n in sizes:
        print("one workspace", dt, K, n, flush=True)
        seen.add(kb.kb_screen_launch(K, n, CODE[dt])["group_size"])
        rn, cn = r[:n], [c[:n] for c in cs]
        orc = oracle_records(rn, cn, atol, rtol, dt=dt)
        locs = oracle_positions_host(rn, cn, dt, atol, rtol, orc)
        ref, cands = to_device(rn, dt, dev), [to_device(c, dt, dev) for c in cn]
        kb.kb_screen_workspace_init(ws)
        st, _ = kb.kb_screen(ref, cands, atol, rtol, kb.KB_FAIL_FAST, ws)
        recs, _ = kb.kb_screen_stats(st, K)
        assert [g["passed"] for g in recs] == [o["passed"] for o in orc]
        st, _ = kb.kb_screen(ref, cands, atol, rtol, 0, ws)
        assert_records_match(kb.kb_screen_stats(st, K)[0], orc, "plain")
        d_loc = kb.alloc_locate(K, dev)
        st, _ = kb.kb_screen(ref, cands, atol, rtol, 0, ws, d_loc=d_loc)
        assert_records_match(kb.kb_screen_stats(st, K)[0], orc, "positions")
        assert kb.read_locate(d_loc, K) == locs
    assert len(seen) >= 3, seen


@pytest.mark.parametrize("dt,K,mib", [("f32", 131, 24), ("f16", 131, 24), ("bf16", 131, 64), ("bf16", 31, 48)])
@pytest.mark.parametrize("past", [0, 1])
def test_long_lists_at_the_limits(dev, dt, K, mib, past):
    """Lists of more than 128 candidates (their table in host memory) and the
    16-bit limit of short lists, up to and past each limit."""
    n = mib * MIB // (K * (4 if dt == "f32" else 2)) + past
    atol, rtol = (1e-5, 1e-3) if dt == "f32" else (1e-3, 1e-2)
    print("long list", dt, K, n, flush=True)
    r, cs = tensors(dt, K, n)
    orc = oracle_records(r, cs, atol, rtol, dt=dt)
    locs = oracle_positions_host(r, cs, dt, atol, rtol, orc)
    ref, cands = to_device(r, dt, dev), [to_device(c, dt, dev) for c in cs]
    ws = kb.alloc_workspace(K, n, CODE[dt], dev, positions=True)
    st, _ = kb.kb_screen(ref, cands, atol, rtol, 0, ws)
    assert_records_match(kb.kb_screen_stats(st, K)[0], orc, "plain")
    d_loc = kb.alloc_locate(K, dev)
    st, _ = kb.kb_screen(ref, cands, atol, rtol, 0, ws, d_loc=d_loc)
    assert_records_match(kb.kb_screen_stats(st, K)[0], orc, "positions")
    assert kb.read_locate(d_loc, K) == locs
