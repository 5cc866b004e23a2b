"""The screening kernel's rare paths in every group size (GPU), against the
oracle.

Short passes take groups of 1 or 2 candidates, so tensors small enough for
hand-made values never reach the kernels of 4 and 8.  Here a second copy of the
library, with its group size fixed through KB_SCREEN_TUNE, screens them: signed
zeros, infinities and NaN on either side, differences too small or too large
for a binary32 square, tied maxima within and across chunks, a mismatch in the
tail alone, and a last group padded with the reference.
"""
import importlib.util
import os
import shutil
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


@pytest.fixture(scope="module")
def dev():
    ensure_built()
    return torch.device("cuda:0")


@pytest.fixture(scope="module", params=[1, 2, 4, 8])
def tuned(request, tmp_path_factory, dev):
    """(group size, the package over a copy of the library that keeps to it)."""
    path = str(tmp_path_factory.mktemp("tuned") / ("libkb_kg%d.so" % request.param))
    shutil.copy(kb.LIB_PATH, path)
    name = "kb_tuned_%d" % request.param
    spec = importlib.util.spec_from_file_location(name, kb.__file__)
    m = importlib.util.module_from_spec(spec)
    sys.modules[name] = m
    spec.loader.exec_module(m)
    m.LIB_PATH = path
    os.environ["KB_SCREEN_TUNE"] = "kg=%d" % request.param
    try:
        assert m.kb_screen_launch(16, 1 << 20, kb.KB_F32)["group_size"] == request.param  # (read once, here)
    finally:
        del os.environ["KB_SCREEN_TUNE"]
    return request.param, m


def tensors(dt, K, n):
    rng = np.random.default_rng(n + K)
    r = rng.standard_normal(n).astype(np.float32)
    r[5::97] = 0.0
    r[6::97] = -0.0
    r[7::193] = 2.0 ** -24 if dt == "f16" else 2.0 ** -133  # subnormal
    r[8::389] = 1.0
    big = 60000.0 if dt == "f16" else 3e38
    r[9::1009] = big
    r[10::2003] = np.inf
    r[11::2003] = -np.inf
    r[12::4001] = np.nan
    cands = []
    for k in range(K):
        c = r.copy()
        if k % 11 == 1:  # signs of zeros only
            c[5::97] = -0.0
        elif k % 11 == 2:  # differences whose squares underflow binary32
            c[5::97] = 2.0 ** -24 if dt == "f16" else 2.0 ** -100
            c[7::193] = 0.0
        elif k % 11 == 3:  # one maximum in many places
            c[8::389] = 1.5
        elif k % 11 == 4:  # NaN and infinities on the candidate's side
            c[100::5003] = np.nan
            c[200::5003] = np.inf
            c[300::5003] = -np.inf
        elif k % 11 == 5:  # finite values whose difference, or its square, is infinite
            c[9::1009] = -big
        elif k % 11 == 6:  # the last element alone
            c[n - 1] = c[n - 1] + 1.0 if np.isfinite(c[n - 1]) else 3.0
        elif k % 11 == 7:  # infinities of the other sign
            c[10::2003] = -np.inf
        elif k % 11 == 8:  # everything, by a little
            c *= np.float32(1.0 + 2.0 ** -7)
        elif k % 11 == 9:  # a zeroed stretch across a chunk boundary
            c[500:530] = 0.0
        elif k % 11 == 10:  # a tie of the relative maximum in the first and the last chunk
            i = np.flatnonzero(r == 1.0)
            c[i[0]] = c[i[-1]] = 3.0
        cands.append(c)
    conv = {"f32": lambda x: x.astype(np.float32), "f16": oracle.f32_to_f16_n, "bf16": oracle.f32_to_bf16_n}[dt]
    with np.errstate(over="ignore"):
        return conv(r), [conv(c) for c in cands]


@pytest.mark.parametrize("dt", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("K,n", [(11, 40 * 512 + 77), (13, 9 * 512), (22, 300 * 512 + 300), (3, 511)])
@pytest.mark.parametrize("equal_nan", [0, kb.KB_EQUAL_NAN])
def test_rare_paths(tuned, dev, dt, K, n, equal_nan):
    kg, m = tuned
    print("rare paths", kg, dt, K, n, equal_nan, flush=True)
    atol, rtol = (1e-5, 1e-5) if dt == "f32" else (1e-3, 1e-3)
    r, cs = tensors(dt, K, n)
    orc = oracle_records(r, cs, atol, rtol, equal_nan, dt=dt)
    locs = oracle_positions_host(r, cs, dt, atol, rtol, orc, equal_nan)
    ref, cands = to_device(r, dt, dev), [to_device(c, dt, dev) for c in cs]
    ws = m.alloc_workspace(K, n, CODE[dt], dev, positions=True)
    for _ in range(2):
        st, _ = m.kb_screen(ref, cands, atol, rtol, equal_nan, ws)
        full, _ = m.kb_screen_stats(st, K)
        assert_records_match(full, orc, "plain")
        d_loc = m.alloc_locate(K, dev)
        st, _ = m.kb_screen(ref, cands, atol, rtol, equal_nan, ws, d_loc=d_loc)
        assert_records_match(m.kb_screen_stats(st, K)[0], orc, "positions")
        assert m.read_locate(d_loc, K) == locs
        st, _ = m.kb_screen(ref, cands, atol, rtol, equal_nan | kb.KB_FAIL_FAST, ws)
        fast, _ = m.kb_screen_stats(st, K)
        for k, (g, f, o) in enumerate(zip(fast, full, orc)):
            if o["mismatches"] == 0:
                assert same_record(g, f), (k, g, f)
            else:
                check_partial(g, o, "fail-fast kg=%d %s cand %d" % (kg, dt, k))
