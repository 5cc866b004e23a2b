"""Performance cases of the screening library, each through its public entry points.

A case is a dict of plain values.  `op` names the call that it stands for:

  screen   Screener.launch(): K candidate outputs against one reference, the
           per-candidate records on the device; with `read` the records are
           also read back and the verdicts formed (Screener.read), as a
           search that decides on the spot does; with `positions` the first
           mismatch and the places of the maxima are found in the same pass;
  reject   the fail-fast screen with the records in pinned host memory and
           the verdicts taken from there (which elements of a failing
           candidate are read depends on timing, so the outputs are the
           verdicts and the sums of the candidates that pass);
  multi    MultiScreener.launch(): candidates that return two tensors, an
           f16 [batch, heads, seq, dim] and an f32 [batch, heads, seq];
  inputs   kb_gen_inputs: `tensors` seeded input tensors of one size;
  build    a synthetic workload made on the device: a reference and K
           candidates with planted changes, into buffers in hand;
  rung     kb_rung_stats and kb_rung_promote: timing samples to statistics,
           scores and the promotion decision.

`data` names the values: "plain" normal outputs with small noise, one
candidate with NaN and one wrong in 1% of its elements; "gemm" normal times 64
with relative noise of 2^-8 .. 2^-6 and two candidates with a zeroed tile;
"softmax" probabilities with added noise of 1e-9 .. 1e-3; "attn" normal with
exact copies, last-bit flips and planted infinities; "heavy" Student-t with
subnormals, signed zeros and infinities, candidates that flip zero signs,
flush subnormals and differ by up to 1e-7.
"""
import math

import numpy as np
import torch

import paper_2608_02611_amd as kb

DEV = "cuda:0"
DT = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
SIZE = {"f32": 4, "f16": 2, "bf16": 2}
TOL = {"plain": (1e-5, 1e-5), "gemm": (1e-2, 1e-2), "softmax": (1e-6, 1e-5), "attn": (1e-3, 1e-3),
       "heavy": (1e-8, 1e-6)}


def listed():
    return [
        # the smallest call: four candidates of 65,536 elements, verdict wanted at once
        dict(name="screen_small_f32", op="screen", data="plain", dtype="f32", K=4, n=65536, cols=256, read=True),
        # a matrix-product output of ordinary size, the candidates of one generation
        dict(name="screen_gemm_bf16", op="screen", data="gemm", dtype="bf16", K=16, n=4096 * 4096, cols=4096),
        # many small candidates (a row-softmax output); the launch table is in host memory
        dict(name="screen_softmax_f32", op="screen", data="softmax", dtype="f32", K=1024, n=256 * 1024, cols=1024,
             read=True),
        # an attention output, a long candidate list
        dict(name="screen_attn_f16", op="screen", data="attn", dtype="f16", K=64, n=8 * 2048 * 4096, cols=4096),
        # the largest tensors: 4 GiB each, heavy-tailed values
        dict(name="screen_heavy_f32", op="screen", data="heavy", dtype="f32", K=8, n=1 << 30, cols=1024),
        # feedback for failed candidates, on a size that is no multiple of anything
        dict(name="positions_odd_bf16", op="screen", data="gemm", dtype="bf16", K=16, n=4095 * 4097, cols=4095,
             positions=True),
        # early rejection of a list of which half fails
        dict(name="reject_attn_f16", op="reject", data="attn", dtype="f16", K=64, n=1 << 24, cols=4096),
        # a kernel that returns its output and the row statistics, odd sequence length
        dict(name="multi_attn", op="multi", data="attn", dtype="f16", K=16, batch=4, heads=32, seq=2047, dim=128),
        # the seeded q, k and v of an attention benchmark
        dict(name="inputs_normal_f16", op="inputs", dist="normal", dtype="f16", n=4 * 32 * 2048 * 128, tensors=3,
             offset=0),
        # workloads made on the device: heavy-tailed fp32, and softmax rows with added noise
        dict(name="build_heavy_f32", op="build", data="heavy", dtype="f32", K=8, n=1 << 24, cols=4096),
        dict(name="build_softmax_f32", op="build", data="softmax", dtype="f32", K=64, n=256 * 1024, cols=1024),
        # a whole rung: 1024 candidates on 3 shapes, 60 timed iterations
        dict(name="rung_1024", op="rung", C=1024, S=3, iters=60, rung=2),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _numel(rng, lo, hi):
    """(n, cols): about half the sizes odd, the others rows of a common width."""
    n = _log_int(rng, lo, hi)
    if rng.random() < 0.5:
        cols = rng.choice([x for x in (128, 256, 768, 1024, 4096) if x <= n])
        return n // cols * cols, cols
    cols = rng.randrange(100, 1025) if n >= 1025 else n
    return n | 1, min(cols, n)


def draw(rng):
    op = rng.choice(["screen", "screen", "screen", "positions", "reject", "multi", "inputs", "build", "rung"])
    if op in ("screen", "positions", "reject"):
        data = rng.choice(["plain", "gemm", "softmax", "attn", "heavy"])
        dtype = rng.choice(["f32", "f16", "bf16"]) if data in ("plain", "gemm", "attn") else "f32"
        K = _log_int(rng, 1, 1024) if rng.random() < 0.3 else _log_int(rng, 2, 64)
        n, cols = _numel(rng, 4096, min(1 << 28, (8 << 30) // (K * SIZE[dtype])))
        if op == "reject":
            return dict(op="reject", data=data, dtype=dtype, K=K, n=n, cols=cols)
        c = dict(op="screen", data=data, dtype=dtype, K=K, n=n, cols=cols)
        if op == "positions":
            c["positions"] = True
        if K * n * SIZE[dtype] < (64 << 20):
            c["read"] = True
        return c
    if op == "multi":
        return dict(op="multi", data="attn", dtype=rng.choice(["f16", "bf16"]), K=_log_int(rng, 2, 32),
                    batch=rng.randrange(1, 5), heads=rng.choice([8, 12, 16, 32]), seq=_log_int(rng, 128, 2048),
                    dim=rng.choice([64, 96, 128]))
    if op == "inputs":
        n, _ = _numel(rng, 4096, 1 << 28)
        return dict(op="inputs", dist=rng.choice(["normal", "normal", "uniform", "student_t3"]),
                    dtype=rng.choice(["f32", "f16", "bf16"]), n=n, tensors=rng.randrange(1, 4),
                    offset=rng.choice([0, 0, 0, rng.randrange(1, 1 << 20)]))
    if op == "build":
        data = rng.choice(["gemm", "softmax", "attn", "heavy"])
        dtype = "f32" if data in ("softmax", "heavy") else rng.choice(["f32", "f16", "bf16"])
        K = _log_int(rng, 2, 64)
        n, cols = _numel(rng, 4096, min(1 << 26, (2 << 30) // (K * SIZE[dtype])))
        return dict(op="build", data=data, dtype=dtype, K=K, n=n // cols * cols, cols=cols)
    return dict(op="rung", C=_log_int(rng, 8, 2048), S=rng.randrange(1, 7), iters=rng.choice([4, 16, 60, 60, 100, 200]),
                rung=rng.randrange(0, 3))


# ------------------------------------------------------------------ inputs ---

def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(0x5EED + 7919 * int(seed))


def _parts(n, step=1 << 26):
    for a in range(0, n, step):
        yield a, min(n, a + step)


def _reference(data, n, cols, dtype, g):
    ref = torch.empty(n, dtype=dtype, device=DEV)
    if data == "softmax":
        rows = n // cols
        head = rows * cols
        ref[:head] = torch.softmax(2.0 * torch.randn(rows, cols, generator=g, device=DEV), dim=1).view(-1)
        ref[head:] = 1.0 / cols
        return ref
    for a, b in _parts(n):
        z = torch.randn(b - a, generator=g, device=DEV)
        if data == "gemm":
            z *= 64.0
        elif data == "heavy":
            chi = torch.zeros_like(z)
            for _ in range(3):
                chi += torch.randn(b - a, generator=g, device=DEV).square_()
            z /= chi.div_(3.0).sqrt_()
            u = torch.rand(b - a, generator=g, device=DEV)
            sign = torch.sign(z)
            z = torch.where(u < 2.0 ** -10, sign * 1e-39, z)
            z = torch.where((u >= 2.0 ** -10) & (u < 2.0 ** -9), sign * 0.0, z)
            z = torch.where((u >= 2.0 ** -9) & (u < 2.0 ** -9 + 2.0 ** -20), sign * math.inf, z)
        ref[a:b] = z
    return ref


def _candidate(ref, data, k, K, cols, g):
    n = ref.numel()
    c = ref.clone()
    if data == "plain":
        if k % 4 == 1:
            c += (torch.rand(n, generator=g, device=DEV) * 2e-6 - 1e-6).to(c.dtype)
        elif k % 4 == 2:
            c[torch.randint(0, n, (5,), generator=g, device=DEV)] = math.nan
        elif k % 4 == 3:
            hit = torch.rand(n, generator=g, device=DEV) < 0.01
            c = torch.where(hit, c * 1.01, c)
    elif data == "gemm":
        s = 2.0 ** (-8.0 + 2.0 * (k % 16) / 15.0)
        for a, b in _parts(n):
            e = torch.rand(b - a, generator=g, device=DEV).mul_(2 * s).sub_(s)
            c[a:b] = torch.addcmul(ref[a:b].float(), ref[a:b].float(), e)
        if k < 2 and n >= 64 * cols and cols >= 64:
            c[:n // cols * cols].view(-1, cols)[:64, :64] = 0.0
    elif data == "softmax":
        c += torch.randn(n, generator=g, device=DEV) * 10.0 ** (-9.0 + 6.0 * k / max(1, K - 1))
    elif data == "attn":
        if k % 2 == 1:
            for a, b in _parts(n):
                bits = c[a:b].view(torch.int32 if c.dtype == torch.float32 else torch.int16)
                bits ^= (torch.rand(b - a, generator=g, device=DEV) < 0.001).to(bits.dtype)
        if k % 4 >= 2:
            i = torch.randint(0, n, (64,), generator=g, device=DEV)
            c[i] = torch.copysign(torch.full_like(c[i], math.inf), ref[i])
    else:  # heavy
        for a, b in _parts(n):
            x = ref[a:b]
            e = torch.rand(b - a, generator=g, device=DEV).mul_(2e-7).sub_(1e-7)
            y = torch.addcmul(x, x, e)
            y = torch.where(x == 0.0, -x, y)
            y = torch.where((x.abs() < 2.0 ** -126) & (x != 0.0), x * 0.0, y)
            y = torch.where(torch.isinf(x), x, y)
            hit = torch.rand(b - a, generator=g, device=DEV) < 0.5
            c[a:b] = torch.where(hit, y, x)
    return c


def _tensors(case, seed):
    """(reference, candidates) of a screening case."""
    g = _gen(seed)
    ref = _reference(case["data"], case["n"], case["cols"], DT[case["dtype"]], g)
    return ref, [_candidate(ref, case["data"], k, case["K"], case["cols"], g) for k in range(case["K"])]


def _multi_tensors(case, seed):
    g = _gen(seed)
    shape = (case["batch"], case["heads"], case["seq"])
    outs = [(shape + (case["dim"],), DT[case["dtype"]]), (shape, torch.float32)]
    refs = [_reference("attn", math.prod(s), case["dim"], t, g).view(s) for s, t in outs]
    cands = [[_candidate(r.view(-1), "attn", k, case["K"], case["dim"], g).view(r.shape) for r in refs]
             for k in range(case["K"])]
    return refs, cands


def _samples(case, seed):
    """Timing samples in us: base latencies that double from shape to shape,
    candidates up to 30 times slower than the best, 0.3% jitter, 3% spikes."""
    g = _gen(seed)
    C, S, N = case["C"], case["S"], case["iters"]
    f64 = dict(generator=g, dtype=torch.float64, device=DEV)
    mean = torch.exp(torch.rand(C, 1, 1, **f64) * math.log(30.0)) * (
        50.0 * 2.0 ** torch.arange(S, dtype=torch.float64, device=DEV).view(1, S, 1))
    t = 1.0 + torch.randn(C, S, N, **f64).abs_() * 0.003
    t += (torch.rand(C, S, N, **f64) < 0.03) * (0.02 + 0.23 * torch.rand(C, S, N, **f64))
    return (mean * t).contiguous()


def _record_views(buf, n):
    """The fields of n records in a uint8 buffer, as views."""
    i64, f64 = buf.view(torch.int64).view(n, 10), buf.view(torch.float64).view(n, 10)
    f32, i32 = buf.view(torch.float32).view(n, 20), buf.view(torch.int32).view(n, 20)
    return {"counts": i64[:, 0:5], "sum_sq_diff": f64[:, 5], "sum_sq_ref": f64[:, 6], "rel_l2": f64[:, 7],
            "max_abs_err": f32[:, 16], "max_rel_err": f32[:, 17], "flags": i32[:, 18:20]}


DIST = {"normal": (kb.KB_DIST_NORMAL, 0.0, 1.0), "uniform": (kb.KB_DIST_UNIFORM, -1.0, 1.0),
        "student_t3": (kb.KB_DIST_STUDENT_T3, 0.0, 1.0)}


def prepare(case, seed):
    torch.cuda.set_device(0)
    op = case["op"]
    if op == "screen":
        atol, rtol = TOL[case["data"]]
        ref, cands = _tensors(case, seed)
        s = kb.Screener(ref, cands, atol, rtol, positions=bool(case.get("positions")))
        out = _record_views(s.d_stats, case["K"])
        if case.get("positions"):
            out["positions"] = s.d_loc.view(torch.int64).view(case["K"], 4)[:, 0:3]
        return dict(case=case, screener=s, out=out)
    if op == "reject":
        atol, rtol = TOL[case["data"]]
        ref, cands = _tensors(case, seed)
        s = kb.Screener(ref, cands, atol, rtol, flags=kb.KB_FAIL_FAST, host_slots=1)
        recs = s.slots[0].numpy()
        return dict(case=case, screener=s, stream=torch.cuda.current_stream(),
                    i64=recs.view(np.int64).reshape(-1, 10), f64=recs.view(np.float64).reshape(-1, 10),
                    i32=recs.view(np.int32).reshape(-1, 20))
    if op == "multi":
        refs, cands = _multi_tensors(case, seed)
        s = kb.MultiScreener(refs, cands, [1e-3, 1e-5], [1e-3, 1e-5])
        return dict(case=case, screener=s, out=_record_views(s.d_stats, 2 * case["K"]))
    if op == "inputs":
        return dict(case=case, seed=seed,
                    out=[torch.empty(case["n"], dtype=DT[case["dtype"]], device=DEV) for _ in range(case["tensors"])])
    if op == "build":
        n, K, shape = case["n"], case["K"], (case["n"] // case["cols"], case["cols"])
        # one buffer, each tensor of it 16-byte aligned
        whole = torch.empty(K + 1, (n + 7) // 8 * 8, dtype=DT[case["dtype"]], device=DEV)[:, :n]
        return dict(case=case, seed=seed, tensors=[whole[k].view(shape) for k in range(K + 1)], out=whole)
    samples = _samples(case, seed)
    C, S = case["C"], case["S"]
    rows = torch.empty(C * S * 80, dtype=torch.uint8, device=DEV)
    scores = torch.empty(C * 32, dtype=torch.uint8, device=DEV)
    out = {"rows": rows.view(torch.float64).view(C * S, 10)[:, 0:9],
           "row_flags": rows.view(torch.int32).view(C * S, 20)[:, 18:20],
           "scores": scores.view(torch.float64).view(C, 4)[:, 0:3],
           "score_flags": scores.view(torch.int32).view(C, 8)[:, 6:8]}
    return dict(case=case, samples=samples, rows=rows, scores=scores, out=out)


# --------------------------------------------------------------------- run ---

def _build(case, seed, out):
    """The synthetic workload recipes: the reference from its stream, each
    candidate the reference with its planted change."""
    data, K, ref = case["data"], case["K"], out[0]
    if data == "heavy":
        kb.kb_gen_inputs(ref, kb.KB_DIST_STUDENT_T3, 0.0, 1.0, seed=seed, stream_id=0x500)
        kb.kb_gen_perturb(ref, ref, kb.KB_PERTURB_SPECIALS, 2.0 ** -10, 2.0 ** -9, 2.0 ** -9 + 2.0 ** -20, seed=seed,
                          stream_id=0x502)
    elif data == "softmax":
        kb.kb_gen_softmax_rows(ref, 2.0, seed=seed, stream_id=0x300)
    else:
        kb.kb_gen_inputs(ref, kb.KB_DIST_NORMAL, 0.0, 64.0 if data == "gemm" else 1.0, seed=seed, stream_id=0x200)
    for k in range(K):
        c = out[k + 1]
        if data == "heavy":
            kb.kb_gen_perturb(c, ref, kb.KB_PERTURB_ZERO_SUBNORMAL_REL, -1e-7, 1e-7, 0.5, seed=seed, stream_id=0x501,
                              sub=k)
        elif data == "softmax":
            kb.kb_gen_perturb(c, ref, kb.KB_PERTURB_ADD_NORMAL, 10.0 ** (-9.0 + 6.0 * k / max(1, K - 1)), seed=seed,
                              stream_id=0x301, sub=k)
        elif data == "gemm":
            s = 2.0 ** (-8.0 + 2.0 * (k % 16) / 15.0)
            kb.kb_gen_perturb(c, ref, kb.KB_PERTURB_REL_UNIFORM, -s, s, seed=seed, stream_id=0x201, sub=k)
        else:
            kb.kb_gen_perturb(c, ref, kb.KB_PERTURB_FLIP_LSB_WHERE, 0.0, 0.0, 0.001 if k % 2 else 0.0, seed=seed,
                              stream_id=0x202, sub=k)
            if k % 4 >= 2:
                idx = kb.kb_gen_indices(64, c.numel(), c.device, seed=seed, stream_id=0x203, sub=k)
                kb.kb_gen_scatter(c, ref, idx, kb.KB_SCATTER_INF_SIGN_OF_REF)


def run(state):
    case = state["case"]
    op = case["op"]
    if op == "screen":
        state["screener"].launch()
        if case.get("read"):
            state["screener"].read()
        return state["out"]
    if op == "reject":
        s = state["screener"]
        s.launch(0)
        state["stream"].synchronize()
        s.summarize(0)
        ok = (state["i32"][:, 19] == kb.KB_STATUS_OK) & (state["i64"][:, 1] == 0)
        return {"passed": ok.astype(np.int32), "status": state["i32"][:, 19].copy(),
                "sum_sq_diff": np.where(ok, state["f64"][:, 5], 0.0),
                "sum_sq_ref": np.where(ok, state["f64"][:, 6], 0.0)}
    if op == "multi":
        state["screener"].launch()
        return state["out"]
    if op == "inputs":
        dist, p0, p1 = DIST[case["dist"]]
        for i, t in enumerate(state["out"]):
            kb.kb_gen_inputs(t, dist, p0, p1, seed=state["seed"], stream_id=0x100, sub=i, offset=case["offset"])
        return state["out"]
    if op == "build":
        _build(case, state["seed"], state["tensors"])
        return state["out"]
    kb.kb_rung_stats(state["samples"], base=0, rung=case["rung"], budget=float(case["iters"]), rows=state["rows"],
                     scores=state["scores"])
    rank, order, promoted = kb.kb_rung_promote(state["scores"], case["C"])
    return dict(state["out"], rank=rank, order=order, promoted=promoted)


# --------------------------------------------------------- work, tolerance ---

def work(case):
    op = case["op"]
    if op in ("screen", "reject"):
        n, K, b = case["n"], case["K"], SIZE[case["dtype"]]
        if op == "reject":  # the candidates that fail need not be read
            fails = {"plain": (2, 3), "attn": (2, 3)}.get(case["data"], ())
            K = max(1, sum(1 for k in range(K) if k % 4 not in fails))
        # per element and candidate: difference, square and add, tolerance and relative tests, maxima
        return {"bytes": (K + 1) * n * b + 80 * case["K"], "flops": 6 * K * n}
    if op == "multi":
        rows = case["batch"] * case["heads"] * case["seq"]
        n, b = rows * case["dim"], SIZE[case["dtype"]]
        return {"bytes": (case["K"] + 1) * (n * b + rows * 4) + 160 * case["K"], "flops": 6 * case["K"] * (n + rows)}
    # transcendental steps of one value, in multiply-adds: a log, a root and a sine or cosine, shared by two normals
    per = {"normal": 80, "uniform": 2, "student_t3": 160}
    if op == "inputs":
        n = case["n"] * case["tensors"]
        return {"bytes": n * SIZE[case["dtype"]], "flops": n * per[case["dist"]]}
    if op == "build":
        n, K, b = case["n"], case["K"], SIZE[case["dtype"]]
        ref = {"heavy": 160, "softmax": 80 + 40}.get(case["data"], 80)
        each = 80 if case["data"] == "softmax" else 4
        return {"bytes": (K + 1) * n * b, "flops": n * (ref + K * each)}
    C, S, N = case["C"], case["S"], case["iters"]
    return {"bytes": 8 * C * S * N + 80 * C * S + 32 * C + 12 * C, "flops": C * S * N * 12}


def tolerance(case):
    op = case["op"]
    if op in ("screen", "reject", "multi"):
        # sums of squares: eight binary32 terms, then binary64 (1.5e-8 from the
        # 64-bit sums); maxima and counts are exact
        return {"rel": 1e-7, "max": 4e-7}
    if op == "rung":
        return "exact"
    # values rounded from binary64: now and then a rounding falls the other
    # way, and a logit's rounding moves its softmax row by up to 1e-6
    if case["dtype"] == "f32":
        return {"rel": 5e-7, "max": 4e-6} if case.get("data") == "softmax" else {"rel": 1e-7, "max": 5e-7}
    return {"rel": 1e-4, "max": 2e-3 if case["dtype"] == "f16" else 1.6e-2}


# ------------------------------------------------------------------- exact ---

def _exact_records(ref, cands):
    """The floating fields of the records in 64 bits (the counts, the flags
    and the positions have no such value)."""
    K, n = len(cands), ref.numel()
    f64 = dict(dtype=torch.float64, device=DEV)
    ssd, ssr, ma, mr = (torch.zeros(K, **f64) for _ in range(4))
    for a, b in _parts(n):
        r = ref[a:b].double()
        fin = torch.isfinite(r)
        ssr += torch.where(fin, r, 0.0).square().sum()
        for k, t in enumerate(cands):
            c = t[a:b].double()
            d = (c - r).abs()
            ssd[k] += torch.where(fin & torch.isfinite(c), d, 0.0).square().sum()
            ma[k] = torch.maximum(ma[k], torch.nan_to_num(d, nan=0.0, posinf=math.inf).max())
            mr[k] = torch.maximum(mr[k], torch.nan_to_num(d / r.abs(), nan=0.0, posinf=math.inf).max())
    return {"counts": None, "sum_sq_diff": ssd, "sum_sq_ref": ssr, "rel_l2": (ssd / ssr).sqrt(), "max_abs_err": ma,
            "max_rel_err": mr, "flags": None}


M32 = 0xFFFFFFFF


def _philox(b, seed, stream_id, sub):
    """The four words (int64 tensors) of Philox4x32-10 blocks b."""
    x0, x1 = b & M32, (b >> 32) & M32
    x2, x3 = torch.full_like(b, sub), torch.full_like(b, stream_id)
    k0, k1 = seed & M32, (seed >> 32) & M32
    for _ in range(10):
        p0, p1 = x0 * 0xD2511F53, x2 * 0xCD9E8D57
        x0, x1, x2, x3 = ((p1 >> 32) & M32) ^ x1 ^ k0, p1 & M32, ((p0 >> 32) & M32) ^ x3 ^ k1, p0 & M32
        k0, k1 = (k0 + 0x9E3779B9) & M32, (k1 + 0xBB67AE85) & M32
    return x0, x1, x2, x3


def _box_muller(xa, xb):
    rho = torch.sqrt(-2.0 * torch.log((xa.double() + 1.0) * 2.0 ** -32))
    theta = (2.0 * math.pi) * (xb.double() * 2.0 ** -32)
    return rho * torch.cos(theta), rho * torch.sin(theta)


def _u01(x):
    return (x >> 8).double() * 2.0 ** -24


def _stream(kind, n, seed, stream_id, sub, offset=0):
    """Elements offset .. offset + n - 1 of a stream in 64 bits: "normal",
    "uniform" (u in [0, 1)), "student_t3", or "words" (the four words of block
    g for element g)."""
    out = [torch.empty(n, dtype=torch.int64, device=DEV) for _ in range(4)] if kind == "words" else torch.empty(
        n, dtype=torch.float64, device=DEV)
    for a, b in _parts(n, 1 << 24):
        if kind in ("words", "student_t3"):
            w = _philox(torch.arange(offset + a, offset + b, device=DEV), seed, stream_id, sub)
            if kind == "words":
                for i in range(4):
                    out[i][a:b] = w[i]
            else:
                z0, z1 = _box_muller(w[0], w[1])
                z2, z3 = _box_muller(w[2], w[3])
                out[a:b] = z0 / torch.sqrt((z1 * z1 + z2 * z2 + z3 * z3) / 3.0)
            continue
        lo, hi = (offset + a) // 4, (offset + b + 3) // 4
        w = _philox(torch.arange(lo, hi, device=DEV), seed, stream_id, sub)
        v = [_u01(x) for x in w] if kind == "uniform" else [*_box_muller(w[0], w[1]), *_box_muller(w[2], w[3])]
        out[a:b] = torch.stack(v, 1).view(-1)[offset + a - 4 * lo:offset + b - 4 * lo]
    return out


def _f32(x):
    return float(np.float32(x))


def _exact_build(case, seed):
    data, n, K = case["data"], case["n"], case["K"]
    dt = DT[case["dtype"]]
    if data == "heavy":
        x = _stream("student_t3", n, seed, 0x500, 0)
        w = _stream("words", n, seed, 0x502, 0)
        v, sign = _u01(w[0]), 1.0 - 2.0 * (w[1] >> 31).double()
        x = torch.where(v < 2.0 ** -9 + 2.0 ** -20, sign * math.inf, x)
        x = torch.where(v < 2.0 ** -9, sign * 0.0, x)
        x = torch.where(v < 2.0 ** -10, sign * ((w[2] & 0x7FFFFF) | 1).double() * 2.0 ** -149, x)
    elif data == "softmax":
        x = torch.softmax(2.0 * _stream("normal", n, seed, 0x300, 0).view(-1, case["cols"]), dim=1).view(-1)
    else:
        x = _stream("normal", n, seed, 0x200, 0) * (64.0 if data == "gemm" else 1.0)
    out = [x]
    x = x.to(dt).double()  # the candidates start from the stored reference
    for k in range(K):
        if data == "heavy":
            w = _stream("words", n, seed, 0x501, k)
            e = _f32(-1e-7) + _u01(w[1]) * (2.0 * _f32(1e-7))
            y = torch.where(x == 0.0, -x, torch.where(x.abs() < 2.0 ** -126, x * 0.0, x * (1.0 + e)))
            y = torch.where(torch.isinf(x), x, y)
            y = torch.where(_u01(w[0]) < 0.5, y, x)
        elif data == "softmax":
            y = x + _stream("normal", n, seed, 0x301, k) * _f32(10.0 ** (-9.0 + 6.0 * k / max(1, K - 1)))
        elif data == "gemm":
            s = _f32(2.0 ** (-8.0 + 2.0 * (k % 16) / 15.0))
            y = x * (1.0 + (_stream("uniform", n, seed, 0x201, k) * (2.0 * s) - s))
        else:
            hit = _stream("uniform", n, seed, 0x202, k) < (_f32(0.001) if k % 2 else 0.0)
            b = x.to(dt).view(torch.int32 if dt == torch.float32 else torch.int16)
            y = (b ^ hit.to(b.dtype)).view(dt).double()
            if k % 4 >= 2:
                i = _drawn(64, n, seed, 0x203, k)
                y[i] = torch.copysign(torch.full_like(y[i], math.inf), x[i])
        out.append(y)
    return torch.stack(out)


def _drawn(m, n, seed, stream_id, sub):
    """The first m distinct draws ((w1 << 32) | w0) mod n."""
    w0, w1, _, _ = (t.tolist() for t in _philox(torch.arange(4 * m + 64, device=DEV), seed, stream_id, sub))
    got = list(dict.fromkeys(((b << 32) | a) % n for a, b in zip(w0, w1)))[:m]
    return torch.tensor(got, device=DEV)


def exact(case, seed):
    torch.cuda.set_device(0)
    op = case["op"]
    if op in ("screen", "reject"):
        ref, cands = _tensors(case, seed)
        out = _exact_records(ref, cands)
        if op == "screen":
            return dict(out, positions=None) if case.get("positions") else out
        atol, rtol = TOL[case["data"]]
        ok = torch.ones(len(cands), dtype=torch.bool)
        for k, c in enumerate(cands):
            for a, b in _parts(ref.numel()):
                r, x = ref[a:b].float(), c[a:b].float()
                tol = torch.where(torch.isfinite(r), atol + rtol * r.abs(), -1.0)
                if not bool(((x == r) | ((x - r).abs() <= tol)).all()):
                    ok[k] = False
        ok = ok.to(DEV)
        return {"passed": None, "status": None, "sum_sq_diff": torch.where(ok, out["sum_sq_diff"], 0.0),
                "sum_sq_ref": torch.where(ok, out["sum_sq_ref"], 0.0)}
    if op == "multi":
        refs, cands = _multi_tensors(case, seed)
        per = [_exact_records(r.view(-1), [c[o].view(-1) for c in cands]) for o, r in enumerate(refs)]
        return {f: None if per[0][f] is None else torch.cat([per[0][f], per[1][f]]) for f in per[0]}
    if op == "inputs":
        scale, shift = (2.0, -1.0) if case["dist"] == "uniform" else (1.0, 0.0)
        if case["n"] * case["tensors"] > 1 << 29:
            return None
        return [_stream(case["dist"], case["n"], seed, 0x100, i, case["offset"]) * scale + shift
                for i in range(case["tensors"])]
    if op == "build":
        if case["n"] * (case["K"] + 1) > 1 << 29:
            return None
        return _exact_build(case, seed)
    t = _samples(case, seed)
    C, S, N = t.shape
    mean = t.mean(2)
    q = torch.quantile(t, torch.tensor([0.5, 0.9, 0.95, 0.99], dtype=torch.float64, device=DEV), dim=2)
    rows = torch.stack([mean, *q, q[1] / q[0], q[2] / q[0], q[3] / q[0], mean[0] / mean], 2).view(C * S, 9)
    lat = mean.mean(1)
    score = 1e6 / lat.clamp(min=1.0) + (kb.RUNG_ALPHA * case["rung"] + kb.RUNG_BETA * case["iters"])
    return {"rows": rows, "row_flags": None, "scores": torch.stack([lat, score, lat[0] / lat], 1), "score_flags": None,
            "rank": None, "order": None, "promoted": None}
