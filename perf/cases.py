"""What this framework is timed on: the calls of a decode step, one at a time.

A decode step is lane attention (lane_attn_forward), the fused LM head with
confidence (lmhead_confidence and, on a weight repacked once at load time,
lmhead_confidence_packed) and the selection (select_unmask).  The listed
cases are those calls at the shapes of the synthetic workloads "tiny",
"llada", "dream", "long" and "wide" (the LLaDA-8B and Dream-7B backbones at
growing lane counts and prefixes) plus the compact-refresh forward over an odd
window; draw() gives other sizes of the same ranges.
"""
import math

import numpy as np
import torch

import paper_2606_08411_amd as al

EOS_ID = 2
DELIM_IDS = (0, 1)


# ------------------------------------------------------------------- cases
def _attn(name, L, B, P, Hq, Hkv, D, tree, depth, n_ref=0):
    return dict(name=name, kind="attn", L=L, B=B, P=P, Hq=Hq, Hkv=Hkv, D=D, tree=tree,
                depth=depth, n_ref=n_ref)


def _lm(name, N, n_rows, d, V, packed):
    return dict(name=name, kind="lmhead", N=N, n_rows=n_rows, d=d, V=V, packed=packed)


def listed():
    return [
        # The smallest step: two lanes, four heads of 64.  Latency and launches.
        _attn("attn_tiny", 2, 32, 128, 4, 4, 64, "random", 1),
        # One layer of an LLaDA-8B decode step: a chain of 4 lanes on a short prompt.
        _attn("attn_llada", 4, 32, 512, 32, 32, 128, "linear", 3),
        # One layer of a Dream-7B decode step: grouped queries (28 heads on 4).
        _attn("attn_dream", 8, 32, 1024, 28, 4, 128, "random", 3),
        # Long generation: 16 lanes over 2048 cached rows.
        _attn("attn_long", 16, 32, 2048, 32, 32, 128, "random", 6),
        # Many lanes, long prefix, and a tenth of the prefix refreshed in the same call.
        _attn("attn_wide", 32, 64, 4096, 32, 32, 128, "random", 8, 410),
        # Compact-refresh forward: every row of an odd window, no lanes (the prefill direction).
        _attn("attn_window", 0, 16, 2563, 32, 32, 128, "random", 0, 2563),
        # A small head as small models and tests have it: latency and launches.
        _lm("lm_tiny", 32, 64, 256, 1024, False),
        # LLaDA-8B head, 77 masked rows, weight packed at load time (the usual decode step).
        _lm("lm_llada", 77, 128, 4096, 126464, True),
        # Dream-7B head, 128 masked rows, packed.
        _lm("lm_dream", 128, 256, 3584, 152064, True),
        # LLaDA-8B head on the weight as the model holds it (no second copy), 205 masked rows.
        _lm("lm_long", 205, 512, 4096, 126464, False),
        # LLaDA-8B head, 614 masked rows, packed: many lanes of one batch.
        _lm("lm_wide", 614, 2048, 4096, 126464, True),
        # Selection over 16 lanes of 32 with lookahead drafts and the boundary rules.
        dict(name="select_long", kind="select", L=16, B=32, N=205, topk=False),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    most = [work(c)["flops"] for c in listed() if c["name"] in ("attn_wide", "lm_wide")]
    while True:
        kind = rng.choice(["attn", "attn", "lmhead", "lmhead", "window", "select"])
        if kind == "attn":
            Hkv, g = rng.choice([(4, 1), (8, 1), (32, 1), (8, 4), (4, 7)])
            P = _log_int(rng, 65, 4096)
            c = dict(kind="attn", L=_log_int(rng, 1, 32), B=rng.choice([16, 32, 32, 48, 64]), P=P,
                     Hq=Hkv * g, Hkv=Hkv, D=rng.choice([64, 128, 128]),
                     tree=rng.choice(["linear", "random", "random"]), depth=rng.randint(1, 8),
                     n_ref=rng.choice([0, 0, P // 10]))
            if work(c)["flops"] <= most[0]:
                return c
        elif kind == "window":
            P = _log_int(rng, 200, 2563)
            Hkv, g = rng.choice([(8, 1), (32, 1), (4, 7)])
            return dict(kind="attn", L=0, B=16, P=P, Hq=Hkv * g, Hkv=Hkv,
                        D=rng.choice([64, 128]), tree="random", depth=0, n_ref=P)
        elif kind == "lmhead":
            N = _log_int(rng, 1, 614)
            d, V = rng.choice([(4096, 126464), (3584, 152064), (4096, _log_int(rng, 1000, 126464)),
                               (8 * _log_int(rng, 32, 512), _log_int(rng, 1000, 126464))])
            c = dict(kind="lmhead", N=N, n_rows=N + rng.randint(0, 2 * N), d=d, V=V,
                     packed=rng.choice([True, True, False]))
            if work(c)["flops"] <= most[1] * (1.0 if c["packed"] else 0.75):
                return c
        else:
            L, B = _log_int(rng, 1, 32), rng.choice([16, 32, 48, 64])
            return dict(kind="select", L=L, B=B, N=rng.randint(1, L * B), topk=rng.random() < 0.4)


# ------------------------------------------------------------------ inputs
def _gen(seed, stream):
    g = torch.Generator(device="cuda")
    g.manual_seed(1000003 * int(seed) + stream)
    return g


def _normal(seed, stream, shape, std=1.0):
    n = math.prod(shape)
    out = torch.empty(n, dtype=torch.bfloat16, device="cuda")
    g = _gen(seed, stream)
    for i in range(0, n, 1 << 26):   # in pieces: the fp32 draws of a whole weight would be 2 GB
        m = min(1 << 26, n - i)
        out[i:i + m] = torch.randn(m, generator=g, device="cuda") * std
    return out.view(shape)


def _tree(case):
    """Lane tree, parent[i] in [-1, i): a chain, or random forks up to a depth (one tree a case:
    what the call has to do depends on it)."""
    L = case["L"]
    rng = np.random.default_rng([L, case["depth"], 71])
    parent = np.full(L, -1, np.int32)
    depth = np.zeros(L, np.int64)
    for i in range(1, L):
        j = i - 1 if case["tree"] == "linear" else int(
            rng.choice(np.nonzero(depth[:i] < max(1, case["depth"]))[0]))
        parent[i] = j
        depth[i] = depth[j] + 1
    return parent


def prepare(case, seed):
    rng = np.random.default_rng([int(seed), 77])
    if case["kind"] == "attn":
        L, B, P, Hq, Hkv, D = (case[k] for k in ("L", "B", "P", "Hq", "Hkv", "D"))
        R, n_ref = L * B, case["n_ref"]
        s = dict(parent=_tree(case), B=B,
                 k_prefix=_normal(seed, 1, (P, Hkv, D)), v_prefix=_normal(seed, 2, (P, Hkv, D)))
        if L:
            s.update(q=_normal(seed, 3, (R, Hq, D)), k_lane=_normal(seed, 4, (R, Hkv, D)),
                     v_lane=_normal(seed, 5, (R, Hkv, D)))
        else:
            s.update(q=None, k_lane=None, v_lane=None)
        if n_ref:
            idx = np.sort(rng.choice(P, n_ref, replace=False)).astype(np.int32)
            s.update(refresh_idx=torch.from_numpy(idx).cuda(), q_ref=_normal(seed, 6, (n_ref, Hq, D)),
                     k_ref=_normal(seed, 7, (n_ref, Hkv, D)), v_ref=_normal(seed, 8, (n_ref, Hkv, D)))
        return dict(case=case, args=s)
    if case["kind"] == "lmhead":
        N, n_rows, d, V = (case[k] for k in ("N", "n_rows", "d", "V"))
        # Per-row logit scale U[1, 6], so confidences range from flat to near 1.
        scale = 1.0 + 5.0 * torch.rand((n_rows, 1), generator=_gen(seed, 11), device="cuda")
        hidden = (_normal(seed, 9, (n_rows, d)).float() * scale).to(torch.bfloat16)
        W = _normal(seed, 10, (V, d), 1.0 / math.sqrt(d))
        rows = np.sort(rng.choice(n_rows, N, replace=False)).astype(np.int32)
        s = dict(case=case, hidden=hidden, row_idx=torch.from_numpy(rows).cuda(),
                 sup=torch.from_numpy(rng.integers(0, 2, N).astype(np.uint8)).cuda())
        s["W"] = al.lmhead_pack_weight(W) if case["packed"] else W
        return s
    L, B, N = case["L"], case["B"], case["N"]
    LB = L * B
    pos = np.sort(rng.choice(LB, N, replace=False)).astype(np.int32)
    masked = np.zeros(LB, np.uint8)
    masked[pos] = 1
    tokens = rng.integers(3, 126464, LB).astype(np.int32)
    delim = rng.random(LB) < 0.05
    tokens[delim] = rng.integers(0, 2, int(delim.sum()))
    tokens[masked == 1] = -1
    # The step's blocks as the host lays them out: tokens, then mask flags, in one buffer.
    blocks = torch.from_numpy(np.concatenate([tokens.view(np.uint8), masked])).cuda()
    work_buf = torch.empty_like(blocks)
    # Result buffers that a decode loop keeps from step to step.
    out = dict(unmask_flag=torch.zeros(N, dtype=torch.uint8, device="cuda"),
               unmasked_pos=torch.zeros(N, dtype=torch.int32, device="cuda"),
               still_masked_pos=torch.zeros(N, dtype=torch.int32, device="cuda"),
               counts=torch.zeros(2, dtype=torch.int32, device="cuda"),
               lane_stats=torch.zeros((L, 6), dtype=torch.int32, device="cuda"),
               delim_flag=torch.zeros(LB, dtype=torch.uint8, device="cuda"))
    return dict(case=case, out=out, blocks=blocks, buf=work_buf, tokens=work_buf[:4 * LB].view(torch.int32),
                masked=work_buf[4 * LB:], row_pos=torch.from_numpy(pos).cuda(),
                conf=torch.from_numpy(rng.random(N).astype(np.float32) ** 0.25).cuda(),
                argmax=torch.from_numpy(rng.integers(0, 126464, N).astype(np.int32)).cuda(),
                role=rng.integers(0, 2, L).astype(np.uint8),
                b_len=np.maximum(1, B - rng.integers(0, B // 2, L)).astype(np.int32),
                t_lane=rng.integers(0, 8, L).astype(np.int32),
                k_lane=rng.integers(0, 5, L).astype(np.int32) if case["topk"] else None)


# -------------------------------------------------------------------- runs
def run(state):
    case = state["case"]
    if case["kind"] == "attn":
        o, lse, o_ref, lse_ref = al.lane_attn_forward(**state["args"])
        out = dict(o=o, lse=lse, o_ref=o_ref, lse_ref=lse_ref)
        if case["n_ref"]:
            out.update(k_prefix=state["args"]["k_prefix"], v_prefix=state["args"]["v_prefix"])
        return out
    if case["kind"] == "lmhead":
        if case["packed"]:
            conf, arg, lse = al.lmhead_confidence_packed(
                state["hidden"], state["W"], case["V"], row_idx=state["row_idx"],
                suppress_eos=state["sup"], eos_id=EOS_ID)
        else:
            conf, arg, lse = al.lmhead_confidence(
                state["hidden"], state["W"], row_idx=state["row_idx"],
                suppress_eos=state["sup"], eos_id=EOS_ID)
        return dict(conf=conf, argmax=arg, lse=lse)
    # Each step brings its blocks anew (one copy), and selection updates them in place.
    state["buf"].copy_(state["blocks"])
    out = al.select_unmask(
        state["conf"], state["argmax"], state["row_pos"], state["tokens"], state["masked"],
        case["L"], case["B"], state["role"], state["b_len"], state["t_lane"],
        mode=al.MODE_TOPK if case["topk"] else al.MODE_THRESHOLD, tau=0.9, fallback_k=1,
        k_lane=state["k_lane"], delim_ids=DELIM_IDS, eos_id=EOS_ID, tau_future=0.95,
        digit_ids=tuple(range(20, 30)), open_ids=(40, 41, 42), close_ids=(43, 44, 45),
        out=state["out"])
    return dict(out, tokens=state["tokens"], masked=state["masked"])


# ------------------------------------------------- work, tolerance, 64 bits
def _depths(case):
    """How many lanes each lane sees: itself and its ancestors."""
    parent = _tree(case)
    n = np.ones(len(parent), np.int64)
    for i, p in enumerate(parent):
        if p >= 0:
            n[i] = n[p] + 1
    return n


def work(case):
    if case["kind"] == "attn":
        L, B, P, Hq, Hkv, D, n_ref = (case[k] for k in ("L", "B", "P", "Hq", "Hkv", "D", "n_ref"))
        keys = sum(B * (P + B * int(n)) for n in _depths(case)) + n_ref * P
        rows = L * B + n_ref
        # q in, o and lse out; the prefix, lane and refreshed K/V rows in (a refreshed prefix row
        # is written, not read).
        move = rows * Hq * (4 * D + 4) + 4 * Hkv * D * (P - n_ref + L * B + 2 * n_ref)
        return dict(bytes=move, flops=4.0 * Hq * D * keys)
    if case["kind"] == "lmhead":
        N, d, V = case["N"], case["d"], case["V"]
        return dict(bytes=2.0 * V * d + 2.0 * N * d + 17.0 * N, flops=2.0 * N * V * d)
    LB, N = case["L"] * case["B"], case["N"]
    return dict(bytes=10.0 * LB + 17.0 * N + 37.0 * case["L"], flops=0)


def tolerance(case):
    """About four times what the calls are off by against exact(), over the listed cases and
    draws of the same ranges: attention 2.0e-3 to 2.9e-3 (probabilities and outputs in bf16),
    largest single value 1.8e-2; the head 0.4e-6 to 4.6e-6 (fp32 sums of up to 4096 products,
    then an exponential), largest 1.9e-5.  A near-tie of two logits may change an argmax."""
    if case["kind"] == "attn":
        return {"rel": 1e-2, "max": 8e-2}
    if case["kind"] == "lmhead":
        return {"rel": 2e-5, "max": 8e-5, "differ": 0.005}
    return "exact"


def _exact_attention(q, k, v, visible, scale):
    """softmax(q k^T scale) v in 64 bits, head by head; visible [rows][keys] or None."""
    Hq, g = q.shape[1], q.shape[1] // k.shape[1]
    o = torch.empty(q.shape, dtype=torch.float64, device=q.device)
    lse = torch.empty(q.shape[:2], dtype=torch.float64, device=q.device)
    for h in range(Hq):
        kh, vh = k[:, h // g].double().contiguous(), v[:, h // g].double().contiguous()
        z = torch.mm(q[:, h].double().contiguous(), kh.t().contiguous()) * scale
        if visible is not None:
            z.masked_fill_(~visible, -math.inf)
        lse[:, h] = torch.logsumexp(z, dim=1)
        o[:, h] = torch.mm(torch.exp(z - lse[:, h:h + 1]), vh)
    return o, lse


def exact(case, seed):
    if case["kind"] == "select":
        return None   # whole numbers and flags: nothing is computed in floating point
    if case["kind"] == "attn":
        a = prepare(case, seed)["args"]
        L, B, P, scale = case["L"], case["B"], case["P"], 1.0 / math.sqrt(case["D"])
        k, v = a["k_prefix"].clone(), a["v_prefix"].clone()
        if case["n_ref"]:
            k[a["refresh_idx"].long()] = a["k_ref"]
            v[a["refresh_idx"].long()] = a["v_ref"]
        out = dict(o=None, lse=None, o_ref=None, lse_ref=None)
        if L:
            see = torch.eye(L, dtype=torch.bool)
            for i, p in enumerate(a["parent"]):
                if p >= 0:
                    see[i] |= see[int(p)]
            lanes = see.repeat_interleave(B, 0).repeat_interleave(B, 1).cuda()
            visible = torch.cat([torch.ones((L * B, P), dtype=torch.bool, device="cuda"), lanes], 1)
            out["o"], out["lse"] = _exact_attention(a["q"], torch.cat([k, a["k_lane"]]),
                                                    torch.cat([v, a["v_lane"]]), visible, scale)
        if case["n_ref"]:
            out["o_ref"], out["lse_ref"] = _exact_attention(a["q_ref"], k, v, None, scale)
            out.update(k_prefix=k, v_prefix=v)
        return out
    s = prepare(dict(case, packed=False), seed)
    h = s["hidden"][s["row_idx"].long()].double()
    z = torch.cat([torch.mm(h, w.double().t().contiguous()) for w in s["W"].split(16384)], dim=1)
    z[s["sup"].bool(), EOS_ID] = -math.inf
    top, arg = z.max(dim=1)
    lse = torch.logsumexp(z, dim=1)
    return dict(conf=torch.exp(top - lse), argmax=arg.to(torch.int32), lse=lse)
