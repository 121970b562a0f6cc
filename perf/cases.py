"""The attention work that a user of this library has it do, as timed cases.

A case is one pass through the public entry points of
paper_2511_13198_amd.pdyattn: a training step of the packed attention
(attn_fwd, then attn_bwd), a forward alone, or one ring step of a
context-parallel device (two partial forwards, their merge, two accumulating
backwards).  Inputs are N(0,1) bf16, as the workloads of this package draw
them; outputs and workspaces are kept over the passes, as a training loop
keeps them, except where a case says that each call allocates its own.

The range: 512 to 638,976 tokens; single sequences, packed batches of long,
short and equal segments, chunk pairs; head dimensions 64 and 128; one to 32
query heads, grouped or not; causal and not.
"""
import math

import numpy as np
import torch

from paper_2511_13198_amd import pdyattn
from paper_2511_13198_amd import workloads as wl


def listed():
    return [
        # the smallest layer of the package's workloads: one 512-token
        # sequence, 8 heads of 64; launches and host work
        _step("step_512_h8_d64", "single", 512, 8, 8, 64, fresh=True),
        # an odd short sequence, three query heads per key head
        _step("step_2500_h6kv2", "single", 2500, 6, 2, 128),
        # one device's 4 heads of a 32-head layer at short and middle lengths
        _step("step_4096_h4", "single", 4096, 4, 4, 128),
        _step("step_16384_h4", "single", 16384, 4, 4, 128),
        # an encoder batch: 32 sequences of 512 tokens, 16 heads of 64, no mask
        _step("step_32x512_h16_d64_full", "equal", 32 * 512, 16, 16, 64, lo=512, hi=512,
              causal=False),
        # a batch of very short samples packed together, grouped heads
        _step("step_packed16384_short_h32kv8", "loguniform", 16384, 32, 8, 128, lo=16, hi=512),
        # the packed batch of the package's workloads: 25 segments of 167 to
        # 7,402 tokens, 32 heads
        _step("step_packed65536_h32", "loguniform", 65536, 32, 32, 128, lo=128, hi=8192),
        # one batch of the long-tailed stream: 53 segments of 258 to 32,746
        # tokens, 32 query heads over 8 key heads
        _step("step_stream262144_h32kv8", "stream", 262144, 32, 8, 128, lo=64, hi=638976, lseed=2),
        # long sequence, heads of 64
        _step("step_65536_h8_d64", "single", 65536, 8, 8, 64),
        # a ring step of context parallelism: 131,072 tokens over 8 devices,
        # a device's 16,384 queries over its own and a visiting earlier chunk
        {"name": "ring_16384_h4", "kind": "ring", "rows": 16384, "q_offset": 65536,
         "visit_rows": 16384, "visit_offset": 16384, "hq": 4, "hkv": 4, "d": 128, "causal": True},
        # the headline length: 131,072 tokens, one device's 4 heads
        _step("step_131072_h4", "single", 131072, 4, 4, 128),
        # the longest sequence ("624K"), evaluation: forward alone, one head
        dict(_step("fwd_638976_h1", "single", 638976, 1, 1, 128), kind="fwd"),
    ]


def _step(name, pattern, tokens, hq, hkv, d, lo=0, hi=0, causal=True, lseed=42, fresh=False):
    """fresh: every call allocates its outputs and workspace, as in a first
    script; otherwise they are kept."""
    return {"name": name, "kind": "step", "pattern": pattern, "tokens": tokens, "hq": hq,
            "hkv": hkv, "d": d, "lo": lo, "hi": hi, "causal": causal, "lseed": lseed,
            "fresh": fresh}


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A case of the same ranges, at most about a sixth of the largest listed
    one's cost."""
    while True:
        d = rng.choice([64, 128, 128])
        hkv = rng.choice([1, 2, 3, 4, 8, 16])
        group = rng.choice([1, 1, 1, 2, 3, 4])
        causal = rng.random() < 0.85
        what = rng.choice(["single", "single", "packed", "packed", "ring"])
        if what == "ring":
            rows = _log_int(rng, 500, 32768)
            visit = rows + rng.choice([0, 0, -1, 1])
            off = rng.randrange(rows, 8 * rows)
            case = {"kind": "ring", "rows": rows, "q_offset": off, "visit_rows": visit,
                    "visit_offset": rng.randrange(0, max(0, off - visit) + 1), "hq": hkv * group, "hkv": hkv, "d": d,
                    "causal": causal}
        else:
            tokens = _log_int(rng, 512, 131072)
            if rng.random() < 0.3:
                tokens = 1 << max(9, tokens.bit_length() - 1)
            pattern, lo, hi = "single", 0, 0
            if what == "packed":
                pattern = rng.choice(["loguniform", "loguniform", "equal"])
                hi = _log_int(rng, 64, min(8192, tokens))
                lo = hi if pattern == "equal" else max(16, hi // rng.choice([8, 32, 64]))
                lo = min(lo, hi)
            case = _step("", pattern, tokens, hkv * group, hkv, d, lo=lo, hi=hi, causal=causal,
                         lseed=rng.randrange(1 << 20), fresh=rng.random() < 0.3)
            del case["name"]
            if rng.random() < 0.2:
                case["kind"] = "fwd"
        if work(case)["flops"] <= 4e13 and case["hq"] * _tokens(case) <= 4 << 20:
            return case


def _tokens(case):
    return case["tokens"] if case["kind"] != "ring" else case["rows"] + case["visit_rows"]


def _lengths(case):
    """The segment lengths of a step or forward, by its pattern."""
    total = case["tokens"]
    if case["pattern"] == "single":
        return [total]
    if case["pattern"] == "loguniform":
        return wl.loguniform_lengths(total, case["lo"], case["hi"], case["lseed"])
    if case["pattern"] == "stream":
        batch = wl.lognormal_stream(case["lseed"] + 1, lo=case["lo"], hi=case["hi"])[case["lseed"]]
        assert sum(batch) == total
        return batch
    n = total // case["hi"]
    rest = total - n * case["hi"]
    return [case["hi"]] * n + ([rest] if rest else [])


def _pairs(rows, q_offset, keys, k_offset, causal):
    """Visible (query, key) pairs of one chunk pair."""
    if not causal:
        return rows * keys
    i = np.arange(rows, dtype=np.int64) + (q_offset - k_offset + 1)
    return int(np.clip(i, 0, keys).sum())


def work(case):
    hq, hkv, d = case["hq"], case["hkv"], case["d"]
    if case["kind"] == "ring":
        t, v = case["rows"], case["visit_rows"]
        pairs = (_pairs(t, 0, t, 0, case["causal"]) +
                 _pairs(t, case["q_offset"], v, case["visit_offset"], case["causal"]))
        keys = t + v
        # q, dout, o (bf16), k, v once; o, lse, dq out; dk, dv of both chunks
        # out, those of the visiting one in
        nbytes = (2 * t * hq * d * 3 + 4 * t * hq + 4 * t * hq * d + 4 * keys * hkv * d +
                  8 * keys * hkv * d + 8 * v * hkv * d)
        return {"bytes": nbytes, "flops": 14 * d * hq * pairs}
    t = case["tokens"]
    lens = _lengths(case)
    pairs = sum(n * (n + 1) // 2 if case["causal"] else n * n for n in lens)
    fwd = 2 * t * d * (2 * hq + 2 * hkv) + 4 * t * hq
    if case["kind"] == "fwd":
        return {"bytes": fwd, "flops": 4 * d * hq * pairs}
    # a step: q, k, v, dout in; o, lse, dq, dk, dv out
    return {"bytes": fwd + 2 * t * d * hq + 4 * t * d * (hq + 2 * hkv),
            "flops": 14 * d * hq * pairs}


def _inputs(case, seed):
    """bf16 q, k, v, do (N(0,1)); for a ring step also the visiting chunk's
    k2, v2 and the gradient sums dk2, dv2 that arrive with it."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    hq, hkv, d = case["hq"], case["hkv"], case["d"]

    def normal(n, h):
        return torch.randn((n, h, d), generator=g, dtype=torch.float32,
                           device="cuda").to(torch.bfloat16)

    t = case["rows"] if case["kind"] == "ring" else case["tokens"]
    x = {"q": normal(t, hq), "k": normal(t, hkv), "v": normal(t, hkv)}
    if case["kind"] != "fwd":
        x["do"] = normal(t, hq)
    if case["kind"] == "ring":
        n = case["visit_rows"]
        x["k2"], x["v2"] = normal(n, hkv), normal(n, hkv)
        for name in ("dk2", "dv2"):
            x[name] = torch.randn((n, hkv, d), generator=g, dtype=torch.float32, device="cuda")
    return x


def prepare(case, seed):
    x = _inputs(case, seed)
    hq, hkv, d = case["hq"], case["hkv"], case["d"]
    q, k = x["q"], x["k"]
    t = q.shape[0]

    def f32(*shape):
        return torch.empty(shape, dtype=torch.float32, device="cuda")

    def scratch(n):
        return torch.empty(max(256, n), dtype=torch.uint8, device="cuda")

    s = {"case": case, "scale": 1.0 / math.sqrt(d), **x}
    if case["kind"] == "ring":
        n = case["visit_rows"]
        s.update(o=torch.empty_like(q), lse=f32(hq, t), o2=torch.empty_like(q), lse2=f32(hq, t),
                 dq=f32(t, hq, d), dk=f32(t, hkv, d), dv=f32(t, hkv, d),
                 sum_k=f32(n, hkv, d), sum_v=f32(n, hkv, d))
        m = max(n, t)
        s["ws"] = scratch(max(pdyattn.fwd_chunk_workspace_size(t, m, hq, hkv, d),
                              pdyattn.bwd_chunk_workspace_size(t, m, hq, hkv, d)))
        return s
    lens = _lengths(case)
    s["cu"] = torch.from_numpy(wl.cu_from_lengths(lens)).cuda()
    s["max"] = max(lens)
    if not case["fresh"]:
        s.update(o=torch.empty_like(q), lse=f32(hq, t))
        s["ws_f"] = scratch(pdyattn.fwd_workspace_size(t, len(lens), s["max"], hq, hkv, d))
        if case["kind"] == "step":
            s.update(dq=f32(t, hq, d), dk=f32(t, hkv, d), dv=f32(t, hkv, d))
            s["ws_b"] = scratch(pdyattn.bwd_workspace_size(t, len(lens), s["max"], hq, hkv, d))
    return s


def run(s):
    case = s["case"]
    causal, scale = case["causal"], s["scale"]
    if case["kind"] == "ring":
        return _run_ring(s)
    if case["fresh"]:
        o, lse = pdyattn.attn_fwd(s["q"], s["k"], s["v"], s["cu"], s["max"], causal, scale)
        if case["kind"] == "fwd":
            return {"o": o, "lse": lse}
        dq, dk, dv = pdyattn.attn_bwd(s["q"], s["k"], s["v"], o, lse, s["do"], s["cu"], s["max"],
                                      causal, scale)
        return {"o": o, "lse": lse, "dq": dq, "dk": dk, "dv": dv}
    o, lse = pdyattn.attn_fwd(s["q"], s["k"], s["v"], s["cu"], s["max"], causal, scale,
                              out=s["o"], lse=s["lse"], workspace=s["ws_f"])
    if case["kind"] == "fwd":
        return {"o": o, "lse": lse}
    dq, dk, dv = pdyattn.attn_bwd(s["q"], s["k"], s["v"], o, lse, s["do"], s["cu"], s["max"],
                                  causal, scale, dq=s["dq"], dk=s["dk"], dv=s["dv"],
                                  workspace=s["ws_b"])
    return {"o": o, "lse": lse, "dq": dq, "dk": dk, "dv": dv}


def _run_ring(s):
    """A device's own chunk and one visiting chunk: forward, merge, backward.
    The visiting chunk's gradient sums arrive in dk2, dv2 and leave with this
    device's part added."""
    case = s["case"]
    causal, scale, ws = case["causal"], s["scale"], s["ws"]
    qo, ko = case["q_offset"], case["visit_offset"]
    q, o, lse = s["q"], s["o"], s["lse"]
    pdyattn.attn_fwd_chunk(q, s["k"], s["v"], qo, qo, causal, scale, out=o, lse=lse, workspace=ws)
    pdyattn.attn_fwd_chunk(q, s["k2"], s["v2"], qo, ko, causal, scale, out=s["o2"],
                           lse=s["lse2"], workspace=ws)
    pdyattn.attn_merge(o, lse, s["o2"], s["lse2"], out=o, lse=lse)
    pdyattn.attn_bwd_chunk(q, s["k"], s["v"], o, lse, s["do"], qo, qo, causal, scale,
                           dq=s["dq"], dk=s["dk"], dv=s["dv"], workspace=ws)
    # the sums that arrive (the pass can be run again on the same state)
    s["sum_k"].copy_(s["dk2"])
    s["sum_v"].copy_(s["dv2"])
    pdyattn.attn_bwd_chunk(q, s["k2"], s["v2"], o, lse, s["do"], qo, ko, causal, scale,
                           dq=s["dq"], dk=s["sum_k"], dv=s["sum_v"], workspace=ws,
                           accumulate=True)
    return {"o": o, "lse": lse, "dq": s["dq"], "dk": s["dk"], "dv": s["dv"],
            "sum_k": s["sum_k"], "sum_v": s["sum_v"]}


def tolerance(case):
    """Probabilities, dS and O are rounded to bf16 (2^-9 relative each), sums
    are 32-bit: against 64 bits every output is 1.5e-3 to 3e-3 off in the
    2-norm.  Two such results that round in another order differ by about as
    much; four times that.  The largest differences, against the root mean
    square, are in the rows (and keys) next to a segment's start: they average
    few terms, so their values and errors are the largest by far, up to 0.27
    against 64 bits in a long sequence; three times that."""
    return {"rel": 1e-2, "max": 0.8}


def _attend(q, k, v, do, mask_from, scale, blocks=2048):
    """64-bit attention of one head: rows q over keys k, v; row i sees the keys
    j < mask_from[i].  Returns o, lse, dq, dk, dv (gradients None without do)."""
    n, m = q.shape[0], k.shape[0]
    o = torch.empty_like(q)
    lse = torch.empty(n, dtype=torch.float64, device=q.device)
    dq = torch.empty_like(q)
    dk, dv = torch.zeros_like(k), torch.zeros_like(v)
    j = torch.arange(m, device=q.device)
    for a in range(0, n, blocks):
        b = min(n, a + blocks)
        end = int(mask_from[a:b].max())
        keys, vals = k[:end], v[:end]
        p = q[a:b] @ keys.T
        p *= scale
        p.masked_fill_(j[None, :end] >= mask_from[a:b, None], -math.inf)
        lse[a:b] = torch.logsumexp(p, 1)
        p -= lse[a:b, None]
        p.exp_()
        o[a:b] = p @ vals
        if do is None:
            continue
        # the gradient that the backward is asked for takes the stored O
        ob = o[a:b].to(torch.bfloat16).double()
        dv[:end] += p.T @ do[a:b]
        ds = do[a:b] @ vals.T
        ds -= (do[a:b] * ob).sum(1, keepdim=True)
        ds *= p
        del p
        dq[a:b] = scale * (ds @ keys)
        dk[:end] += scale * (ds.T @ q[a:b])
    return (o, lse, dq, dk, dv) if do is not None else (o, lse, None, None, None)


def exact(case, seed):
    # about 0.2 s for 1e9 pairs; the longest forward would take over a minute
    if work(case)["flops"] / ((4 if case["kind"] == "fwd" else 14) * case["d"]) > 6e10:
        return None
    x = _inputs(case, seed)
    hq, hkv, d = case["hq"], case["hkv"], case["d"]
    scale, group = 1.0 / math.sqrt(d), hq // hkv
    dev = x["q"].device
    ring = case["kind"] == "ring"
    t = x["q"].shape[0]

    def zeros(n, h):
        return torch.zeros((n, h, d), dtype=torch.float64, device=dev)

    if ring:
        # the own chunk's keys, then the visiting chunk's that are visible: for
        # the mask the visiting chunk comes second, with its own bounds
        n = case["visit_rows"]
        r = {"o": zeros(t, hq), "lse": zeros(1, 1).new_zeros((hq, t)), "dq": zeros(t, hq),
             "dk": zeros(t, hkv), "dv": zeros(t, hkv), "sum_k": x["dk2"].double(),
             "sum_v": x["dv2"].double()}
        i = torch.arange(t, device=dev)
        for h in range(hq):
            c = h // group
            q, do = x["q"][:, h].double(), x["do"][:, h].double()
            k = torch.cat([x["k"][:, c], x["k2"][:, c]]).double()
            v = torch.cat([x["v"][:, c], x["v2"][:, c]]).double()
            own = i + 1 if case["causal"] else torch.full_like(i, t)
            vis = ((i + 1 + case["q_offset"] - case["visit_offset"]).clamp(0, n)
                   if case["causal"] else torch.full_like(i, n))
            o, lse, dq, dk, dv = _attend_two(q, k, v, do, own, vis, t, scale)
            r["o"][:, h], r["lse"][h], r["dq"][:, h] = o, lse, dq
            r["dk"][:, c] += dk[:t]
            r["dv"][:, c] += dv[:t]
            r["sum_k"][:, c] += dk[t:]
            r["sum_v"][:, c] += dv[t:]
        return r
    r = {"o": zeros(t, hq), "lse": zeros(1, 1).new_zeros((hq, t))}
    step = case["kind"] == "step"
    if step:
        r.update(dq=zeros(t, hq), dk=zeros(t, hkv), dv=zeros(t, hkv))
    a = 0
    for n in _lengths(case):
        b = a + n
        i = torch.arange(n, device=dev)
        see = i + 1 if case["causal"] else torch.full_like(i, n)
        for h in range(hq):
            c = h // group
            o, lse, dq, dk, dv = _attend(x["q"][a:b, h].double(), x["k"][a:b, c].double(),
                                         x["v"][a:b, c].double(),
                                         x["do"][a:b, h].double() if step else None, see, scale)
            r["o"][a:b, h], r["lse"][h, a:b] = o, lse
            if step:
                r["dq"][a:b, h] = dq
                r["dk"][a:b, c] += dk
                r["dv"][a:b, c] += dv
        a = b
    return r


def _attend_two(q, k, v, do, own, vis, split, scale, blocks=2048):
    """As _attend over two key chunks in one row of keys: row i sees own[i]
    keys of the first `split` and vis[i] of the rest."""
    n, m = q.shape[0], k.shape[0]
    o, dq = torch.empty_like(q), torch.empty_like(q)
    lse = torch.empty(n, dtype=torch.float64, device=q.device)
    dk, dv = torch.zeros_like(k), torch.zeros_like(v)
    j = torch.arange(m, device=q.device)
    for a in range(0, n, blocks):
        b = min(n, a + blocks)
        hide = torch.where(j[None] < split, j[None] >= own[a:b, None],
                           j[None] - split >= vis[a:b, None])
        p = (q[a:b] @ k.T * scale).masked_fill_(hide, -math.inf)
        lse[a:b] = torch.logsumexp(p, 1)
        p = (p - lse[a:b, None]).exp_()
        o[a:b] = p @ v
        ob = o[a:b].to(torch.bfloat16).double()
        dv += p.T @ do[a:b]
        ds = p * (do[a:b] @ v.T - (do[a:b] * ob).sum(1, keepdim=True))
        dq[a:b] = scale * (ds @ k)
        dk += scale * (ds.T @ q[a:b])
    return o, lse, dq, dk, dv

