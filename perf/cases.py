"""The work a user of this framework has it do, as cases that can be timed and compared.

A case names an entry point ("kind"), the lengths of a batch of replay trees as text ("P:R,R,R;P:R,R" - one tree per
";", its prompt length, then its branch lengths), the head layout and the replay mode. Kinds:

* ``op``     the differentiable op: group_attention forward, then its backward through torch.autograd. What a training
             script calls.
* ``score``  the op without gradients: the forward pass that computes log-probabilities under a reference or old policy.
* ``step``   SharedStep.run: the explicit two-call step on buffers that a program keeps (trainers with their own autograd).
* ``calls``  SharedStep(path="calls"): the six separate entry points, as a program that shards a tree strings them.
* ``plain``  prefill_fwd + prefill_bwd over packed causal sequences without branches (the pre-training or SFT half of a
             mixed batch). Written as "P;P;P".
* ``merge``  lse_merge of partial attention states, as after an exchange between prompt shards ("parts", "rows").

Lengths come from the named workloads of ``paper_2609_33133_amd.inputs`` (tiny, prompt, response, short_resp) or are
generic chat-like ones, odd on purpose. Inputs are N(0, 1) (logits of standard deviation one, as trained heads with
normalised queries and keys have them), drawn on the GPU from the seed.
"""
import math

import numpy as np
import torch

from paper_2609_33133_amd import api
from paper_2609_33133_amd.api import REPLAY_AUTO, REPLAY_FUSED, REPLAY_SPLIT, GroupBatch
from paper_2609_33133_amd.autograd import group_attention
from paper_2609_33133_amd.group_attention import SharedStep

MODES = {"fused": REPLAY_FUSED, "split": REPLAY_SPLIT, "auto": REPLAY_AUTO}
# (query heads, KV heads, head dimension): a full 8-KV-head model, a 7B model's 28 / 4, one rank's share of the first
# under 4-way tensor parallelism, a d = 64 model, and the small d = 64 layout without grouped heads
HEADS = ((32, 8, 128), (28, 4, 128), (8, 2, 128), (16, 4, 64), (4, 4, 64))


def _tree_case(name, kind, lengths, heads, mode="fused"):
    hq, hkv, d = heads
    return {"name": name, "kind": kind, "lengths": lengths, "hq": hq, "hkv": hkv, "d": d, "mode": mode}


def listed():
    h32, h28, h8, h64, h4 = HEADS
    return [
        # the smallest call: a unit test, a debugging run, the last layer of a toy model; launches and host time count
        _tree_case("tiny_step", "step", "256:128,128", h4),
        # one rank's microbatch of a group-relative RL step on chat data: a few prompts, 4-8 sampled answers each
        _tree_case("op_chat", "op", "417:311,198,977,64,523,402;1130:640,87,333,1204;233:58,120,77,96,41,205,150,88;"
                   "1811:455,702,391,128,260", h32),
        # the same kind of batch on one rank under tensor parallelism (8 query / 2 KV heads left)
        _tree_case("op_chat_tp", "op", "905:512,731,288,1040,196,655,870,333;384:290,411,176,620;1337:702,530,911,404",
                   h8),
        # a small d = 64 model, one prompt and its samples
        _tree_case("op_d64", "op", "1500:801,644,1022,377,590,1210,455,930", h64),
        # long document, many short answers (extraction, judging); the per-group rule picks the replay form
        _tree_case("step_short_answers", "step", "16384:" + ",".join(["64"] * 32), h32, "auto"),
        # scoring many candidate continuations of one long context: forward only, odd and very short branches
        _tree_case("score_candidates", "score", "8191:" + ",".join(str(5 + (11 * i) % 53) for i in range(24)), h32),
        # the headline workload: long prompt, eight answers
        _tree_case("step_prompt_heavy", "step", "32768:" + ",".join(["2048"] * 8), h32),
        # long reasoning traces from a short prompt (the largest case)
        _tree_case("step_response_heavy", "step", "2048:" + ",".join(["16384"] * 16), h32),
        # several trees of very different shape in one call, 28 / 4 heads
        _tree_case("step_ragged", "step", "6011:1733,402,2950,811;611:3207,5122,1999,2480,4017,777,1500,2222;"
                   "9474:350,268,1201,519,904,300,427,655;2048:1024,1024,1024,1024", h28),
        # the six entry points one by one with the split replay (partial states and merge), as a sharded caller runs them
        _tree_case("calls_split", "calls", "4096:512,700,333,640,512,480,900,411;1025:300,513,129,770", h32, "split"),
        # ordinary packed causal sequences, forward and backward
        _tree_case("plain_causal", "plain", "2717;901;4096;333;1580;3001", h32),
        # partial states of four prompt shards combined
        {"name": "merge_shards", "kind": "merge", "parts": 4, "rows": 12289, "hq": 32, "d": 128},
    ]


def _lengths(text):
    ps, rs = [], []
    for tree in text.split(";"):
        p, _, r = tree.partition(":")
        ps.append(int(p))
        rs.append([int(x) for x in r.split(",")] if r else [])
    return ps, rs


def _pairs(ps, rs):
    n = 0
    for p, br in zip(ps, rs):
        n += p * (p + 1) // 2 + sum(p * r + r * (r + 1) // 2 for r in br)
    return n


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: the kinds above over their whole ranges (prompts 16 .. 32768, branches 1 .. 16384, 1 .. 6 trees,
    every head layout and replay mode), at most 140 TFLOP and 300,000 tokens."""
    kind = rng.choice(["op", "op", "op", "step", "step", "step", "score", "score", "calls", "plain", "plain", "merge"])
    if kind == "merge":
        return {"kind": kind, "parts": rng.randint(2, 8), "rows": _log(rng, 64, 16384), "hq": rng.choice([8, 28, 32]),
                "d": rng.choice([64, 128])}
    hq, hkv, d = rng.choice(HEADS[:4])
    while True:
        ps, rs = [], []
        if kind == "plain":
            ps = [_log(rng, 16, 16384) for _ in range(rng.randint(1, 8))]
            rs = [[] for _ in ps]
        else:
            for _ in range(rng.randint(1, 6)):
                ps.append(_log(rng, 16, 32768))
                mid = _log(rng, 8, 8192)  # branches of one tree are within a factor of two of their tree's length
                rs.append([max(1, min(16384, _log(rng, mid / 2, mid * 2))) for _ in range(rng.choice([2, 4, 8, 16, 32]))])
        tokens = sum(ps) + sum(sum(r) for r in rs)
        if tokens <= 300_000 and 14 * d * hq * _pairs(ps, rs) <= 140e12:
            break
    text = ";".join(str(p) + (":" + ",".join(map(str, r)) if r else "") for p, r in zip(ps, rs))
    mode = "split" if kind == "calls" and rng.random() < 0.5 else rng.choice(["fused", "fused", "auto"])
    case = _tree_case("", kind, text, (hq, hkv, d), "fused" if kind == "plain" else mode)
    del case["name"]
    return case


def _batch(case):
    ps, rs = _lengths(case["lengths"])
    if case["kind"] == "plain":  # prefill entry points read the prompt offsets only
        rs = [[1] for _ in ps]
    cu = lambda v: np.concatenate([[0], np.cumsum(v)])
    return GroupBatch(cu(ps), cu([len(r) for r in rs]), cu([x for r in rs for x in r]), case["hq"], case["hkv"], case["d"])


def _inputs(case, seed, device="cuda"):
    gen = torch.Generator(device=device).manual_seed(1_000_003 * int(seed) + 17)

    def normal(*shape, dtype=torch.bfloat16):
        return torch.randn(*shape, generator=gen, device=device, dtype=torch.float32).to(dtype)

    hq, d = case["hq"], case["d"]
    if case["kind"] == "merge":
        n, rows = case["parts"], case["rows"]
        return {"o": normal(n, rows, hq, d, dtype=torch.float32), "lse": 3 * normal(n, hq, rows, dtype=torch.float32)}
    ps, rs = _lengths(case["lengths"])
    tp, tr, hkv = sum(ps), sum(sum(r) for r in rs), case["hkv"]
    x = {}
    for side, t in (("p", tp), ("r", tr)):
        for n, h in (("q", hq), ("k", hkv), ("v", hkv), ("do", hq)):
            x[n + "_" + side] = normal(t, h, d)
    return x


LEAVES = ("q_p", "k_p", "v_p", "q_r", "k_r", "v_r")


def prepare(case, seed):
    kind = case["kind"]
    s = {"kind": kind, "x": _inputs(case, seed)}
    if kind == "merge":
        return s
    s["batch"] = b = _batch(case)
    s["mode"] = MODES[case["mode"]]
    if kind == "op":
        for n in LEAVES:
            s["x"][n].requires_grad_(True)
    elif kind in ("step", "calls"):
        s["step"] = SharedStep(b, "cuda", mode=s["mode"], path="tree" if kind == "step" else "calls")
    return s


def run(state):
    kind, x = state["kind"], state["x"]
    if kind == "merge":
        o, _, lse = api.lse_merge(x["o"], x["lse"])
        return {"o": o, "lse": lse}
    b = state["batch"]
    if kind == "op":
        o_p, o_r = group_attention(*(x[n] for n in LEAVES), b, mode=state["mode"])
        grads = torch.autograd.grad((o_p, o_r), [x[n] for n in LEAVES], (x["do_p"], x["do_r"]))
        return {"o_p": o_p.detach(), "o_r": o_r.detach(), **{"d" + n: g for n, g in zip(LEAVES, grads)}}
    if kind == "score":
        with torch.no_grad():
            o_p, o_r = group_attention(*(x[n] for n in LEAVES), b, mode=state["mode"])
        return {"o_p": o_p, "o_r": o_r}
    if kind == "plain":
        o, lse = api.prefill_fwd(b, x["q_p"], x["k_p"], x["v_p"])
        dq, _, dkv = api.prefill_bwd(b, x["q_p"], x["k_p"], x["v_p"], o, lse, x["do_p"])
        return {"o_p": o, "lse_p": lse, "dq_p": dq, "dk_p": dkv[0], "dv_p": dkv[1]}
    state["step"].run(x)
    return state["step"].outputs()


def work(case):
    if case["kind"] == "merge":
        n, rh, d = case["parts"], case["rows"] * case["hq"], case["d"]
        return {"bytes": rh * (n * (4 * d + 4) + 2 * d + 4), "flops": rh * n * 2 * d}
    ps, rs = _lengths(case["lengths"])
    t, hq, hkv, d = sum(ps) + sum(sum(r) for r in rs), case["hq"], case["hkv"], case["d"]
    forward_only = case["kind"] == "score"
    q, kv = t * hq * d * 2, t * hkv * d * 2
    # forward: Q, K, V in, O out (LSE is internal to the op but written for the backward); backward adds dO in and
    # dQ, dK, dV out; two products forward, five backward (S is needed again)
    nbytes = 2 * q + 2 * kv + (0 if forward_only else 2 * q + 2 * kv + 4 * t * hq)
    return {"bytes": nbytes, "flops": (4 if forward_only else 14) * d * hq * _pairs(ps, rs)}


def tolerance(case):
    # fp32 sums of a few terms with bf16 results (2^-9 worst, ~1.7e-3 rms rounding)
    if case["kind"] == "merge":
        return {"rel": 5e-3}
    # bf16 operands and results with fp32 sums; P and dS are rounded to bf16 before their products
    return {"rel": 1e-2}


def exact(case, seed):
    """The same outputs in 64 bits from the definition: softmax over the visible keys and its derivatives, in blocks of
    query rows, one KV head at a time."""
    if case["kind"] == "merge":
        x = _inputs(case, seed)
        o, lse = x["o"].double(), x["lse"].double()
        tot = torch.logsumexp(lse, 0)
        w = torch.exp(lse - tot).transpose(1, 2).unsqueeze(-1)
        return {"o": (w * o).sum(0), "lse": tot}
    ps, rs = _lengths(case["lengths"])
    hq, hkv, d = case["hq"], case["hkv"], case["d"]
    if 14 * d * hq * _pairs(ps, rs) > 100e12:
        return None
    x = _inputs(case, seed)
    g, scale = hq // hkv, 1.0 / math.sqrt(d)
    f64 = dict(dtype=torch.float64, device="cuda")
    out = {}
    for side in ("p", "r"):
        t = x["q_" + side].shape[0]
        out["o_" + side], out["dq_" + side] = torch.zeros(t, hq, d, **f64), torch.zeros(t, hq, d, **f64)
        out["dk_" + side], out["dv_" + side] = torch.zeros(t, hkv, d, **f64), torch.zeros(t, hkv, d, **f64)
        out["lse_" + side] = torch.zeros(hq, t, **f64)

    def rows_of(side, r0, r1, segs, pos0, kvh):
        """Query rows r0 .. r1 - 1 of `side` (positions pos0 ..) against the segments: (side, first row, length, causal)."""
        hs = slice(kvh * g, kvh * g + g)
        n = r1 - r0
        q = x["q_" + side][r0:r1, hs].double().transpose(0, 1)          # [g, n, d]
        do = x["do_" + side][r0:r1, hs].double().transpose(0, 1)
        k = torch.cat([x["k_" + s][a:a + m, kvh].double() for s, a, m, _ in segs])
        v = torch.cat([x["v_" + s][a:a + m, kvh].double() for s, a, m, _ in segs])
        s_ = torch.matmul(q, k.t().contiguous()).mul_(scale)
        at = 0
        for _, _, m, causal in segs:
            if causal:
                i = torch.arange(n, device="cuda")[:, None] + pos0
                s_[:, :, at:at + m].masked_fill_(torch.arange(m, device="cuda")[None] > i, -math.inf)
            at += m
        lse = torch.logsumexp(s_, -1)
        p = s_.sub_(lse.unsqueeze(-1)).exp_()
        o = torch.matmul(p, v)
        out["o_" + side][r0:r1, hs] = o.transpose(0, 1)
        out["lse_" + side][hs, r0:r1] = lse
        if case["kind"] == "score":
            return
        ds = torch.matmul(do, v.t().contiguous()).sub_((do * o).sum(-1, keepdim=True)).mul_(p)
        out["dq_" + side][r0:r1, hs] = torch.matmul(ds, k).transpose(0, 1) * scale
        flat = lambda m_: m_.reshape(g * n, -1)
        dk = torch.matmul(flat(ds).t(), flat(q)) * scale
        dv = torch.matmul(flat(p).t(), flat(do))
        at = 0
        for sd, a, m, _ in segs:
            out["dk_" + sd][a:a + m, kvh] += dk[at:at + m]
            out["dv_" + sd][a:a + m, kvh] += dv[at:at + m]
            at += m

    def blocks(length, keys):
        """Row blocks whose [g, rows, keys] arrays of 8 bytes stay near 2 GB."""
        step = max(64, int(2.5e8 / (g * max(1, keys))))
        return [(a, min(length, a + step)) for a in range(0, length, step)]

    p0 = r0 = 0
    for p, br in zip(ps, rs):
        for kvh in range(hkv):
            for a, e in blocks(p, p):
                rows_of("p", p0 + a, p0 + e, [("p", p0, e, True)], a, kvh)
            b0 = r0
            for r in br:
                for a, e in blocks(r, p + r):
                    rows_of("r", b0 + a, b0 + e, [("p", p0, p, False), ("r", b0, e, True)], a, kvh)
                b0 += r
        p0 += p
        r0 += sum(br)
    if case["kind"] == "score":
        names = ("o_p", "o_r")
    elif case["kind"] == "plain":
        names = ("o_p", "lse_p", "dq_p", "dk_p", "dv_p")
    elif case["kind"] == "op":
        names = ("o_p", "o_r", "dq_p", "dk_p", "dv_p", "dq_r", "dk_r", "dv_r")
    else:
        names = ("o_p", "lse_p", "o_r", "lse_r", "dq_p", "dk_p", "dv_p", "dq_r", "dk_r", "dv_r")
    return {n: out[n] for n in names}
