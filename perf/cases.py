"""The calls whose speed is watched, over the sizes, types and options a serving program uses.

A case is one of:
  compress   one layer's prompt cache compressed (score, pool, select, gather) into caller-owned buffers
  decode     one decode step over a layer's compressed cache, with the rows generated since (if any):
             the new token's K and V rows are appended first, then attended with the rest
  stack      several layers as a program runs them: each compressed with its row copy on a second
             stream beside the next layer's scoring, then one decode step per layer

Shapes are the repository's workloads' (the tiny fp32 layer, Qwen2.5-7B's 28 query and 4 KV heads,
Qwen3-32B's 64 and 8, head dimension 128) at prompts from 1K to 1M tokens. Every case holds the
buffers a serving loop holds: workspace, outputs, the offsets on device and host.

Inputs: a window's rows agree on what matters (the observation that makes a final window a useful
selector), so every KV head has one direction u its window queries share and its keys carry by a
coefficient that is constant over spans of 16 tokens; the rest of both is N(0,1) noise. Logits then
have a shared part of standard deviation 2.5 and a per-row part of 1, so window scores span several
orders of magnitude, as attention weights do. The first four tokens carry a large coefficient
(attention sinks).
"""
import math

import numpy as np
import torch

import paper_2609_03235_amd as sg

SHARED = 2.5  # standard deviation of the logits' part that a window's rows share
SPAN = 16     # tokens that share a coefficient

_DT = {"bf16": torch.bfloat16, "f32": torch.float32}
_BITS = {"bf16": torch.int16, "f32": torch.int32}  # gathered rows are copies: compared as bits
_AGG = {"mean": sg.GROUP_MEAN, "ipt_max": sg.GROUP_IPT_MAX, "ipt_mean": sg.GROUP_IPT_MEAN,
        "ipt_only": sg.GROUP_IPT_ONLY}


def _compress(name, B, C, *, hq=28, hkv=4, d=128, w=64, kp=7, sink=1024, recent=1024, ratio=0.25, dtype="bf16",
              agg="mean", question=0, lse=False, scores="beta"):
    return dict(name=name, kind="compress", B=B, C=C, hq=hq, hkv=hkv, d=d, w=w, kp=kp, sink=sink, recent=recent,
                ratio=ratio, dtype=dtype, agg=agg, question=question, lse=lse, scores=scores)


def _decode(name, B, C, *, hq=28, hkv=4, d=128, sink=1024, recent=1024, ratio=0.25, dtype="bf16", out="f32", new=0,
            cap=0, scores="beta"):
    return dict(name=name, kind="decode", B=B, C=C, hq=hq, hkv=hkv, d=d, sink=sink, recent=recent, ratio=ratio,
                dtype=dtype, out=out, new=new, cap=cap, scores=scores)


def listed():
    return [
        # the smallest call: the fp32 2K layer of the end-to-end check and of small test models
        _compress("compress_2k_f32", 1, 2048, hq=4, hkv=2, d=64, w=32, sink=4, recent=32, dtype="f32", scores="uniform"),
        # a short chat or retrieval prompt of a length nobody chose
        _compress("compress_6k", 1, 6143, sink=128, recent=128),
        # one long prompt at a time: a Qwen2.5-7B layer at 32K, the interactive case
        _compress("compress_32k", 1, 32768),
        # a batch of long prompts, the throughput case: a Qwen2.5-7B layer at 128K x 8
        _compress("compress_128k_b8", 8, 131072),
        # the paper's main setting: a 128-token window and the Ipt. max aggregation, one odd-length
        # prompt; the window sits before the prompt's last 200 tokens (the question)
        _compress("compress_100k_w128_iptmax", 1, 100003, w=128, agg="ipt_max", question=200),
        # prefill attention hands over the window rows' log-sum-exp: a Qwen3-32B layer at 64K x 4
        _compress("compress_64k_b4_lse", 4, 65536, hq=64, hkv=8, sink=128, recent=128, lse=True),
        # the longest prompts: a Qwen2.5-7B layer at 1M x 4 with skewed head scores
        _compress("compress_1m_b4", 4, 1 << 20, scores="skewed"),
        # a generation step at batch 1 over what a 32K prompt leaves: latency
        _decode("decode_32k", 1, 32768),
        # the throughput step: 128K x 8
        _decode("decode_128k_b8", 8, 131072),
        # in the middle of a generation: 41 of 256 rows appended, this step's the 42nd, bf16 output,
        # unequal segments of an odd-length prompt
        _decode("decode_50k_b3_appended", 3, 49999, out="bf16", new=41, cap=256, scores="skewed"),
        # the largest cache: a Qwen3-32B layer at 256K x 16, a 10 % budget
        _decode("decode_256k_b16", 16, 262144, hq=64, hkv=8, sink=128, recent=128, ratio=0.10),
        # eight layers of a 32K prompt as a program chains them, and the first generated token
        dict(_compress("stack_32k_8l", 1, 32768), kind="stack", layers=8),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A compress or decode case of the listed ones' ranges: prompts of 1K to 1M tokens (odd lengths
    among them), batches and heads, windows, pooling widths, budgets, aggregations, types."""
    hq, hkv, d = rng.choice([(28, 4, 128), (28, 4, 128), (64, 8, 128), (16, 2, 128), (8, 8, 64), (4, 2, 64)])
    compress = rng.random() < 0.6
    f32 = rng.random() < (0.15 if compress else 0.25)
    # a short prompt keeps fewer initial and recent rows; both always fit the smallest budget here
    C = _log_int(rng, 1024, 1 << 20)
    recent = rng.choice([r for r in (32, 128, 1024) if r * 32 <= C] or [32])
    w = rng.choice([v for v in (32, 48, 64, 64, 128) if v <= recent and v * (hq // hkv) <= 1024])
    # K rows in all: no more window logits than the largest listed case's, a sixteenth of that for fp32
    most = min(16 << 20, (16 << 20) * 448 // (w * hq // hkv)) if compress else 16 << 20
    most //= 16 if f32 else 1
    C = max(recent * 32, min(C, most // hkv))
    if rng.random() < 0.5:
        C -= 1 - C % 2  # an odd length
    B = min(_log_int(rng, 1, 32), max(1, most // (hkv * C)))
    common = dict(hq=hq, hkv=hkv, d=d, sink=rng.choice([4, recent]), recent=recent,
                  ratio=round(rng.uniform(0.10, 0.50), 3), dtype="f32" if f32 else "bf16",
                  scores=rng.choice(["beta", "skewed", "uniform"]))
    if not compress:
        cap = rng.choice([0, 0, 64, 256])
        case = _decode("", B, C, out=rng.choice(["f32", "bf16"]), cap=cap, new=rng.randrange(cap) if cap else 0, **common)
    else:
        agg = rng.choice(["mean", "mean", "mean", "ipt_max", "ipt_mean", "ipt_only"])
        case = _compress("", B, C, w=w, kp=rng.choice([1, 5, 7, 7, 13, 21]), agg=agg,
                         question=rng.choice([0, 0, (recent - w) // 2]), lse=rng.random() < 0.2, **common)
    del case["name"]
    return case


# ------------------------------------------------------------------ inputs
def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 2654435761 % (1 << 62) + 12345)
    return g


def _randn(g, *shape):
    return torch.randn(shape, generator=g, device="cuda", dtype=torch.float32)


def _directions(case, g):
    u = _randn(g, case["B"], case["hkv"], 1, case["d"])
    return u / u.norm(dim=-1, keepdim=True)


def _keys(case, g, u, b, n):
    """Keys of sequence b [hkv, n, d]: noise plus the span coefficient along the head's direction."""
    t = _randn(g, case["hkv"], (n + SPAN - 1) // SPAN, 1).repeat_interleave(SPAN, dim=1)[:, :n]
    if n > 4:
        t[:, :4] = 5.0
    x = _randn(g, case["hkv"], n, case["d"])
    return x.addcmul_(t, u[b])


def _queries(case, g, u, rows):
    """Query rows [B, hq, rows, d] whose logits share a part of standard deviation SHARED."""
    B, hq, hkv, d = case["B"], case["hq"], case["hkv"], case["d"]
    q = _randn(g, B, hkv, hq // hkv, rows, d)
    q += SHARED * math.sqrt(d) * u.view(B, hkv, 1, 1, d)
    return q.view(B, hq, rows, d)


def _head_scores(case, seed):
    rng = np.random.Generator(np.random.PCG64(seed))
    n = case["hkv"]
    if case["scores"] == "uniform":
        return rng.uniform(0.0, 1.0, n)
    if case["scores"] == "beta":
        return rng.beta(0.5, 2.0, n) + 1e-3
    out = rng.uniform(0.0, 0.1, n)
    out[rng.permutation(n)[: max(1, n // 5)]] = rng.uniform(0.8, 1.0)
    return out


def _total(case):
    return sg.total_from_ratio(case["ratio"], 1, case["hkv"], case["C"], case["sink"], case["recent"], of_middle=1)


def _budgets(case, seed):
    return sg.allocate_budgets(_head_scores(case, seed), 1, case["hkv"], case["C"], case["sink"], case["recent"],
                               _total(case))


def _win0(case):
    return case["C"] - case["question"] - case["w"]


def _qhead_scores(case, seed):
    if case["agg"] == "mean":
        return None
    return np.random.Generator(np.random.PCG64(seed + 7)).uniform(0.05, 1.0, case["hq"])


def _layer(case, seed):
    """Window queries, K, V of one layer, and its decode queries."""
    g, dt = _generator(seed), _DT[case["dtype"]]
    B, C, hkv, d = case["B"], case["C"], case["hkv"], case["d"]
    u = _directions(case, g)
    k = torch.empty((B, hkv, C, d), dtype=dt, device="cuda")
    v = torch.empty((B, hkv, C, d), dtype=dt, device="cuda")
    for b in range(B):
        k[b].copy_(_keys(case, g, u, b, C))
        v[b].copy_(_randn(g, hkv, C, d))
    q_win = _queries(case, g, u, case["w"]).to(dt)
    q = _queries(case, g, u, 1)[:, :, 0].to(dt)
    return dict(q_win=q_win, k=k, v=v, q=q)


def _window_logits(case, x, b, h, dtype):
    """Logits [G*w, keys] of a KV head's window rows over the keys [0, win0 + w), masked causally."""
    G, w, d, win0 = case["hq"] // case["hkv"], case["w"], case["d"], _win0(case)
    n = win0 + w
    q = x["q_win"][b, h * G:(h + 1) * G].reshape(G * w, d).to(dtype)
    logits = q @ x["k"][b, h, :n].to(dtype).T
    logits *= 1.0 / math.sqrt(d)
    mask = torch.ones((w, w), dtype=torch.bool, device="cuda").triu(1)
    logits.view(G, w, n)[:, :, win0:].masked_fill_(mask, -math.inf)
    return logits


def _lse_given(case, x):
    """What prefill attention would hand over: the window rows' log-sum-exp, rounded to fp32."""
    B, hq, hkv, w = case["B"], case["hq"], case["hkv"], case["w"]
    out = torch.empty((B, hkv, hq // hkv * w), dtype=torch.float32, device="cuda")
    for b in range(B):
        for h in range(hkv):
            out[b, h] = torch.logsumexp(_window_logits(case, x, b, h, torch.float32), dim=1)
    return out.view(B, hq, w)


def _compress_state(case, seed):
    x = _layer(case, seed)
    budgets = _budgets(case, seed)
    B, d, rows = case["B"], case["d"], int(case["B"] * budgets.sum())
    out = dict(k_c=torch.empty((rows, d), dtype=_DT[case["dtype"]], device="cuda"),
               v_c=torch.empty((rows, d), dtype=_DT[case["dtype"]], device="cuda"),
               kept_pos=torch.empty(rows, dtype=torch.int32, device="cuda"),
               offsets=torch.empty(B * case["hkv"] + 1, dtype=torch.int64, device="cuda"),
               scores=torch.empty((B, case["hkv"], _win0(case)), dtype=torch.float32, device="cuda"))
    bits = _BITS[case["dtype"]]
    x.update(budgets=budgets, out=out, lse=_lse_given(case, x) if case["lse"] else None,
             whole=dict(k_c=out["k_c"].view(bits), v_c=out["v_c"].view(bits), kept_pos=out["kept_pos"],
                        offsets=out["offsets"], scores=out["scores"]),
             args=dict(pool_kernel=case["kp"], b_sink=case["sink"], b_window=case["recent"],
                       group_agg=_AGG[case["agg"]], qhead_scores=_qhead_scores(case, seed),
                       window_pos=_win0(case) if case["question"] else -1))
    return x


def _compress_workspace(x):
    a = x["args"]
    desc = sg.compress_desc(x["q_win"], x["k"], pool_kernel=a["pool_kernel"], b_sink=a["b_sink"], b_window=a["b_window"])
    return sg.alloc_workspace(sg.compress_workspace_size(desc), "cuda")


def _cache(case, seed):
    """A compressed cache as the compression leaves it, decode queries, and the appended rows."""
    g, dt = _generator(seed), _DT[case["dtype"]]
    B, hkv, d = case["B"], case["hkv"], case["d"]
    offsets = sg.segment_offsets(_budgets(case, seed), B)
    u = _directions(case, g)
    k_c = torch.empty((int(offsets[-1]), d), dtype=dt, device="cuda")
    v_c = torch.empty_like(k_c)
    for s in range(B * hkv):
        b, h, lo, hi = s // hkv, s % hkv, int(offsets[s]), int(offsets[s + 1])
        one = dict(case, hkv=1)
        k_c[lo:hi].copy_(_keys(one, g, u[:, h:h + 1], b, hi - lo)[0])
        v_c[lo:hi].copy_(_randn(g, hi - lo, d))
    x = dict(q=_queries(case, g, u, 1)[:, :, 0].to(dt), k_c=k_c, v_c=v_c, offsets_host=offsets,
             offsets=torch.from_numpy(offsets).cuda(), k_new=None, v_new=None)
    if case["cap"]:
        x["k_new"], x["v_new"] = (_randn(g, B, hkv, case["cap"], d).to(dt) for _ in range(2))
        x["k_step"], x["v_step"] = (_randn(g, B, hkv, d).to(dt) for _ in range(2))
    return x


def prepare(case, seed):
    if case["kind"] == "compress":
        x = _compress_state(case, seed)
        x["ws"] = _compress_workspace(x)
        return dict(case=case, **x)
    if case["kind"] == "decode":
        x = _cache(case, seed)
        out_dtype = _DT[case["out"]]
        desc = sg.decode_desc(x["q"], case["hkv"], out_dtype)
        x["ws"] = sg.alloc_workspace(sg.decode_workspace_size(desc, x["offsets_host"], case["cap"]), "cuda")
        x["out"] = torch.empty((case["B"], case["hq"], case["d"]), dtype=out_dtype, device="cuda")
        x["lse"] = torch.empty((case["B"], case["hq"]), dtype=torch.float32, device="cuda")
        return dict(case=case, **x)
    layers = [_compress_state(case, seed * 64 + l) for l in range(case["layers"])]
    ws_d = 0
    for x in layers:
        x["offsets_host"] = sg.segment_offsets(x["budgets"], case["B"])
        ws_d = max(ws_d, sg.decode_workspace_size(sg.decode_desc(x["q"], case["hkv"], torch.float32), x["offsets_host"]))
        x["dec"] = torch.empty((case["B"], case["hq"], case["d"]), dtype=torch.float32, device="cuda")
        x["dec_lse"] = torch.empty((case["B"], case["hq"]), dtype=torch.float32, device="cuda")
    return dict(case=case, layers=layers, ws=_compress_workspace(layers[0]), ws_d=sg.alloc_workspace(ws_d, "cuda"),
                gather=torch.cuda.Stream())


# --------------------------------------------------------------------- run
def run(state):
    case = state["case"]
    if case["kind"] == "compress":
        sg.compress_layer(state["q_win"], state["k"], state["v"], state["budgets"], window_lse=state["lse"],
                          workspace=state["ws"], out=state["out"], **state["args"])
        return state["whole"]
    if case["kind"] == "decode":
        new = 0
        if case["cap"]:
            new = case["new"] + 1
            sg.append_kv(state["q"], state["k_step"], state["v_step"], state["k_new"], state["v_new"], case["new"])
        sg.decode_attention(state["q"], state["k_c"], state["v_c"], state["offsets"], state["offsets_host"],
                            case["hkv"], out_dtype=state["out"].dtype, k_new=state["k_new"], v_new=state["v_new"],
                            n_new=new, workspace=state["ws"], out=state["out"], lse=state["lse"])
        return dict(out=state["out"], lse=state["lse"])
    last = len(state["layers"]) - 1
    for i, x in enumerate(state["layers"]):
        sg.compress_layer(x["q_win"], x["k"], x["v"], x["budgets"], workspace=state["ws"], out=x["out"],
                          gather_stream=state["gather"] if i < last else None, **x["args"])
    torch.cuda.current_stream().wait_stream(state["gather"])
    for x in state["layers"]:
        sg.decode_attention(x["q"], x["out"]["k_c"], x["out"]["v_c"], x["out"]["offsets"], x["offsets_host"],
                            case["hkv"], out_dtype=torch.float32, workspace=state["ws_d"], out=x["dec"],
                            lse=x["dec_lse"])
    return [dict(scores=x["out"]["scores"], kept_pos=x["out"]["kept_pos"], k_c=x["whole"]["k_c"],
                 v_c=x["whole"]["v_c"], out=x["dec"], lse=x["dec_lse"]) for x in state["layers"]]


def work(case):
    eb = 2 if case["dtype"] == "bf16" else 4
    B, C, hq, hkv, d = case["B"], case["C"], case["hq"], case["hkv"], case["d"]
    kept = B * _total(case)
    row = d * eb
    dec = dict(bytes=2 * kept * row + B * hq * (row + 4 * d + 4) + 8 * (B * hkv + 1), flops=4 * kept * hq // hkv * d)
    if case["kind"] == "decode":
        if case["cap"]:  # this step's rows read and written, the earlier ones read
            dec["bytes"] += 2 * B * hkv * row * (case["new"] + 2)
            dec["flops"] += 4 * B * hq * d * (case["new"] + 1)
        return dec
    # K once, the kept V rows; the kept rows, their positions and the scores out; the logits once
    com = dict(bytes=B * hkv * C * row + B * hq * case["w"] * row + 3 * kept * row + 4 * kept + 4 * B * hkv * _win0(case),
               flops=2 * B * hq * case["w"] * d * (_win0(case) + case["w"] // 2))
    if case["kind"] == "compress":
        return com
    return {m: case["layers"] * (com[m] + dec[m]) for m in com}


def tolerance(case):
    """About four times what the calls are off from `exact` (scores up to 4.7e-6, decode outputs 6e-7
    in fp32 and 1.8e-3 in bf16, over the listed cases and six drawn ones). Scores: fp32 logits (each off by up to 2^-23 of
    the sum of its products' magnitudes) through an exponential, so their relative error is the
    logit's absolute one. Kept rows: two rows whose scores are equal to within that error may change
    places at the budget's edge, which moves the kept rows between them by one. Decode: sums of fp32
    products; bf16 outputs are rounded to 2^-9."""
    if case["kind"] == "decode":
        return {"rel": 7e-3, "max": 1e-2} if case["out"] == "bf16" else {"rel": 1e-5, "max": 1e-4}
    return {"rel": 2e-5, "max": 1e-4, "differ": 1e-2}


# ------------------------------------------------------------------- exact
def _exact_scores(case, x, seed):
    B, hq, hkv, w, kp, win0 = case["B"], case["hq"], case["hkv"], case["w"], case["kp"], _win0(case)
    G, agg = hq // hkv, case["agg"]
    sigma = _qhead_scores(case, seed)
    given = _lse_given(case, x).double() if case["lse"] else None
    out = torch.empty((B, hkv, win0), dtype=torch.float64, device="cuda")
    for b in range(B):
        for h in range(hkv):
            logits = _window_logits(case, x, b, h, torch.float64)
            lse = torch.logsumexp(logits, 1) if given is None else given[b, h * G:(h + 1) * G].reshape(-1)
            p = logits[:, :win0].sub_(lse[:, None]).exp_()
            heads = p.view(G, w, win0).sum(1)
            del p, logits
            if agg == "mean":
                a = heads.mean(0)
            else:
                s = torch.from_numpy(sigma[h * G:(h + 1) * G]).cuda()
                if agg == "ipt_max":
                    a = (heads * s[:, None]).amax(0)
                elif agg == "ipt_mean":
                    a = (heads * s[:, None]).mean(0)
                else:
                    a = heads[int(s.argmax())]
            run_sum = torch.nn.functional.pad(a, (kp // 2, kp // 2)).unfold(0, kp, 1)
            out[b, h] = run_sum.sum(1) / kp
    return out


def _exact_decode(case, q, k_c, v_c, offsets, k_new=None, v_new=None):
    hq, hkv, d = case["hq"], case["hkv"], case["d"]
    G, B = hq // hkv, case["B"]
    out = torch.zeros((B, hq, d), dtype=torch.float64, device="cuda")
    lse = torch.empty((B, hq), dtype=torch.float64, device="cuda")
    for s in range(B * hkv):
        b, h, lo, hi = s // hkv, s % hkv, int(offsets[s]), int(offsets[s + 1])
        k, v = k_c[lo:hi].double(), v_c[lo:hi].double()
        if k_new is not None:
            k, v = torch.cat([k, k_new[b, h].double()]), torch.cat([v, v_new[b, h].double()])
        logits = q[b, h * G:(h + 1) * G].double() @ k.T / math.sqrt(d)
        lse[b, h * G:(h + 1) * G] = torch.logsumexp(logits, 1)
        out[b, h * G:(h + 1) * G] = torch.softmax(logits, 1) @ v
    return dict(out=out, lse=lse)


def exact(case, seed):
    if case["kind"] == "compress":
        x = _layer(case, seed)
        return dict(scores=_exact_scores(case, x, seed), k_c=None, v_c=None, kept_pos=None, offsets=None)
    if case["kind"] == "decode":
        x = _cache(case, seed)
        new = [None, None]
        if case["cap"]:
            at = case["new"]
            x["k_new"][:, :, at], x["v_new"][:, :, at] = x["k_step"], x["v_step"]
            new = [x[n][:, :, : at + 1] for n in ("k_new", "v_new")]
        return _exact_decode(case, x["q"], x["k_c"], x["v_c"], x["offsets_host"], *new)
    # the decode over a stack's caches depends on which of two equal rows was kept: no exact value
    return [dict(scores=_exact_scores(case, _layer(case, seed * 64 + l), seed * 64 + l), kept_pos=None, k_c=None,
                 v_c=None, out=None, lse=None) for l in range(case["layers"])]
