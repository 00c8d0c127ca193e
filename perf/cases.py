"""The work a user of this library has it do, as cases that can be timed.

Three kinds, each through the public calls of `paper_2510_13797_amd.bc`:

  decode   tokens of a generation through a stack of layers, one cache (`bc.Runtime`) per layer: append,
           attention over [prompt | beacons | window], eviction (`decode_step`, or `decode_step` with the
           beacon's own `beacon_step` behind a full window).  Small steps are captured once as a HIP graph
           and replayed, as a serving loop does; the large ones are called one by one.
  prefill  the beacon-masked attention of training: forward and gradients, or the forward alone with a
           workspace (scoring trajectories without training on them).
  distill  the top-k KL loss over the vocabulary and its gradient.

A decode pass starts by putting the caches' tables back (one small copy), so that every pass does the same
tokens of the rollout; everything else in a pass is what a user's program calls.
"""
import math

import numpy as np
import torch

from paper_2510_13797_amd import bc

RATIOS = (2, 4, 8, 16, 32)              # the compression ratios of the evaluation; c = 0: never compress
HEADS = ((12, 2), (32, 8), (14, 2), (24, 8), (4, 1), (8, 8), (16, 2), (5, 1))      # (query, KV) heads
MOST_STEP_BYTES = 290e6                 # K and V of one decode step: the largest listed one
MOST_PREFILL_FLOPS = 1.5e12
MOST_LOGITS = 4096 * 151936


def _decode(name, **kw):
    case = dict(kind="decode", dtype="bf16", B=64, Hq=12, Hkv=2, d=128, P_lo=256, P_hi=256, c=16, gen_lo=4095,
                gen_hi=4095, tokens=1, layers=16, graph=True, own_beacon=False, sort=False, peaked=False, shape=1)
    case.update(kw)
    return dict(name=name, **case) if name else case


def _prefill(name, **kw):
    case = dict(kind="prefill", B=16, Hq=12, Hkv=2, d=128, P_lo=256, P_hi=256, R_lo=7936, R_hi=7936, c=16,
                backward=True, shape=1)
    case.update(kw)
    return dict(name=name, **case) if name else case


def _distill(name, **kw):
    case = dict(kind="distill", T=4096, V=151936, k=100, dtype="bf16")
    case.update(kw)
    return dict(name=name, **case) if name else case


def listed():
    return [
        # one window of the small fp32 configuration, called step by step: latency of the calls themselves
        _decode("decode_tiny_f32_window", dtype="f32", B=2, Hq=4, Hkv=1, d=64, P_lo=32, P_hi=32, gen_lo=128, gen_hi=128,
                tokens=16, layers=1, graph=False),
        # one user's long generation: a single sequence, one token through 16 layers
        _decode("decode_single_stream", B=1, Hq=32, Hkv=8, P_lo=512, P_hi=512, gen_lo=16383, gen_hi=16383),
        # the headline: 64 sequences, token 4096 of the rollout (it closes a window) through 16 layers
        _decode("decode_batch64"),
        # a small model (head dimension 64), odd batch, prompts of different length, every ratio at once
        _decode("decode_d64_ragged", B=45, Hq=14, Hkv=2, d=64, P_lo=37, P_hi=411, c=-1, gen_lo=300, gen_hi=3000),
        # a server's ragged batch: 256 sequences of all ages and ratios, dispatch order refreshed once per pass
        _decode("decode_ragged256", B=256, P_lo=64, P_hi=512, c=-1, gen_lo=1, gen_hi=4428, tokens=8, layers=2,
                graph=False, sort=True),
        # the end of a long reasoning rollout with peaked keys; the window closes and the beacon attends itself
        _decode("decode_long_own_beacon", B=32, Hq=32, Hkv=8, P_lo=512, P_hi=512, c=32, gen_lo=32732, gen_hi=32732,
                tokens=4, layers=4, graph=False, own_beacon=True, peaked=True),
        # the uncompressed control at the headline's shape
        _decode("decode_uncompressed", c=0, gen_lo=4092, gen_hi=4092, tokens=4, layers=4, graph=False),
        # the training step's attention at full size: 16 trajectories of 8688 rows, forward and gradients
        _prefill("prefill_train_full"),
        # a micro-batch of a few short trajectories of odd length
        _prefill("prefill_train_short", B=3, P_lo=19, P_hi=130, R_lo=150, R_hi=700, c=-1),
        # scoring: forward alone with a workspace, ragged, four query heads per KV head
        _prefill("prefill_score_ragged", B=8, Hq=32, Hkv=8, P_lo=100, P_hi=600, R_lo=900, R_hi=4100, c=-1,
                 backward=False),
        # the distillation loss and its gradient over a large vocabulary
        _distill("distill_full"),
        # a smaller vocabulary of odd size: rows that start at any 2-byte boundary
        _distill("distill_odd_rows", T=509, V=50257),
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    def heads():
        return rng.choice(HEADS)

    kind = rng.choice(("decode", "decode", "prefill", "prefill", "distill"))
    while True:
        shape = rng.randrange(1, 1 << 20)
        if kind == "decode":
            Hq, Hkv = heads()
            d, dtype = rng.choice((64, 128)), rng.choice(("bf16", "bf16", "bf16", "f32"))
            B, P = log_int(1, 256), log_int(8, 512)
            c = rng.choice((0, -1) + RATIOS)
            gen = log_int(16, 4096) if c == 0 else log_int(16, 32768 if c > 0 else 8192)
            graph = rng.random() < 0.5
            case = _decode(None, dtype=dtype, B=B, Hq=Hq, Hkv=Hkv, d=d, P_lo=max(1, P // rng.choice((1, 4))), P_hi=P, c=c,
                           gen_lo=max(1, gen // rng.choice((1, 8))), gen_hi=gen, tokens=1 if graph else rng.choice((2, 4)),
                           layers=8 if graph else 2, graph=graph, own_beacon=False, sort=B > 96 and c == -1,
                           peaked=rng.random() < 0.25, shape=shape)
            if work(case)["bytes"] / (case["tokens"] * case["layers"]) <= MOST_STEP_BYTES:
                return case
        elif kind == "prefill":
            Hq, Hkv = heads()
            R = log_int(60, 8000)
            case = _prefill(None, B=log_int(1, 16), Hq=Hq, Hkv=Hkv, d=rng.choice((64, 128, 128)), P_lo=rng.choice((0, 16, 64)),
                            P_hi=log_int(64, 512), R_lo=max(1, R // rng.choice((1, 4))), R_hi=R, c=rng.choice((0, -1) + RATIOS),
                            backward=rng.random() < 0.6, shape=shape)
            if work(case)["flops"] <= MOST_PREFILL_FLOPS and int(_trajectories(case)[2][-1]) <= 150000:
                return case
        else:
            V, T = log_int(1000, 152064), log_int(1, 4096)
            case = _distill(None, T=T, V=V, k=log_int(1, 256), dtype=rng.choice(("bf16", "bf16", "f32")))
            if T * V * (2 if case["dtype"] == "f32" else 1) <= MOST_LOGITS:
                return case


# ---------------------------------------------------------------------------
# shapes of a case, from the case alone
# ---------------------------------------------------------------------------
def _ints(r, lo, hi, n):
    return r.integers(lo, hi + 1, size=n).astype(np.int64)


def _ratios(r, case):
    if case["c"] >= 0:
        return np.full(case["B"], case["c"], dtype=np.int64)
    return r.choice(np.array(RATIOS, dtype=np.int64), size=case["B"])


def _caches(case):
    """(P, c, generated tokens, capacity) of every sequence, all [B]."""
    r = np.random.default_rng([case["shape"], 1])
    P, c = _ints(r, case["P_lo"], case["P_hi"], case["B"]), _ratios(r, case)
    gen = _ints(r, case["gen_lo"], case["gen_hi"], case["B"])
    end = gen + case["tokens"]
    cap = np.where(c > 0, P + end // np.maximum(c, 1) + c + 1, P + end)
    return P, c, gen, cap


def _tables(c, gen):
    cc = np.maximum(c, 1)
    return np.where(c > 0, gen // cc, 0), np.where(c > 0, gen % cc, gen)


def _trajectories(case):
    """(P, c, row offsets [B+1]) of the trajectories: prompt, response, one beacon per c response tokens."""
    r = np.random.default_rng([case["shape"], 2])
    P, c = _ints(r, case["P_lo"], case["P_hi"], case["B"]), _ratios(r, case)
    R = _ints(r, case["R_lo"], case["R_hi"], case["B"])
    rows = P + R + np.where(c > 0, R // np.maximum(c, 1), 0)
    return P, c, np.concatenate([[0], np.cumsum(rows)])


def _visible_pairs(rows, P, c):
    i = np.arange(rows, dtype=np.int64)
    if c <= 0:
        return int((i + 1).sum())
    u = np.maximum(i - P, 0)
    return int(np.where(i < P, i + 1, P + u // (c + 1) + u % (c + 1) + 1).sum())


# ---------------------------------------------------------------------------
def prepare(case, seed):
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev).manual_seed(int(seed))
    if case["kind"] == "decode":
        return _prepare_decode(case, dev, gen)
    if case["kind"] == "prefill":
        P, c, off = _trajectories(case)
        rows, d = int(off[-1]), case["d"]

        def rnd(h):
            return torch.randn(rows, h, d, generator=gen, device=dev).to(torch.bfloat16)

        state = dict(case=case, P=P.astype(np.int32), c=c.astype(np.int32), off=off, q=rnd(case["Hq"]), k=rnd(case["Hkv"]),
                     v=rnd(case["Hkv"]))
        if case["backward"]:
            state["dout"] = rnd(case["Hq"])
        return state
    # student logits N(0, 2^2); the teacher is the student plus N(0, 1), of which the k largest are kept
    T, V, k = case["T"], case["V"], case["k"]
    z = torch.empty(T, V, dtype=torch.bfloat16 if case["dtype"] == "bf16" else torch.float32, device=dev)
    tl = torch.empty(T, k, dtype=torch.float32, device=dev)
    idx = torch.empty(T, k, dtype=torch.int32, device=dev)
    for t in range(0, T, 1024):
        z[t:t + 1024] = 2.0 * torch.randn(z[t:t + 1024].shape, generator=gen, device=dev)
        teacher = z[t:t + 1024].float() + torch.randn(z[t:t + 1024].shape, generator=gen, device=dev)
        top = torch.topk(teacher, k, dim=1)
        tl[t:t + 1024], idx[t:t + 1024] = top.values, top.indices
    return dict(case=case, z=z, teacher=tl, idx=idx)


def _prepare_decode(case, dev, gen):
    B, Hq, Hkv, d, layers, tokens = (case[x] for x in ("B", "Hq", "Hkv", "d", "layers", "tokens"))
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    P, c, generated, cap = _caches(case)
    n = int(cap.sum()) * Hkv * d

    def rnd(*shape):
        return torch.randn(*shape, generator=gen, device=dev, dtype=torch.float32).to(dt)

    # one arena for the K (and V) rows of all layers, one tensor for all tables
    k_rows, v_rows = (torch.empty(layers, n, dtype=dt, device=dev) for _ in range(2))
    for layer in range(layers):
        k_rows[layer], v_rows[layer] = rnd(n), rnd(n)
    if case["peaked"]:
        k_rows.view(-1, d)[63::64] *= 4.0
    tables = torch.zeros(layers, 2, B, dtype=torch.int32, device=dev)
    start = torch.from_numpy(np.stack(_tables(c, generated)).astype(np.int32)).to(dev).expand(layers, 2, B).contiguous()
    caches = []
    for layer in range(layers):
        rt = bc.Runtime(B, Hq, Hkv, d, case["dtype"], 1.0 / math.sqrt(d), P, c, cap, dev)
        rt.k_slab, rt.v_slab, rt.nb, rt.w = k_rows[layer], v_rows[layer], tables[layer, 0], tables[layer, 1]
        rt.cache.k_slab, rt.cache.v_slab = rt.k_slab.data_ptr(), rt.v_slab.data_ptr()
        rt.cache.nb, rt.cache.w = rt.nb.data_ptr(), rt.w.data_ptr()
        caches.append(rt)
    state = dict(case=case, caches=caches, k_rows=k_rows, v_rows=v_rows, tables=tables, start=start, ends=c > 0,
                 outs=torch.zeros(tokens, layers, B, Hq, d, dtype=torch.float32, device=dev),
                 beacon_outs=torch.zeros(layers, B, Hq, d, dtype=torch.float32, device=dev),
                 new=[[dict(k=rnd(B, Hkv, d), v=rnd(B, Hkv, d), q=rnd(B, Hq, d), bk=rnd(B, Hkv, d), bv=rnd(B, Hkv, d))
                       for _ in range(layers)] for _ in range(tokens)])
    if case["graph"]:
        stream = torch.cuda.Stream()
        torch.cuda.synchronize()
        with torch.cuda.stream(stream):
            _tokens(state)                      # once by itself: nothing is loaded during the capture
            stream.synchronize()
            state["graph"] = torch.cuda.CUDAGraph()
            with torch.cuda.graph(state["graph"], stream=stream):
                _tokens(state)
        stream.synchronize()
    return state


def _tokens(s):
    case, caches = s["case"], s["caches"]
    torch.add(s["start"], 0, out=s["tables"])
    if case["sort"]:
        for rt in caches:
            rt.sort_by_length()
    compress = case["c"] != 0 and not case["own_beacon"]
    for t in range(case["tokens"]):
        for layer, rt in enumerate(caches):
            x = s["new"][t][layer]
            rt.decode_step(x["k"], x["v"], x["q"], x["bk"] if compress else None, x["bv"] if compress else None,
                           out=s["outs"][t, layer])
    if case["own_beacon"]:
        for layer, rt in enumerate(caches):
            x = s["new"][-1][layer]
            rt.beacon_step(x["bk"], x["bv"], x["q"], out=s["beacon_outs"][layer])


def run(state):
    case = state["case"]
    if case["kind"] == "decode":
        if case["graph"]:
            state["graph"].replay()
        else:
            _tokens(state)
        return [state["outs"], state["beacon_outs"], state["tables"], state["k_rows"], state["v_rows"]]
    if case["kind"] == "prefill":
        args = (state["off"], state["P"], state["c"], case["Hq"], case["Hkv"], case["d"], 1.0 / math.sqrt(case["d"]))
        q, k, v = state["q"], state["k"], state["v"]
        if not case["backward"]:
            return bc.prefill_attn(q, k, v, *args, workspace=True)
        out, lse = bc.prefill_attn(q, k, v, *args)
        return (out, lse) + tuple(bc.prefill_attn_bwd(q, k, v, out, lse, state["dout"], *args))
    loss, lse, mean = bc.topk_kl_loss(state["z"], state["teacher"], state["idx"])
    dz = bc.topk_kl_loss_bwd(state["z"], state["teacher"], state["idx"], lse, 1.0 / case["T"])
    return loss, lse, mean, dz


def work(case):
    if case["kind"] == "decode":
        P, c, gen, _ = _caches(case)
        es = 2 if case["dtype"] == "bf16" else 4
        entry, qrow = case["Hkv"] * case["d"] * 2 * es, case["Hq"] * case["d"]
        rows = 0
        for t in range(case["tokens"]):
            nb, w = _tables(c, gen + t)
            rows += int((P + nb + w + 1).sum())
        steps = case["tokens"]
        if case["own_beacon"]:
            nb, w = _tables(c, gen + case["tokens"] - 1)
            rows += int((P + nb + w + 2).sum())
            steps += 1
        # K and V rows in, the new row in and out again, the query in, the output (fp32) out
        byts = rows * entry + steps * case["B"] * (2 * entry + qrow * (es + 4))
        return {"bytes": case["layers"] * byts, "flops": case["layers"] * 4 * rows * qrow}
    if case["kind"] == "prefill":
        P, c, off = _trajectories(case)
        pairs = sum(_visible_pairs(int(off[b + 1] - off[b]), int(P[b]), int(c[b])) for b in range(case["B"]))
        rows, qrow, kvrow = int(off[-1]), case["Hq"] * case["d"], case["Hkv"] * case["d"]
        # forward: q, k, v in, out (fp32) and lse out; 2 products of every visible pair
        byts, flops = rows * (2 * qrow + 4 * kvrow + 4 * qrow + 4 * case["Hq"]), 4 * pairs * qrow
        if case["backward"]:         # the same and dout, out, lse in, dq, dk, dv (fp32) out; 5 products
            byts += rows * (2 * qrow + 4 * kvrow + 2 * qrow + 4 * qrow + 4 * case["Hq"] + 4 * qrow + 8 * kvrow)
            flops += 10 * pairs * qrow
        return {"bytes": byts, "flops": flops}
    es = 2 if case["dtype"] == "bf16" else 4
    T, V, k = case["T"], case["V"], case["k"]
    # the logits in for the loss, in again and the gradient out; the teacher's logits and ids twice
    return {"bytes": 3 * T * V * es + 2 * T * k * 8 + 3 * T * 4, "flops": 6 * T * V}


def tolerance(case):
    """About four times what the outputs differ by from the same sums in 64 bits."""
    if case["kind"] == "decode":
        # fp32 rows 1.2e-7; bf16 rows, whose softmax weights keep about 16 bits, 2e-6 (largest 1.4e-5)
        return {"rel": 1e-6, "max": 1e-5} if case["dtype"] == "f32" else {"rel": 1e-5, "max": 6e-5}
    if case["kind"] == "prefill":
        # 2.9e-6 (largest 8.9e-5), gradients included; the workspace form keeps 11 bits: 1.7e-4 (3e-3)
        return {"rel": 1.2e-5, "max": 3.6e-4} if case["backward"] else {"rel": 7e-4, "max": 1.2e-2}
    # the gradient is rounded to bf16 (1.6e-3, largest 2^-8); in fp32 loss and gradient are 8e-7 off (3e-5
    # where a probability and the teacher's cancel)
    return {"rel": 3e-3, "max": 8e-3} if case["dtype"] == "bf16" else {"rel": 4e-6, "max": 1.3e-4}
