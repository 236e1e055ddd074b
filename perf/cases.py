"""The band-attention work a user of this library has it do, as measurable cases.

Every case goes through the entry points of ``paper_2302_13451_amd.binding``:

* ``sa_forward``: inference over whole utterances (no log-sum-exp kept);
* ``sa_train`` / ``llsa_train`` / ``paper_train``: one attention layer's
  forward and backward, as a training step runs them;
* ``sa_stream`` / ``llsa_stream``: a whole session of S streams, one frame per
  step, from the first frame to the last emitted one.

A case's sizes: B utterances padded to T frames (the longest has T frames, the
others between T // 2 and T unless the case is not ``ragged``), H heads of d
features, windows of Lb past and La look-ahead frames, element type f32 or
bf16. For the streams B is the number of streams and T their frames.
"""

import math

import torch

from paper_2302_13451_amd import binding as bd

DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}
ELEM_BYTES = {"bf16": 2, "f32": 4}


def _case(op, dtype, B, T, H, d, Lb, La, ragged=True, name=None):
    c = {"op": op, "dtype": dtype, "B": B, "T": T, "H": H, "d": d, "Lb": Lb, "La": La,
         "ragged": ragged}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest call: one short utterance, a layer of two 32-wide heads,
        # float32 (a single request; launch and call latency)
        _case("sa_forward", "f32", 1, 64, 2, 32, 8, 2, False, "sa_infer_f32_one_utterance"),
        # the paper's l32_r8 window on a batch of ten-second utterances of a
        # base-size encoder (12 heads of 64): plain inference
        _case("sa_forward", "bf16", 8, 500, 12, 64, 32, 8, False, "sa_infer_l32_r8"),
        # a training step of the same encoder at the benchmark's window, batch
        # of 8 to 16 second utterances padded to the longest
        _case("sa_train", "bf16", 16, 800, 12, 64, 64, 8, True, "sa_train_l64_r8"),
        # the widest window of the paper's memory experiment (W = 490, 1000
        # frames, 16 heads), training
        _case("sa_train", "bf16", 4, 1000, 16, 64, 481, 8, True, "sa_train_w490"),
        # many short utterances of a small model with 32-wide heads
        _case("sa_train", "bf16", 96, 131, 8, 32, 64, 8, True, "sa_train_short_d32"),
        # float32 training (the paper's PyTorch modules run in float32)
        _case("sa_train", "f32", 8, 500, 12, 64, 32, 8, True, "sa_train_f32_l32_r8"),
        # two-branch LLSA training at the benchmark's window
        _case("llsa_train", "bf16", 16, 800, 12, 64, 64, 8, True, "llsa_train_l64_r8"),
        # two-branch LLSA on half-minute utterances with an odd, wider window
        _case("llsa_train", "bf16", 3, 1501, 8, 64, 181, 12, True, "llsa_train_w194"),
        # two-branch LLSA in float32 at the paper's l32_r16 window
        _case("llsa_train", "f32", 4, 500, 12, 64, 32, 16, True, "llsa_train_f32_l32_r16"),
        # the paper's own LLSA, nine channels, training: the largest case
        _case("paper_train", "bf16", 16, 800, 12, 64, 64, 8, True, "llsa_paper_train_l64_r8"),
        # streaming serving: 64 streams of about three seconds
        _case("sa_stream", "bf16", 64, 152, 12, 64, 64, 8, True, "sa_stream_64"),
        # LLSA streaming with many streams, l32_r16
        _case("llsa_stream", "bf16", 250, 100, 12, 64, 32, 16, True, "llsa_stream_250"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# how often a drawn case takes each kind of work
_OPS = ["sa_forward"] * 3 + ["sa_train"] * 4 + ["llsa_train"] * 4 + ["paper_train"] * 2 + \
       ["sa_stream", "llsa_stream"]


def draw(rng):
    """One more case of the same ranges: 1 to 128 utterances of 20 to 3000
    frames (a minute at 20 ms), 1 to 256 streams, 1 to 16 heads of 32 or 64,
    look-back 0 to 481, look-ahead 0 to 32 (the paper's form: up to 128 and 16,
    that is 17 channels), both element types."""
    top = work(next(c for c in listed() if c["name"] == "llsa_paper_train_l64_r8"))
    while True:
        op = rng.choice(_OPS)
        dtype = "f32" if rng.random() < 0.35 else "bf16"
        d = 32 if rng.random() < 0.25 else 64
        H = rng.choice([1, 2, 3, 4, 6, 8, 12, 12, 16])
        Lb = rng.choice([0, 16, 32, 64]) if rng.random() < 0.3 else _log_int(rng, 4, 481)
        La = rng.choice([0, 8, 16]) if rng.random() < 0.5 else rng.randint(1, 32)
        ragged = rng.random() < 0.75
        if op.endswith("stream"):
            B, T = _log_int(rng, 1, 256), rng.randint(40, 200)
        else:
            B, T = _log_int(rng, 1, 128), _log_int(rng, 20, 3000)
        if op == "paper_train":
            La = min(La, 16)
            Lb = min(Lb, 128)
        if Lb + La == 0:  # a frame that sees only itself is no attention
            continue
        c = _case(op, dtype, B, T, H, d, Lb, La, ragged)
        w = work(c)
        # float32 has a fifteenth of the bfloat16 matrix rate and twice the bytes
        most = 0.06 if dtype == "f32" else 0.5
        if w["bytes"] <= 0.5 * top["bytes"] and w["flops"] <= most * top["flops"]:
            return c


def _lengths(case, seed):
    """Valid frames of every utterance (stream): the longest has T."""
    B, T = case["B"], case["T"]
    if not case["ragged"]:
        return [T] * B
    g = torch.Generator().manual_seed(1000003 * int(seed) + 17)
    L = torch.randint(max(1, T // 2), T + 1, (B,), generator=g).tolist()
    L[B // 2] = T
    return L


def _channels(case):
    return {"llsa_train": 2, "paper_train": case["La"] + 1}.get(case["op"], 0)


def _inputs(case, seed):
    """q, k, v, dout ([channels][B][T][H][d], no leading dimension for SA),
    N(0, 1) in the case's type (scores then have a standard deviation of one),
    padding frames zero; lengths int32 [B] (None when every utterance is full)."""
    B, T, H, d, C = case["B"], case["T"], case["H"], case["d"], _channels(case)
    shape = ((C,) if C else ()) + (B, T, H, d)
    g = torch.Generator(device="cuda").manual_seed(int(seed))
    L = _lengths(case, seed)
    ln = torch.tensor(L, dtype=torch.int32).cuda() if case["ragged"] else None
    x = {}
    for n in ("q", "k", "v", "dout"):
        x[n] = torch.randn(shape, generator=g, device="cuda").to(DTYPES[case["dtype"]])
        if ln is not None:
            pad = torch.arange(T, device="cuda")[None, :] >= ln[:, None]
            x[n].masked_fill_(pad.view((1,) * bool(C) + (B, T, 1, 1)), 0)
    return x, ln


def _frames(case, seed):
    """A session's frames: one [B][H][d] tensor per step and input, N(0, 1)."""
    B, H, d = case["B"], case["H"], case["d"]
    g = torch.Generator(device="cuda").manual_seed(int(seed))
    names = ("q", "k", "v") if case["op"] == "sa_stream" else ("qc", "kc", "vc", "ql", "kl", "vl")
    steps = case["T"] + case["La"]
    return {n: torch.randn((steps, B, H, d), generator=g, device="cuda").to(DTYPES[case["dtype"]])
            for n in names}


def prepare(case, seed):
    if not case["op"].endswith("stream"):
        x, ln = _inputs(case, seed)
        return {"case": case, "x": x, "lengths": ln}
    f = _frames(case, seed)
    kind = bd.StreamState if case["op"] == "sa_stream" else bd.LlsaStreamState
    st = kind(case["B"], case["H"], case["d"], case["Lb"], case["La"],
              lengths=_lengths(case, seed) if case["ragged"] else None,
              dtype=DTYPES[case["dtype"]])
    # frames arrive one by one: what a step has in hand is one contiguous frame
    # of every stream
    return {"case": case, "state": st, "frames": [list(t.unbind(0)) for t in f.values()]}


def run(state):
    case = state["case"]
    op, Lb, La = case["op"], case["Lb"], case["La"]
    if op.endswith("stream"):
        st, fr = state["state"], state["frames"]
        steps = case["T"] + La
        st.step_ctr.zero_()  # a new session
        if op == "sa_stream":
            out = torch.empty((steps,) + tuple(fr[0][0].shape), dtype=fr[0][0].dtype, device="cuda")
            for o, q, k, v in zip(out.unbind(0), *fr):
                bd.sa_stream_step(st, q, k, v, o)
            return {"out": out}
        out = torch.empty((2, steps) + tuple(fr[0][0].shape), dtype=fr[0][0].dtype, device="cuda")
        for oc, ol, qc, kc, vc, ql, kl, vl in zip(out[0].unbind(0), out[1].unbind(0), *fr):
            bd.llsa_stream_step(st, qc, kc, vc, ql, kl, vl, oc, ol)
        return {"out": out}
    x, ln = state["x"], state["lengths"]
    q, k, v = x["q"], x["k"], x["v"]
    if op == "sa_forward":
        out, _ = bd.sa_forward(q, k, v, Lb, La, ln, want_lse=False)
        return {"out": out}
    fwd, bwd = {"sa_train": (bd.sa_forward, bd.sa_backward),
                "llsa_train": (bd.llsa_forward, bd.llsa_backward),
                "paper_train": (bd.llsa_paper_forward, bd.llsa_paper_backward)}[op]
    out, lse = fwd(q, k, v, Lb, La, ln)
    dq, dk, dv = bwd(q, k, v, out, lse, x["dout"], Lb, La, ln)
    return {"out": out, "lse": lse, "dq": dq, "dk": dk, "dv": dv}


def _pairs(L, Lb, La):
    """(query, key) pairs of one utterance of L frames and one head."""
    return sum(min(L - 1, t + La) - max(0, t - Lb) + 1 for t in range(L))


def work(case):
    B, T, H, d, Lb, La = (case[n] for n in ("B", "T", "H", "d", "Lb", "La"))
    e = ELEM_BYTES[case["dtype"]]
    # utterances of the mean length (the lengths themselves come with the seed)
    L = (3 * T + 3) // 4 if case["ragged"] else T
    frames = B * L
    if case["op"].endswith("stream"):
        row = H * d * e
        pairs = B * _pairs(L, Lb, La)
        if case["op"] == "sa_stream":
            # per emitted frame its window's keys and values, the query and the
            # output; per arriving frame q, k, v in and into the rings
            return {"bytes": row * (2 * pairs + 2 * frames + 6 * frames),
                    "flops": 4 * d * H * pairs}
        # one window serves both outputs; 4 keys and values in and into the rings
        return {"bytes": row * (2 * pairs + 4 * frames + 8 * frames),
                "flops": 2 * 4 * d * H * pairs}
    C = max(1, _channels(case))
    if case["op"] == "llsa_train":
        pairs = _pairs(L, Lb + La, 0) + _pairs(L, Lb, La)
    elif case["op"] == "paper_train":
        pairs = sum(_pairs(L, La + Lb - c, c) for c in range(La + 1))
    else:
        pairs = _pairs(L, Lb, La)
    pairs *= B * H
    if case["op"] == "sa_forward":
        return {"bytes": 4 * frames * H * d * e, "flops": 4 * d * pairs}
    # forward: q, k, v in, out and lse out; backward: q, k, v, out, dout and lse
    # in, dq, dk, dv out (12 products of d per pair, nothing recomputed)
    return {"bytes": C * frames * H * (12 * d * e + 8), "flops": 12 * d * pairs}


def tolerance(case):
    """About four times the largest error of any output against 64 bits, over
    the listed cases and forty drawn ones: float32 4.9e-7 (largest element
    1.2e-5 of its tensor's root mean square); bfloat16 outputs 2.3e-3 (2.4e-2)
    from an MFMA forward with weights rounded to bfloat16 and 1.7e-3 (3.9e-3)
    from the streaming steps, gradients 2.9e-3 (6.8e-2)."""
    if case["dtype"] == "f32":
        return {"rel": 2e-6, "max": 5e-5}
    if case["op"].endswith("stream"):
        return {"rel": 7e-3, "max": 0.016}
    if case["op"] == "sa_forward":
        return {"rel": 9e-3, "max": 0.1}
    return {"rel": 1.2e-2, "max": 0.27}


def _attend(q, k, v, segs, ln):
    """Band attention of one output in 64 bits: q [B][T][H][d], k and v lists
    of such tensors (one per branch), segs a list of (branch, lo, hi): query t
    reads frames t + lo .. t + hi of that branch, clipped to the utterance.
    Returns out [B][T][H][d] and lse [B][H][T]."""
    B, T, H, d = q.shape
    dev = q.device
    pos = torch.arange(T, device=dev)
    n = ln.view(B, 1, 1, 1)
    outs, lses = [], []
    step = 128
    for t0 in range(0, T, step):
        t1 = min(T, t0 + step)
        tq = pos[t0:t1].view(1, 1, -1, 1)
        qc = q[:, t0:t1].transpose(1, 2).contiguous()
        zs, vs = [], []
        for br, lo, hi in segs:
            a, b = max(0, t0 + lo), min(T, t1 + hi)
            if a >= b:
                continue
            kc = k[br][:, a:b].permute(0, 2, 3, 1).contiguous()
            tk = pos[a:b].view(1, 1, 1, -1)
            z = torch.matmul(qc, kc) / math.sqrt(d)
            inside = (tk >= tq + lo) & (tk <= tq + hi) & (tk < n)
            zs.append(z.masked_fill(~inside, float("-inf")))
            vs.append(v[br][:, a:b].transpose(1, 2))
        z = torch.cat(zs, 3)
        pad = (tq >= n)
        m = torch.logsumexp(z.masked_fill(pad, 0.0), 3, keepdim=True)
        p = torch.exp(z - m).masked_fill(pad, 0.0)
        outs.append(torch.matmul(p, torch.cat(vs, 2).contiguous()).transpose(1, 2))
        lses.append(m.masked_fill(pad, float("-inf"))[..., 0])
    return torch.cat(outs, 1), torch.cat(lses, 2)


def _segments(case):
    """Per output its window segments (branch, lo, hi); output o takes the
    query of branch o."""
    Lb, La = case["Lb"], case["La"]
    if case["op"] in ("sa_forward", "sa_train", "sa_stream"):
        return [[(0, -Lb, La)]]
    if case["op"] in ("llsa_train", "llsa_stream"):
        return [[(1, -La - Lb, -La), (0, 1 - La, 0)], [(1, -Lb, 0), (0, 1, La)]]
    return [[(La, c - La - Lb, c - La)] + [(i, c - i, c - i) for i in range(La)]
            for c in range(La + 1)]


def _all_outputs(case, q, k, v, ln):
    r = [_attend(q[o], k, v, segs, ln) for o, segs in enumerate(_segments(case))]
    return [x[0] for x in r], [x[1] for x in r]


def exact(case, seed):
    B, T, La = case["B"], case["T"], case["La"]
    if case["op"].endswith("stream"):
        f = {n: x.double() for n, x in _frames(case, seed).items()}
        ln = torch.tensor(_lengths(case, seed)).cuda()
        sa = case["op"] == "sa_stream"
        x = {}
        for n, t in f.items():
            # branch L's frame t arrives at step t + La
            lead = La if not sa and n.endswith("l") else 0
            x[n] = t[lead:lead + T].transpose(0, 1)
        if case["ragged"]:
            end = ln
        else:
            # open-ended: every step's frame counts, to the last one fed
            end = torch.full((B,), T + La, device="cuda")
            x = {n: t[(La if not sa and n.endswith("l") else 0):].transpose(0, 1)
                 for n, t in f.items()}
            if not sa:
                x = {n: torch.cat([t, torch.zeros_like(t[:, :La])], 1) if n.endswith("l") else t
                     for n, t in x.items()}
        if sa:
            q, k, v = [x["q"]], [x["k"]], [x["v"]]
        else:
            q, k, v = ([x[n + "c"], x[n + "l"]] for n in "qkv")
        out, _ = _all_outputs(case, q, k, v, end)
        steps = T + La
        def at_steps(o, late):
            o = o.transpose(0, 1)
            o = torch.cat([torch.zeros_like(o[:late]), o])[:steps]
            return torch.cat([o, torch.zeros_like(o[:1]).expand(steps - o.shape[0], -1, -1, -1)])
        if sa:
            return {"out": at_steps(out[0], La)}
        return {"out": torch.stack([at_steps(out[0], 0), at_steps(out[1], La)])}
    x, ln = _inputs(case, seed)
    ln = torch.full((B,), T, device="cuda") if ln is None else ln.long()
    x = {n: t.double() for n, t in x.items()}
    if not _channels(case):
        x = {n: t[None] for n, t in x.items()}
    if case["op"] == "sa_forward":
        out, _ = _all_outputs(case, x["q"], x["k"], x["v"], ln)
        return {"out": out[0]}
    q, k, v = (x[n].requires_grad_(True) for n in "qkv")
    outs, lses, grads = [], [], [torch.zeros_like(q) for _ in range(3)]
    for o, segs in enumerate(_segments(case)):  # one output at a time bounds the graph kept
        out, lse = _attend(q[o], k, v, segs, ln)
        for acc, gr in zip(grads, torch.autograd.grad(out, (q, k, v), x["dout"][o])):
            acc += gr
        outs.append(out.detach())
        lses.append(lse.detach())
    r = {"out": torch.stack(outs), "lse": torch.stack(lses), "dq": grads[0], "dk": grads[1],
         "dv": grads[2]}
    return r if _channels(case) else {n: t[0] for n, t in r.items()}
