"""What is timed of this library: calls of its C ABI on one frozen projection, as a base executor makes them.

A case is one projection, one flattened batch of clients and one flow:

  serve     forward of inference clients (decode steps of one token, prompts), every client's adapter fused
  tune      forward of all clients, then adapter gradients and input gradient of the fine-tuning ones, in the
            order and with the workspace hand-over of a training step (Hs from the forward, dH between the two)
  executor  what the paper's executor does alone: forward and input gradient without adapters
  private   the privacy flow: noise added to the activations, forward that takes the noise effect off again

One-token inference clients come first in a batch, as the batching queue forms it; the rows of the
fine-tuning clients are then a contiguous view, so that no gather is part of a pass.  Shapes, client counts, ranks and
value laws are those of `synth` (Llama2-7B-, Granite-20B-, Gemma2-27B-shaped layers, the mixed batch), plus ragged ones.
"""
import functools
import math
import random

import torch

from paper_2507_03220_amd import binding as sb

BF16 = torch.bfloat16
NONE, LORA, IA3, IA3_IN = sb.SYMB_ADAPTER_NONE, sb.SYMB_ADAPTER_LORA, sb.SYMB_ADAPTER_IA3, sb.SYMB_ADAPTER_IA3_IN


def _case(flow, d_in, d_out, decode=0, clients=0, tokens=0, equal=False, ranks="", ia3=0.0, ia3_in=0.0, bias=False, conv1d=False,
          per_client=False, mix=1):
    """decode: one-token inference clients; clients / tokens: the longer ones and their tokens together (equal: all of one length);
    ranks: the LoRA ranks in use ("" = no LoRA client); ia3 / ia3_in: shares of clients that scale outputs / inputs instead; mix:
    seed of lengths, ranks and kinds."""
    return dict(flow=flow, d_in=d_in, d_out=d_out, decode=decode, clients=clients, tokens=tokens, equal=equal, ranks=ranks, ia3=ia3,
                ia3_in=ia3_in, bias=bias, conv1d=conv1d, per_client=per_client, mix=mix)


def listed():
    def c(name, *a, **k):
        return dict(_case(*a, **k), name=name)
    return [
        # one user's decode step through an attention projection: the smallest call there is
        c("decode_one", "serve", 4096, 4096, decode=1, ranks="16"),
        # a small decode batch of clients with adapters of their own, up projection
        c("decode_sixteen", "serve", 4096, 11008, decode=16, ranks="4,8,16,32,64", ia3=0.25, mix=2),
        # the decode half of the mixed batch: 48 clients, half of them IA3, ranks to 128, down projection
        c("decode_mixed", "serve", 11008, 4096, decode=48, ranks="4,8,16,32,64,128", ia3=0.5, mix=3),
        # training step of one client with the shortest sequence of the mixed workload
        c("tune_short", "tune", 4096, 4096, clients=1, tokens=16, ranks="16"),
        # training step of the tiny configuration: 4 clients x 64 tokens on a 768-wide layer
        c("tune_tiny", "tune", 768, 768, clients=4, tokens=256, equal=True, ranks="8"),
        # three prompts of uneven length with eight decode steps riding along, biased layer
        c("prefill_ragged", "serve", 4096, 11008, decode=8, clients=3, tokens=389, ranks="8,16,32,64", bias=True, mix=4),
        # the executor of the paper on an input-major (Conv1D) weight, every client in a buffer of its own
        c("executor_conv1d", "executor", 6144, 6144, clients=5, tokens=731, bias=True, conv1d=True, per_client=True, mix=5),
        # clients that hide their activations, LoRA on top
        c("private", "private", 4608, 4096, clients=4, tokens=2000, ranks="16", bias=True, mix=6),
        # eight fine-tuning clients on a Llama2-7B-shaped attention projection, ranks 8 to 64
        c("tune_llama_q", "tune", 4096, 4096, clients=8, tokens=10240, ranks="8,16,32,64", mix=7),
        # the mixed batch on its widest projection: 48 decode steps beside 16 fine-tuning clients, LoRA to rank 128 and IA3
        c("mixed_gate", "tune", 4096, 11008, decode=48, clients=16, tokens=9001, ranks="4,8,16,32,64,128", ia3=0.5, mix=8),
        # multi-query key/value projection: a narrow output, where the adapter passes weigh most
        c("tune_mqa_kv", "tune", 6144, 256, clients=16, tokens=16384, equal=True, ranks="8"),
        # the gate projection of the Gemma2-27B-shaped training step: the largest launch
        c("tune_gemma_gate", "tune", 4608, 36864, clients=20, tokens=20480, equal=True, ranks="8,16", mix=9),
    ]


# rough cost of a pass, used to keep drawn cases below the largest listed one: products, and passes over the rows
def _cost(c):
    rows = c["decode"] + c["tokens"]
    return rows * c["d_in"] * c["d_out"] * (2 if c["flow"] in ("tune", "executor") else 1)


def draw(rng):
    """Flows, options and sizes of the same ranges: widths 256..36864 (the configurations' own and ragged multiples of 8), batches
    of 1 to 20480 rows, 1 to 64 clients."""
    most = max(_cost(c) for c in listed())
    while True:
        flow = rng.choice(["serve", "serve", "tune", "tune", "tune", "executor", "private"])

        def width():
            if rng.random() < 0.5:
                return rng.choice([768, 2048, 4096, 4608, 6144, 11008, 24576, 36864])
            return 8 * int(round(math.exp(rng.uniform(math.log(32), math.log(2048)))))
        d_in, d_out = width(), width()
        decode = rng.choice([0, 1, rng.randint(2, 16), rng.randint(17, 64)]) if flow in ("serve", "tune") else 0
        clients = rng.randint(0 if decode and flow == "serve" else 1, 20)
        tokens = 0
        if clients:
            tokens = max(clients, int(math.exp(rng.uniform(math.log(16), math.log(20480)))))
        per_client = flow in ("serve", "executor") and rng.random() < 0.3
        ranks, ia3, ia3_in = "", 0.0, 0.0
        if flow != "executor":
            ranks = rng.choice(["8", "16", "8,16", "8,16,32,64", "4,8,16,32,64,128", "5,12,23,40,100"])
            # (a per-client forward has no pre-adapter output: IA3 there is for inference)
            ia3 = rng.choice([0.0, 0.0, 0.25, 0.5])
            ia3_in = rng.choice([0.0, 0.0, 0.25]) if flow != "private" else 0.0
        c = _case(flow, d_in, d_out, decode, clients, tokens, rng.random() < 0.3, ranks, ia3, ia3_in, rng.random() < 0.3,
                  rng.random() < 0.2, per_client, rng.randrange(1 << 20))
        if _cost(c) <= most:
            return c


def _segments(c):
    """[(tokens, kind, rank, scale, fine-tuning)] of the batch, from the case alone."""
    r = random.Random(c["mix"])
    lens = []
    if c["clients"]:
        if c["equal"]:
            base, more = divmod(c["tokens"], c["clients"])
            lens = [base + (i < more) for i in range(c["clients"])]
        else:                                     # uneven: exponential shares, at least one token each
            w = [r.expovariate(1.0) + 0.05 for _ in range(c["clients"])]
            left = c["tokens"] - c["clients"]
            lens = [1 + int(left * x / sum(w)) for x in w]
            lens[0] += c["tokens"] - sum(lens)
    ranks = [int(x) for x in c["ranks"].split(",") if x]
    segs = []
    for i, n in enumerate([1] * c["decode"] + lens):
        u, kind, rank, scale = r.random(), NONE, 0, 0.0
        if u < c["ia3"]:
            kind = IA3
        elif u < c["ia3"] + c["ia3_in"]:
            kind = IA3_IN
        elif ranks:
            kind, rank, scale = LORA, r.choice(ranks), 2.0
        segs.append((n, kind, rank, scale, i >= c["decode"]))
    return segs


@functools.lru_cache(maxsize=None)
def _handle():
    return sb.symb_create(torch.cuda.current_device())


def _make(c, seed):
    """The tensors of a case: values by the laws of `synth`."""
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 1000003 + 17)

    def normal(*shape, std=1.0, mean=0.0):
        t = torch.randn(*shape, device="cuda", dtype=BF16, generator=g)
        return t if std == 1.0 and mean == 0.0 else (t.float() * std + mean).to(BF16)
    d_in, d_out, segs = c["d_in"], c["d_out"], _segments(c)
    off = [0]
    for s in segs:
        off.append(off[-1] + s[0])
    t0 = c["decode"]                                           # first row of the fine-tuning clients
    d = dict(c=c, segs=segs, off=off, t0=t0, X=normal(off[-1], d_in))
    w = normal(d_out, d_in, std=1.0 / math.sqrt(d_in))
    d["W"] = w.t().contiguous() if c["conv1d"] else w
    d["bias"] = normal(d_out, std=0.5) if c["bias"] else None
    d["ad"] = []
    for n, kind, rank, scale, _ in segs:
        if kind == LORA:
            d["ad"].append((normal(rank, d_in, std=1.0 / math.sqrt(d_in)), normal(d_out, rank, std=1.0 / math.sqrt(rank))))
        elif kind in (IA3, IA3_IN):
            d["ad"].append((normal(d_out if kind == IA3 else d_in, std=0.1, mean=1.0), None))
        else:
            d["ad"].append((None, None))
    if c["flow"] in ("tune", "executor"):
        d["dY"] = normal(off[-1] - t0, d_out)
    if c["flow"] == "private":
        d["noise"] = normal(off[-1], d_in)
        # what a client keeps for a noise value: the layer's response to it, in 16 bits
        w32 = (d["W"].t() if c["conv1d"] else d["W"]).float()
        eff = d["noise"].float() @ w32.t()
        for i, (n, kind, rank, scale, _) in enumerate(segs):
            rows = slice(off[i], off[i + 1])
            if kind == LORA:
                eff[rows] += scale * (d["noise"][rows].float() @ d["ad"][i][0].float().t()) @ d["ad"][i][1].float().t()
            elif kind == IA3:
                eff[rows] *= d["ad"][i][0].float()
        d["noise_effect"] = eff.to(BF16)
    return d


def prepare(case, seed):
    s = _make(case, seed)
    c, segs, off, t0 = s["c"], s["segs"], s["off"], s["t0"]
    d_in, d_out, T = c["d_in"], c["d_out"], off[-1]
    s["h"], s["stream"] = _handle(), torch.cuda.current_stream().cuda_stream
    layout = sb.SYMB_WEIGHT_CONV1D if c["conv1d"] else sb.SYMB_WEIGHT_LINEAR
    ads = [sb.Adapter(k, r, sc, A, B) for (n, k, r, sc, _), (A, B) in zip(segs, s["ad"])]
    s["fwd"] = sb.Batch(d_in, d_out, off, ads, layout)
    s["Y"] = torch.empty(T, d_out, device="cuda", dtype=BF16)
    need = sb.symb_workspace_bytes(s["fwd"], sb.SYMB_OP_FWD)
    flow, tuned = c["flow"], range(c["decode"], len(segs))
    if flow == "tune":
        s["has_ia3"] = any(segs[i][1] == IA3 for i in tuned)
        s["has_in"] = any(segs[i][1] == IA3_IN for i in tuned)
        s["Ybase"] = torch.empty_like(s["Y"]) if s["has_ia3"] else None
        s["dXbase"] = torch.empty(T - t0, d_in, device="cuda", dtype=BF16) if s["has_in"] else None
        n = [sum(segs[i][2] for i in tuned) * d_in, sum(segs[i][2] for i in tuned) * d_out,
             sum({IA3: d_out, IA3_IN: d_in}.get(segs[i][1], 0) for i in tuned)]
        s["dA"], s["dB"], s["dl"] = (torch.zeros(x, device="cuda") for x in n)
        a = b = l = 0
        back = []
        for i in tuned:
            _, k, r, sc, _ = segs[i]
            x = sb.Adapter(k, r, sc, *s["ad"][i])
            if k == LORA:
                x.dA, x.dB = s["dA"][a:], s["dB"][b:]
                a, b = a + r * d_in, b + r * d_out
            elif k in (IA3, IA3_IN):
                x.dA = s["dl"][l:]
                l += d_out if k == IA3 else d_in
            back.append(x)
    elif flow == "executor":
        back = [sb.Adapter() for _ in tuned]
    if flow in ("tune", "executor"):
        s["bwd"] = sb.Batch(d_in, d_out, [off[i] - t0 for i in range(c["decode"], len(segs) + 1)], back, layout)
        s["dX"] = torch.empty(T - t0, d_in, device="cuda", dtype=BF16)
        need = max(need, sb.symb_workspace_bytes(s["bwd"], sb.SYMB_OP_BWD_INPUT), sb.symb_workspace_bytes(s["bwd"], sb.SYMB_OP_ADAPTER_GRAD))
    if flow == "private":
        s["Xn"] = torch.empty_like(s["X"])
        cut = list(zip(off, off[1:]))
        s["n_seg"], s["e_seg"] = [s["noise"][a:b] for a, b in cut], [s["noise_effect"][a:b] for a, b in cut]
    if c["per_client"]:                                         # one arena each, a buffer per client in it
        cut = list(zip(off, off[1:]))
        s["X_seg"], s["Y_seg"] = [s["X"][a:b] for a, b in cut], [s["Y"][a:b] for a, b in cut]
        if flow == "executor":
            s["dY_seg"], s["dX_seg"] = [s["dY"][a:b] for a, b in cut], [s["dX"][a:b] for a, b in cut]
    s["ws"] = torch.empty(max(need, 256), device="cuda", dtype=torch.uint8)
    return s


def run(s):
    c, h, ws, stream = s["c"], s["h"], s["ws"], s["stream"]
    flow = c["flow"]
    if flow == "private":
        sb.symb_noise_add(h, s["fwd"], s["X"], s["n_seg"], s["Xn"], stream)
        sb.symb_base_linear_fwd_denoise(h, s["fwd"], s["Xn"], s["W"], s["bias"], s["e_seg"], s["Y"], ws, stream)
        return {"Xn": s["Xn"], "Y": s["Y"]}
    if c["per_client"]:
        sb.symb_base_linear_fwd_seg(h, s["fwd"], s["X_seg"], s["W"], s["bias"], s["Y_seg"], ws, stream)
        if flow == "serve":
            return {"Y": s["Y"]}
        sb.symb_base_linear_bwd_input_seg(h, s["bwd"], s["dY_seg"], s["W"], s["dX_seg"], sb.SYMB_BWD_BASE_ONLY, ws, stream)
        return {"Y": s["Y"], "dX": s["dX"]}
    sb.symb_base_linear_fwd(h, s["fwd"], s["X"], s["W"], s["bias"], s["Y"], s.get("Ybase"), ws, stream)
    if flow == "serve":
        return {"Y": s["Y"]}
    if flow == "executor":
        sb.symb_base_linear_bwd_input(h, s["bwd"], s["dY"], s["W"], s["dX"], sb.SYMB_BWD_BASE_ONLY, ws, stream)
        return {"Y": s["Y"], "dX": s["dX"]}
    t0 = s["t0"]
    X, Ybase = s["X"][t0:], s["Ybase"][t0:] if s["has_ia3"] else None
    hs = sb.SYMB_GRAD_REUSE_HS if t0 == 0 else 0                # the forward's batch is the backward's only without decode steps
    if s["has_in"]:                                             # dl of an input scale needs the input gradient before it
        sb.symb_base_linear_bwd_input_ex(h, s["bwd"], s["dY"], s["W"], s["dX"], s["dXbase"], sb.SYMB_BWD_FULL, ws, stream)
        sb.symb_adapter_grad_ex(h, s["bwd"], X, s["dY"], Ybase, s["dXbase"], sb.SYMB_GRAD_REUSE_DH | hs, ws, stream)
    else:
        sb.symb_adapter_grad(h, s["bwd"], X, s["dY"], Ybase, sb.SYMB_GRAD_OVERWRITE | hs, ws, stream)
        sb.symb_base_linear_bwd_input(h, s["bwd"], s["dY"], s["W"], s["dX"], sb.SYMB_BWD_REUSE_DH, ws, stream)
    out = {"Y": s["Y"], "dX": s["dX"], "dA": s["dA"], "dB": s["dB"], "dl": s["dl"]}
    if Ybase is not None:
        out["Ybase"] = s["Ybase"]
    return {k: v for k, v in out.items() if v.numel()}


def work(case):
    """Each tensor once; products of 2 rows d_in d_out per direction and 2 r (d_in + d_out) per LoRA token and pass over it."""
    c, segs = case, _segments(case)
    d_in, d_out = c["d_in"], c["d_out"]
    T = sum(s[0] for s in segs)
    Tb = T - c["decode"]
    back = c["flow"] in ("tune", "executor")
    nbytes = 2.0 * (T * (d_in + d_out) + d_in * d_out + (d_out if c["bias"] else 0))
    flops = 2.0 * T * d_in * d_out
    if back:
        nbytes += 2.0 * Tb * (d_in + d_out)
        flops += 2.0 * Tb * d_in * d_out
    if c["flow"] == "private":
        nbytes += 2.0 * T * (2 * d_in + d_out)                  # the noise, its sum with X, the noise effect
        flops += T * (d_in + d_out)
    for n, kind, rank, _, ft in segs:
        grads = c["flow"] == "tune" and ft
        if kind == LORA:
            nbytes += (2.0 + (4.0 if grads else 0.0)) * rank * (d_in + d_out)
            flops += (6.0 if grads else 2.0) * n * rank * (d_in + d_out)
        elif kind in (IA3, IA3_IN):
            w = d_out if kind == IA3 else d_in
            nbytes += (2.0 + (4.0 if grads else 0.0)) * w + (2.0 * n * w if grads else 0.0)
            flops += (3.0 if grads else 1.0) * n * w
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """Outputs are bf16 values rounded once from fp32 sums: 1.7e-3 of the result's norm and 1.4e-2 of its root mean square off
    the 64-bit result, at every size."""
    return {"rel": 7e-3, "max": 6e-2}


def exact(case, seed):
    s = _make(case, seed)
    c, segs, off, t0 = s["c"], s["segs"], s["off"], s["t0"]
    f64 = torch.float64
    W = (s["W"].t() if c["conv1d"] else s["W"]).to(f64)         # [d_out][d_in]
    X = s["X"]
    out = {}
    if c["flow"] == "private":
        X = (X.float() + s["noise"].float()).to(BF16)
        out["Xn"] = X.to(f64)
    rows = [slice(a, b) for a, b in zip(off, off[1:])]
    Xs = X.to(f64)
    for i, seg in enumerate(segs):
        if seg[1] == IA3_IN:
            Xs[rows[i]] *= s["ad"][i][0].to(f64)
    Y = Xs @ W.t()
    del Xs
    if c["bias"]:
        Y += s["bias"].to(f64)
    keep_base = c["flow"] == "tune" and any(k == IA3 for _, k, _, _, ft in segs if ft)
    if keep_base:
        out["Ybase"] = Y.clone()
    tune = c["flow"] == "tune"
    dA, dB, dl = [], [], []
    if c["flow"] in ("tune", "executor"):
        G = s["dY"].to(f64)
        for i in range(c["decode"], len(segs)):
            if segs[i][1] == IA3:
                G[off[i] - t0:off[i + 1] - t0] *= s["ad"][i][0].to(f64)
        dX = G @ W
        del G
    for i, (n, kind, rank, scale, ft) in enumerate(segs):
        A, B = (None if t is None else t.to(f64) for t in s["ad"][i])
        back = tune and ft
        if back:
            br = slice(off[i] - t0, off[i + 1] - t0)
            x, dy = X[rows[i]].to(f64), s["dY"][br].to(f64)
        if kind == LORA:
            H = scale * (X[rows[i]].to(f64) @ A.t())
            if back:
                dH = scale * (dy @ B)
                dA.append((dH.t() @ x).reshape(-1))
                dB.append((dy.t() @ H).reshape(-1))
                dX[br] += dH @ A
            Y[rows[i]] += H @ B.t()
        elif kind == IA3:
            if back:
                dl.append((dy * Y[rows[i]]).sum(0))
            Y[rows[i]] *= A
        elif kind == IA3_IN and back:
            dl.append((x * dX[br]).sum(0))
            dX[br] *= A
    if c["flow"] == "private":
        Y -= s["noise_effect"].to(f64)
    out["Y"] = Y
    if c["flow"] in ("tune", "executor"):
        out["dX"] = dX
    for k, v in (("dA", dA), ("dB", dB), ("dl", dl)):
        if v:
            out[k] = torch.cat(v)
    return out
