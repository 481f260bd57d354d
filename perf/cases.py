"""The work a Gated DeltaNet layer's serving loop has this library do, as a list of measurable cases.

Four kinds of pass (`op`), each through the entry points of paper_2605_19049_amd.kvb:

  decode  `steps` tokens for each of B requests, one kvb_decode_flush call a token.  Requests stand at
          independent buffer fills, as under continuous batching, so in each step about one request in C
          folds its buffer into the state.
  spec    one round of speculative decoding: kvb_verify of T drafts (or kvb_verify_tree and kvb_compact
          where the drafts form a tree), then kvb_flush of what was accepted.
  prefill kvb_direct over ragged contexts of 1 .. Lmax tokens; with `fold` a kvb_flush into the state
          after it, the way a context enters the chunkwise regime.
  kvonly  kvb_direct, then `steps` kvb_decode calls without a state: a short context that lives in its
          buffer alone.

Every pass can be repeated on the same store: decode and spec leave fills within the buffer, prefill and
kvonly start by overwriting the fill.  Inputs are synthetic with the distributions of
paper_2605_19049_amd/synth.py (unit keys and queries, normal values, log decays in -0.5 .. 0, sigmoid
betas), drawn on the GPU from the seed.
"""
import math

import torch

from paper_2605_19049_amd import kvb, traffic

_CODE = {"f32": kvb.F32, "bf16": kvb.BF16, "f16": kvb.F16}
_SPARE = 4   # a serving store has more slots than a batch has requests: one in four here


def _case(op, B, Hk, Hv, d, C, cap, in_dtype, rec_dtype, **more):
    c = dict(op=op, B=B, Hk=Hk, Hv=Hv, d=d, C=C, cap=cap, in_dtype=in_dtype, rec_dtype=rec_dtype, block=0, steps=0, T=0, tree=False,
             Lmax=0, fold=False, graph=False)
    c.update(more)
    return c


def listed():
    cases = [
        # One user, one request: the latency of a token is a chain of tiny launches, replayed from a graph as
        # a decoding loop does at this size.
        dict(_case("decode", 1, 16, 32, 128, 16, 16, "bf16", "f32", steps=16, graph=True), name="decode_single"),
        # A small batch on one of four tensor-parallel ranks (4 of 16 key heads, 8 of 32 value heads), in the
        # all-16-bit storage regime, odd batch size.
        dict(_case("decode", 13, 4, 8, 128, 32, 32, "f16", "f16", steps=16, graph=True), name="decode_tp4_shard"),
        # The Qwen3-Next layer at an ordinary serving batch.
        dict(_case("decode", 64, 16, 32, 128, 16, 16, "bf16", "f32", steps=16), name="decode_batch64"),
        # The largest batch: 1 GB of state that no cache holds, long buffers in paged 16-record blocks.
        dict(_case("decode", 500, 16, 32, 128, 64, 64, "bf16", "f32", steps=4, block=16), name="decode_batch500_paged"),
        # Speculative decoding with a draft head, an ordinary batch: 4 drafts, chunks of 16.
        dict(_case("spec", 128, 16, 32, 128, 16, 20, "bf16", "f32", T=4), name="spec_batch128"),
        # Tree drafts for a few interactive users, 16-bit records, long buffers.
        dict(_case("spec", 7, 16, 32, 128, 64, 72, "f16", "f16", T=8, tree=True, graph=True), name="spec_tree_few"),
        # Prefill of a burst of short prompts.
        dict(_case("prefill", 256, 16, 32, 128, 64, 64, "bf16", "f32", Lmax=64), name="prefill_burst64"),
        # Prefill of a single short prompt: time to first token.
        dict(_case("prefill", 2, 16, 32, 128, 64, 64, "bf16", "f32", Lmax=50), name="prefill_pair"),
        # Prompts up to the head size, folded into states at once.
        dict(_case("prefill", 96, 16, 32, 128, 128, 128, "bf16", "f32", Lmax=128, fold=True), name="prefill_fold128"),
        # Short conversations served without a state, 16-bit regime: prompt, then 16 tokens from the buffer alone.
        dict(_case("kvonly", 128, 16, 32, 128, 128, 128, "f16", "f16", Lmax=100, steps=16), name="kvonly_chat"),
        # A model with smaller heads (64): prefill and fold.
        dict(_case("prefill", 48, 8, 16, 64, 64, 64, "bf16", "f32", Lmax=64, fold=True), name="prefill_fold_d64"),
        # Full-precision evaluation (fp32 vectors) with drafts.
        dict(_case("spec", 24, 16, 16, 128, 16, 24, "f32", "f32", T=5), name="spec_fp32"),
    ]
    return cases


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges, no larger than the largest listed one."""
    op = rng.choice(["decode", "decode", "spec", "spec", "prefill", "kvonly"])
    in_dtype, rec_dtype = rng.choice([("bf16", "f32")] * 4 + [("f16", "f16")] * 3 + [("f16", "f32"), ("bf16", "bf16"), ("f32", "f32")])
    d = rng.choice([128] * 7 + [64, 64, 32])
    Hk, Hv = rng.choice([(16, 32), (16, 32), (8, 16), (4, 8), (2, 4), (16, 16), (3, 9)])
    B = _log_int(rng, 1, 500)
    wide = d == 128 and in_dtype != "f32"
    block = rng.choice([0, 0, 0, 8, 16])
    if op == "decode":
        C = rng.choice([8, 16, 24, 32, 64, 128])
        c = _case(op, B, Hk, Hv, d, C, C, in_dtype, rec_dtype, block=block, steps=rng.choice([4, 8, 16]))
    elif op == "spec":
        C, T = rng.choice([8, 16, 32, 64, 96]), rng.randint(2, 8)
        cap = C - 1 + T + rng.randint(0, 3)
        c = _case(op, B, Hk, Hv, d, C, cap, in_dtype, rec_dtype, block=block, T=T, tree=rng.random() < 0.3 and B <= 64)
    else:
        Lmax = _log_int(rng, 8, 112 if wide else 64)
        steps = rng.choice([4, 8, 16]) if op == "kvonly" else 0
        fold = op == "prefill" and rng.random() < 0.5
        c = _case(op, B, Hk, Hv, d, Lmax + steps, Lmax + steps, in_dtype, rec_dtype, block=block, Lmax=Lmax, steps=steps, fold=fold)
    if c["block"]:   # whole blocks
        c["cap"] = min(128, -(-c["cap"] // c["block"]) * c["block"])
    most = max(work(x)["bytes"] for x in listed())
    while c["B"] > 1 and work(c)["bytes"] > most:
        c["B"] = (c["B"] + 1) // 2
    # launches outweigh the kernels at the smallest sizes, where a serving loop replays a graph
    c["graph"] = work(c)["bytes"] < 4e7 * max(1, c["steps"]) and (op != "prefill" or c["fold"])   # (one launch needs none)
    return c


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _tokens(gen, lead, c):
    """Tokens with leading sizes `lead`, rounded to the case's input type."""
    dt, dev = kvb.torch_dtype(_CODE[c["in_dtype"]]), "cuda"
    Hk, Hv, d = c["Hk"], c["Hv"], c["d"]

    def unit(*size):
        x = torch.randn(size, generator=gen, device=dev)
        return (x / x.norm(dim=-1, keepdim=True)).to(dt)

    return {"q": unit(*lead, Hk, d), "k": unit(*lead, Hk, d), "v": torch.randn(*lead, Hv, d, generator=gen, device=dev).to(dt),
            "g": -0.5 * torch.rand(*lead, Hv, generator=gen, device=dev),
            "beta": torch.sigmoid(torch.randn(*lead, Hv, generator=gen, device=dev))}


def _ints(gen, lo, hi, *size):
    return torch.randint(lo, hi + 1, size, generator=gen, device="cuda", dtype=torch.int32)


def _inputs(c, seed):
    """Everything a pass reads, as plain tensors; records as [n_slots, heads, cap, d] whatever the layout."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    B, Hk, Hv, d, cap, T = c["B"], c["Hk"], c["Hv"], c["d"], c["cap"], c["T"]
    n = B + B // _SPARE + 1
    x = {"n": n, "slot": torch.randperm(n, generator=gen, device="cuda")[:B].to(torch.int32)}
    if c["op"] in ("decode", "spec"):
        rec = _tokens(gen, (n, cap), c)   # the chunk so far: keys, delta values, cumulative decays
        x["rec_k"] = rec["k"].transpose(1, 2).contiguous()
        x["rec_u"] = (0.6 * rec["v"].float()).to(kvb.torch_dtype(_CODE[c["rec_dtype"]])).transpose(1, 2).contiguous()
        x["rec_G"] = rec["g"].cumsum(1).transpose(1, 2).contiguous()
        x["fill"] = _ints(gen, 0, c["C"] - 1, n)
    else:
        x["rec_k"] = torch.zeros((n, Hk, cap, d), dtype=kvb.torch_dtype(_CODE[c["in_dtype"]]), device="cuda")
        x["rec_u"] = torch.zeros((n, Hv, cap, d), dtype=kvb.torch_dtype(_CODE[c["rec_dtype"]]), device="cuda")
        x["rec_G"] = torch.zeros((n, Hv, cap), device="cuda")
        x["fill"] = torch.zeros(n, dtype=torch.int32, device="cuda")
    x["state"] = None
    if c["op"] in ("decode", "spec"):
        x["state"] = 0.5 * torch.randn(n, Hv, d, d, generator=gen, device="cuda")
    elif c["fold"]:   # a context that enters the chunkwise regime folds into a fresh state
        x["state"] = torch.zeros((n, Hv, d, d), device="cuda")
    if c["op"] == "decode":
        x["tok"] = _tokens(gen, (c["steps"], B), c)
    elif c["op"] == "spec":
        x["tok"] = _tokens(gen, (B, T), c)
        x["accepted"] = _ints(gen, 0, T, B)
        if c["tree"]:
            u = torch.rand(B, T, generator=gen, device="cuda")
            i = torch.arange(T, device="cuda")
            x["parent"] = (torch.floor(u * (i + 1)) - 1).clamp(max=i - 1).to(torch.int32)   # uniform over -1 .. i-1
            # the accepted root path: the ancestors of a random node (none for "accepted" 0)
            par, leaf = x["parent"].tolist(), (x["accepted"] - 1).tolist()
            path, plen = [], []
            for b in range(B):
                nodes, v = [], leaf[b]
                while v >= 0:
                    nodes.append(v)
                    v = par[b][v]
                nodes.reverse()
                path.append(nodes + [0] * (T - len(nodes)))
                plen.append(len(nodes))
            x["leaf"] = x["accepted"] - 1
            x["path"] = torch.tensor(path, dtype=torch.int32, device="cuda")
            x["accepted"] = torch.tensor(plen, dtype=torch.int32, device="cuda")
    else:
        x["ctx"] = _tokens(gen, (B, c["Lmax"]), c)
        x["len"] = _ints(gen, 1, c["Lmax"], B)
        if c["steps"]:
            x["tok"] = _tokens(gen, (c["steps"], B), c)
    if c["block"]:
        mb = cap // c["block"]
        blocks = n * mb + 3   # a pool that other requests use too
        x["table"] = torch.randperm(blocks, generator=gen, device="cuda")[:n * mb].reshape(n, mb).to(torch.int32)
        x["blocks"] = blocks
    return x


def _to_pool(c, x, dense):
    """[n_slots, heads, cap, ...] records in the store's layout: as they are, or dealt over the block pool."""
    if not c["block"]:
        return dense
    n, h, mb, bs = dense.shape[0], dense.shape[1], c["cap"] // c["block"], c["block"]
    tail = dense.shape[3:]
    pool = torch.zeros((x["blocks"], h, bs) + tail, dtype=dense.dtype, device=dense.device)
    by_block = dense.reshape((n, h, mb, bs) + tail).transpose(1, 2)
    pool[x["table"].long()] = by_block
    return pool


def prepare(case, seed):
    c, x = case, _inputs(case, seed)
    code, rec = _CODE[c["in_dtype"]], _CODE[c["rec_dtype"]]
    out_dtype = rec if rec != kvb.F32 else kvb.F32   # the 16-bit regime returns 16-bit outputs
    ds = kvb.DeviceStore(x["n"], c["Hk"], c["Hv"], c["d"], c["d"], c["cap"], code, with_state=x["state"] is not None, rec_dtype=rec,
                         **({"block_size": c["block"], "n_blocks": x["blocks"], "block_table": x["table"]} if c["block"] else {}))
    if x["state"] is not None:
        ds.state.copy_(x["state"])
    ds.buf_k.copy_(_to_pool(c, x, x["rec_k"]))
    ds.buf_u.copy_(_to_pool(c, x, x["rec_u"]))
    ds.buf_G.copy_(_to_pool(c, x, x["rec_G"]))
    ds.fill.copy_(x["fill"])
    sh = kvb.shape(c["B"], c["Hk"], c["Hv"], c["d"], c["d"], c["cap"], code, scale=c["d"] ** -0.5, out_dtype=out_dtype, rec_dtype=rec)
    s = {"case": c, "ds": ds, "sh": sh, "st": ds.c(c["op"] != "kvonly"), "slot": x["slot"], "keep": []}
    odt = kvb.torch_dtype(out_dtype)
    for key in ("tok", "ctx", "len", "accepted", "parent", "path"):
        if key in x:
            s[key] = x[key]
    if "tok" in s:
        s["out"] = torch.zeros(s["tok"]["v"].shape, dtype=odt, device="cuda")
    if "ctx" in s:
        s["ctx_out"] = torch.zeros(s["ctx"]["v"].shape, dtype=odt, device="cuda")
        s["st_none"] = ds.c(False)
    if c["op"] in ("decode", "kvonly"):
        t = s["tok"]
        s["step"] = [[t[key][i] for key in ("q", "k", "v", "g", "beta")] + [s["out"][i]] for i in range(c["steps"])]
    elif c["op"] == "spec":
        s["args"] = [s["tok"][key] for key in ("q", "k", "v", "g", "beta")] + [s["out"]]
    if c["op"] in ("prefill", "kvonly"):
        s["ctx_args"] = [s["ctx"][key] for key in ("q", "k", "v", "g", "beta")] + [s["ctx_out"]]
    s["result"] = {"out": s.get("out"), "ctx_out": s.get("ctx_out"), "state": ds.state, "k": ds.buf_k, "u": ds.buf_u, "G": ds.buf_G,
                   "fill": ds.fill, "status": ds.status}
    s["result"] = {key: v for key, v in s["result"].items() if v is not None}
    if c["graph"]:
        s["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(s["graph"]):
            for name, args in _calls(s):
                getattr(kvb, name)(*args)
    else:   # marshalled once, as a serving loop does
        stream = torch.cuda.current_stream().cuda_stream
        s["bound"] = [kvb.bind(name, *args, stream) for name, args in _calls(s)]
    return s


def _calls(s):
    """The entry points of one pass, in order, with their arguments."""
    c, sh, slot = s["case"], s["sh"], s["slot"]
    if c["op"] == "decode":
        return [("kvb_decode_flush", (sh, s["st"], slot, *a, c["C"])) for a in s["step"]]
    if c["op"] == "spec":
        commit = [("kvb_flush", (sh, s["st"], slot, s["accepted"], c["C"]))]
        if c["tree"]:
            return [("kvb_verify_tree", (sh, s["st"], slot, c["T"], s["parent"], *s["args"])),
                    ("kvb_compact", (sh, s["st"], slot, c["T"], s["path"], s["accepted"]))] + commit
        return [("kvb_verify", (sh, s["st"], slot, c["T"], *s["args"]))] + commit
    calls = [("kvb_direct", (sh, s["st_none"], slot, s["len"], c["Lmax"], *s["ctx_args"]))]
    if c["op"] == "kvonly":
        calls += [("kvb_decode", (sh, s["st_none"], slot, *a)) for a in s["step"]]
    elif c["fold"]:
        calls += [("kvb_flush", (sh, s["st"], slot, None, 1))]
    return calls


def run(state):
    if "graph" in state:
        state["graph"].replay()
    else:
        for call in state["bound"]:
            call()
    return state["result"]


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------
def work(case):
    """Every array element the calls have to read or write, once, at the mean fill, length and acceptance of
    the case's distributions; multiply-adds of the chunkwise form (two products with the state a token, two
    with each record, two Gram products, one rank-1 update a record)."""
    c = case
    out = c["rec_dtype"]
    lay = traffic.layout(c["in_dtype"], c["rec_dtype"], out, r=c["Hv"] / c["Hk"], dk=c["d"], dv=c["d"])
    d, units = c["d"], c["B"] * c["Hv"]
    if c["op"] == "decode":
        f = (c["C"] - 1) / 2
        nbytes = c["steps"] * sum(traffic.fused_cycle_rw(lay, c["C"]))
        flops = c["steps"] * (4 * d * d + 8 * f * d + 2 * d * d)
    elif c["op"] == "spec":
        f, T, a = (c["C"] - 1) / 2, c["T"], c["T"] / 2
        folds = a / c["C"]
        m = c["C"] - 1 + (a + 1) / 2
        nbytes = sum(traffic.verify_rw(lay, f, T)) + folds * sum(traffic.flush_rw(lay, m))
        flops = T * (4 * d * d + 8 * (f + T / 2) * d) + folds * 2 * m * d * d
    else:
        L = (c["Lmax"] + 1) / 2
        L2 = (c["Lmax"] + 1) * (2 * c["Lmax"] + 1) / 6   # mean square length
        nbytes = sum(traffic.direct_rw(lay, L))
        flops = 4 * L2 * d
        if c["op"] == "kvonly":
            f = L + (c["steps"] - 1) / 2
            nbytes += c["steps"] * sum(traffic.decode_rw(lay, f, with_state=False))
            flops += c["steps"] * 8 * f * d
        elif c["fold"]:
            nbytes += sum(traffic.flush_rw(lay, L))
            flops += 2 * L * d * d
    return {"bytes": float(units * nbytes), "flops": float(units * flops)}


def tolerance(case):
    """fp32 records: sums of up to a few hundred fp32 products, 1e-7 .. 6e-7 off the 64-bit result, so another
    order of them may be four times that away.  16-bit records and outputs: 1.2e-4 .. 2.9e-4 off with fp16 (half
    a unit of the type, spread over the values), eight times that with bf16; a value that lands on the other
    side of a rounding boundary moves by a whole unit (2^-10 or 2^-7 of itself), and what reads it follows."""
    return {"f32": {"rel": 3e-6, "max": 3e-5}, "f16": {"rel": 1.2e-3, "max": 1e-2}, "bf16": {"rel": 1e-2, "max": 8e-2}}[case["rec_dtype"]]


# ---------------------------------------------------------------------------
# the same in 64 bits: the token-by-token recurrence
# ---------------------------------------------------------------------------
def _expand(t, c):
    """[.., Hk, d] of the key heads for every value head, in fp64."""
    return t.double().repeat_interleave(c["Hv"] // c["Hk"], dim=-2)


def _token(S, t, c, scale):
    """One token: (new state, delta value, output); S [B, Hv, d, d], t holds [B, H, d] / [B, Hv] tensors."""
    q, k, v = _expand(t["q"], c), _expand(t["k"], c), t["v"].double()
    S = S * torch.exp(t["g"].double())[..., None, None]
    u = t["beta"].double()[..., None] * (v - (S * k[..., None]).sum(-2))
    S = S + k[..., None] * u[..., None, :]
    return S, u, scale * (S * q[..., None]).sum(-2)


def _at(tok, *index):
    return {key: v[index] for key, v in tok.items()}


def exact(case, seed):
    c = case
    x = _inputs(c, seed)
    B, Hv, d, scale = c["B"], c["Hv"], c["d"], c["d"] ** -0.5
    slot = x["slot"].long()
    rec = {"k": x["rec_k"].double(), "u": x["rec_u"].double(), "G": x["rec_G"].double()}
    fill = x["fill"].clone()
    state = x["state"].double() if x["state"] is not None else None
    b_all = torch.arange(B, device="cuda")
    f = fill[slot].long()
    res = {}

    def append(at, who, t, u, G):
        """Record `at` (one place per request of `who`)."""
        s = slot[who]
        rec["k"][s, :, at] = t["k"].double()[who]
        rec["u"][s, :, at] = u[who]
        rec["G"][s, :, at] = G[who]

    if c["op"] in ("decode", "spec"):
        # the state that the committed state and the buffered records stand for
        last = (f - 1).clamp(min=0)
        G = torch.where(f[:, None] > 0, rec["G"][slot, :, last], 0.0)
        live = torch.arange(c["cap"], device="cuda")[None, :] < f[:, None]
        w = torch.where(live[:, None, :], torch.exp(G[..., None] - rec["G"][slot]), 0.0)
        S = state[slot] * torch.exp(G)[..., None, None]
        kx = rec["k"][slot].repeat_interleave(Hv // c["Hk"], dim=1)
        S += torch.matmul((kx * w[..., None]).transpose(-1, -2).contiguous(), rec["u"][slot])
        del kx, w
    else:
        S = torch.zeros((B, Hv, d, d), dtype=torch.float64, device="cuda")
        G = torch.zeros((B, Hv), dtype=torch.float64, device="cuda")

    if c["op"] == "spec":
        out = torch.zeros(B, c["T"], Hv, d, dtype=torch.float64, device="cuda")
        # the state and the decay before the first draft and after each one (index i + 1: after draft i)
        Ss, Gs = [S], [G]
        done = {0: (S, G)}
        a = x["accepted"].long()
        leaf = x["leaf"].long() if c["tree"] else a - 1
        final = S.clone()
        for i in range(c["T"]):
            t = _at(x["tok"], slice(None), i)
            if c["tree"]:
                p = x["parent"][:, i].long() + 1
                S0 = torch.stack([Ss[int(p[b])][b] for b in range(B)])
                G0 = torch.stack([Gs[int(p[b])][b] for b in range(B)])
            else:
                S0, G0 = Ss[-1], Gs[-1]
            S1, u, out[:, i] = _token(S0, t, c, scale)
            G1 = G0 + t["g"].double()
            append(f + i, b_all, t, u, G1)
            Ss = Ss + [S1] if c["tree"] else [S1]
            Gs = Gs + [G1] if c["tree"] else [G1]
            final = torch.where((leaf == i)[:, None, None, None], S1, final)
        del done
        if c["tree"]:
            for j in range(c["T"]):
                who = b_all[a > j]
                src = f[who] + x["path"][who, j].long()
                for key in rec:
                    rec[key][slot[who], :, f[who] + j] = rec[key][slot[who], :, src]
        m = f + a
        who = b_all[m >= c["C"]]
        state[slot[who]] = final[who]
        fill[slot] = torch.where(m >= c["C"], 0, m).to(torch.int32)
        res["out"] = out
    elif c["op"] == "decode":
        out = torch.zeros(c["steps"], B, Hv, d, dtype=torch.float64, device="cuda")
        for i in range(c["steps"]):
            t = _at(x["tok"], i)
            S, u, out[i] = _token(S, t, c, scale)
            G = G + t["g"].double()
            append(f, b_all, t, u, G)
            f = f + 1
            who = b_all[f >= c["C"]]
            state[slot[who]] = S[who]
            G[who] = 0.0
            f[who] = 0
        fill[slot] = f.to(torch.int32)
        res["out"] = out
    else:
        L = x["len"].long()
        ctx_out = torch.zeros(B, c["Lmax"], Hv, d, dtype=torch.float64, device="cuda")
        for i in range(c["Lmax"]):
            who = b_all[L > i]
            if who.numel() == 0:
                break
            t = _at(x["ctx"], slice(None), i)
            S1, u, o = _token(S[who], {key: v[who] for key, v in t.items()}, c, scale)
            S[who] = S1
            G[who] += t["g"].double()[who]
            ctx_out[who, i] = o
            s = slot[who]
            rec["k"][s, :, i] = t["k"].double()[who]
            rec["u"][s, :, i] = u
            rec["G"][s, :, i] = G[who]
        res["ctx_out"] = ctx_out
        f = L
        if c["op"] == "kvonly":
            out = torch.zeros(c["steps"], B, Hv, d, dtype=torch.float64, device="cuda")
            for i in range(c["steps"]):
                t = _at(x["tok"], i)
                S, u, out[i] = _token(S, t, c, scale)
                G = G + t["g"].double()
                append(f, b_all, t, u, G)
                f = f + 1
            res["out"] = out
        elif c["fold"]:
            state[slot] = S
            f = torch.zeros_like(f)
        fill[slot] = f.to(torch.int32)
    if state is not None:
        res["state"] = state
    for key in rec:
        res[key] = _to_pool(c, x, rec[key])
    res["fill"] = fill
    res["status"] = torch.zeros_like(fill)
    return res
