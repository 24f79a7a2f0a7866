"""The work that users of this package have it do, as cases with sizes: one MoE layer from its smallest call to a
large prefill, a stack of resident layers, the attention-derived token score and the two halves of the
error-compensated quantiser.  Every case goes through the package's public entry points.

listed() names the cases; draw() gives further ones from the ranges they stand for; prepare() makes what a program
holds before the call (inputs from the seed, weights in the formats the call reads, buffers); run() makes the call;
exact() is the same result in 64 bits with plain torch; work() counts what the call cannot do without.
"""
import math

import torch

from paper_2603_19172_amd import binding as B
from paper_2603_19172_amd.layer import ExpertStore, MoELayer
from paper_2603_19172_amd.stack import HostExpertPool, ResidentDecodeStack

GROUP = 64
WEIGHT_STD = 0.02
BYTES_PER_WEIGHT = {16: 2.0, 8: 1.0 + 4.0 / GROUP, 4: 0.5 + 4.0 / GROUP, 2: 0.25 + 4.0 / GROUP, 0: 0.0}


def _layer(name, T, H, F, E, k, phase, tiers, quantize, zipf=0.0, out="bf16"):
    return {"name": name, "kind": "layer", "T": T, "H": H, "F": F, "E": E, "k": k, "phase": phase, "tiers": tiers,
            "quantize": quantize, "zipf": zipf, "out": out}


def listed():
    return [
        # the tiny layer every parity test starts from: a chain of launches and latencies, nothing else
        _layer("layer_tiny_16", 16, 256, 512, 8, 2, "prefill", "16/4/2", True, out="f32"),
        # the package's flagship: one decode token on a Mixtral-8x7B-shaped layer, the whole hot path, with the
        # experts that the token selects quantised on first use
        _layer("decode_mixtral_1", 1, 4096, 14336, 8, 2, "decode", "16/4/2", True),
        # the same layer serving a batch of 24 sequences, every format resident: each expert meets a few tokens
        _layer("decode_mixtral_24", 24, 4096, 14336, 8, 2, "decode", "16/4/2", False),
        # one decode token on the fine-grained layer (128 experts of 768, top-8), formats resident
        _layer("decode_fine_1", 1, 2048, 768, 128, 8, "decode", "16/4/2", False),
        # the fine-grained layer serving an odd batch in the paper's own "4/2" mode, fp32 output
        _layer("decode_fine_61", 61, 2048, 768, 128, 8, "decode", "4/2", False, out="f32"),
        # prefill of 512 tokens on the Mixtral-shaped layer, formats resident
        _layer("prefill_mixtral_512", 512, 4096, 14336, 8, 2, "prefill", "16/4/2", False),
        # a long, ragged prefill with an 8-bit top tier and fp32 output
        _layer("prefill_mixtral_1357", 1357, 4096, 14336, 8, 2, "prefill", "8/4/2", False, out="f32"),
        # the fine-grained layer's prefill, whole hot path, Zipf-skewed expert load
        _layer("prefill_fine_2048", 2048, 2048, 768, 128, 8, "prefill", "16/4/2", True, zipf=1.2),
        # the token score taken from attention: a prompt of 4096 tokens, grouped-query heads
        {"name": "attention_4096", "kind": "attention", "T": 4096, "heads": 32, "kv_heads": 8, "d": 128, "causal": True},
        # preparing experts off line: Hessian of 2048 calibration tokens and its factor ...
        {"name": "gptq_factor_4096", "kind": "factor", "n": 2048, "K": 4096},
        # ... and the compensated sweep over one of the matrices that share it
        {"name": "gptq_sweep_mixtral", "kind": "sweep", "N": 14336, "K": 4096, "bits": 4},
        # eight Mixtral-shaped layers with all experts resident, one token through all of them, "4/2" mode with the
        # cosine depth schedule
        {"name": "stack_mixtral_8", "kind": "stack", "L": 8, "H": 4096, "F": 14336, "E": 8, "k": 2},
    ]


def _log_int(rng, lo, hi, step=1):
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return max(step, int(round(v / step)) * step)


def draw(rng):
    most = max(_cost(c) for c in listed())
    while True:
        u = rng.random()
        if u < 0.64:
            H, F = _log_int(rng, 256, 4096, 128), _log_int(rng, 256, 14336, 128)
            E = rng.choice([4, 8, 8, 16, 30, 60, 64, 128])
            k = min(E, rng.choice([1, 2, 2, 4, 6, 8]))
            T = _log_int(rng, 1, 2500)
            if H * F * E > 4096 * 14336 * 8:
                continue
            phase = rng.choice(["decode", "decode", "prefill"]) if T <= 128 else "prefill"
            case = _layer("", T, H, F, E, k, phase, rng.choice(["16/4/2", "16/4/2", "8/4/2", "4/2"]),
                          rng.random() < 0.4, zipf=rng.choice([0.0, 0.0, 1.2]) if E >= 30 else 0.0,
                          out=rng.choice(["bf16", "f32"]))
        elif u < 0.75:
            kv = rng.choice([4, 8])
            case = {"kind": "attention", "T": _log_int(rng, 33, 6000), "heads": kv * rng.choice([1, 4, 4]), "kv_heads": kv,
                    "d": rng.choice([64, 128, 128]), "causal": rng.random() < 0.7}
        elif u < 0.83:
            case = {"kind": "factor", "n": _log_int(rng, 130, 4096), "K": _log_int(rng, 256, 4096, 64)}
        elif u < 0.92:
            case = {"kind": "sweep", "N": _log_int(rng, 200, 14336), "K": _log_int(rng, 256, 4096, 64),
                    "bits": rng.choice([2, 4, 4, 8])}
        else:
            case = {"kind": "stack", "L": rng.randint(2, 8), "H": _log_int(rng, 512, 4096, 128),
                    "F": _log_int(rng, 768, 14336, 128), "E": rng.choice([8, 16]), "k": 2}
            if case["H"] * case["F"] * case["E"] > 4096 * 14336 * 8:
                continue
        case.pop("name", None)
        if _cost(case) <= most:
            return case


def _cost(case):
    w = work(case)
    # the fp32 contractions of the compensated quantiser run on the vector units
    return max(w["bytes"] / 5e12, w["flops"] / (5e13 if case["kind"] in ("factor", "sweep") else 9e14))


# ---------------------------------------------------------------------------------------------------------- inputs

def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _randn(g, *shape, std=1.0):
    """bf16 normals, one leading slice at a time so that the fp32 draw stays small."""
    out = torch.empty(shape, dtype=torch.bfloat16, device="cuda")
    rows = out.view(-1, shape[-1])
    step = max(1, (1 << 26) // shape[-1])
    for r in range(0, rows.shape[0], step):
        n = min(step, rows.shape[0] - r)
        rows[r:r + n] = torch.randn((n, shape[-1]), generator=g, device="cuda") * std
    return out


def _tiers(case):
    """(experts per tier, bits per tier): 10 % / 30 % / 60 % for three tiers, three quarters critical for "4/2"."""
    bits = [int(b) for b in case["tiers"].split("/")]
    E = case["E"]
    if len(bits) == 2:
        top = math.ceil(0.75 * E)
        return [top, E - top], bits
    a = max(1, math.ceil(0.1 * E))
    b = min(E, max(a, math.ceil(0.4 * E)))
    return [a, b - a, E - b], bits


def _k_hh(case):
    return max(1, round(0.05 * case["T"]))


def _layer_inputs(case, seed):
    """x, router, router bias and the experts' bf16 matrices W1 [E,F,H], W3 [E,F,H], W2 [E,H,F].  A prefill has heavy
    hitters (5 % of the tokens, eight times as loud)."""
    g = _gen(seed)
    T, H, F, E = case["T"], case["H"], case["F"], case["E"]
    x = _randn(g, T, H)
    if case["phase"] == "prefill":
        heavy = torch.randperm(T, generator=g, device="cuda")[:_k_hh(case)]
        x[heavy] *= 8
    wg = _randn(g, E, H, std=WEIGHT_STD)
    bias = None
    if case["zipf"]:
        rank = torch.randperm(E, generator=g, device="cuda") + 1
        bias = (-case["zipf"] * torch.log(rank.double())).float()
    w = [_randn(g, E, F, H, std=WEIGHT_STD), _randn(g, E, F, H, std=WEIGHT_STD), _randn(g, E, H, F, std=WEIGHT_STD)]
    return x, wg, bias, w


def _attention_inputs(case, seed):
    """Queries that share a direction per head and keys of which 5 % carry it: those tokens receive more attention."""
    g = _gen(seed)
    T, nh, nkv, d = case["T"], case["heads"], case["kv_heads"], case["d"]
    q = torch.randn((T, nh, d), generator=g, device="cuda")
    k = torch.randn((T, nkv, d), generator=g, device="cuda")
    u = torch.randn((nkv, d), generator=g, device="cuda")
    u *= 0.5 * math.sqrt(d) / u.norm(dim=1, keepdim=True)
    q += u.repeat_interleave(nh // nkv, dim=0)
    k[torch.randperm(T, generator=g, device="cuda")[:max(1, T // 20)]] += u
    return q.bfloat16(), k.bfloat16()


def _calibration(n, K, g):
    """Correlated channels of uneven loudness, as the activations of trained models are."""
    x = torch.randn((n, K), generator=g, device="cuda")
    x += 1.5 * (torch.randn((n, 4), generator=g, device="cuda") @ torch.randn((4, K), generator=g, device="cuda"))
    return (x * torch.exp2(2 * torch.rand((1, K), generator=g, device="cuda") - 1)).bfloat16()


def _factor64(hess, damp=0.01):
    """U upper triangular with (H + damp mean(diag H) I)^-1 = U^T U, in 64 bits."""
    K = hess.shape[0]
    a = hess.double().clone()
    dg = a.diagonal()
    dg[dg == 0] = 1.0
    dg += damp * dg.mean()
    low = torch.linalg.cholesky(a.flip(0, 1))
    return torch.linalg.solve_triangular(low, torch.eye(K, dtype=torch.float64, device="cuda"), upper=False).flip(0, 1)


def _sweep_inputs(case, seed):
    g = _gen(seed)
    w = _randn(g, case["N"], case["K"], std=WEIGHT_STD)
    x = _calibration(2 * case["K"], case["K"], g).double()
    return w, _factor64(x.T @ x).float().contiguous()


def _stack_inputs(case, seed):
    """A token, a router per layer, and a pool of E distinct experts that the layers' experts are drawn from."""
    g = _gen(seed)
    H, F, E = case["H"], case["F"], case["E"]
    h0 = _randn(g, 1, H)
    routers = [_randn(g, E, H, std=WEIGHT_STD) for _ in range(case["L"])]
    return h0, routers, [_randn(g, E, F, H, std=WEIGHT_STD), _randn(g, E, F, H, std=WEIGHT_STD),
                         _randn(g, E, H, F, std=WEIGHT_STD)]


def _stack_tiers(case):
    t = [B.depth_schedule(l, case["L"], 0.5, case["E"]) for l in range(case["L"])]
    return [(v, case["E"] - v) for v in t], (4, 2)


STACK_ALPHA = 0.125
_ctx = []


def _context():
    if not _ctx:
        _ctx.append(B.Context(0))
    return _ctx[0]


# --------------------------------------------------------------------------------------------------------- the calls

def prepare(case, seed):
    ctx = _context()
    st = {"case": case, "ctx": ctx}
    if case["kind"] == "layer":
        T, H, F, E, k = (case[n] for n in ("T", "H", "F", "E", "k"))
        counts, bits = _tiers(case)
        x, wg, bias, w = _layer_inputs(case, seed)
        layer = MoELayer(ctx, T, H, F, E, k, case["phase"], counts, bits, k_hh=_k_hh(case),
                         out_dtype=B.OUT_F32 if case["out"] == "f32" else B.OUT_BF16)
        tiled = layer.layout == B.LAYOUT_TILE
        formats = [b for b in bits if b not in (0, 16)]
        store = ExpertStore([[m[e] for m in w] for e in range(E)], H, F, "cuda:0", formats=formats,
                            ctx=ctx if tiled and 16 in bits else None)
        if not case["quantize"]:
            for b in formats:
                ctx.quantize_experts(store.table, torch.full((E,), b, dtype=torch.uint8, device="cuda"), None, E, H, F,
                                     layout=layer.layout)
        st.update(x=x, wg=wg, bias=bias, layer=layer, store=store)
    elif case["kind"] == "attention":
        q, k = _attention_inputs(case, seed)
        n = int(B.lib.dymoe_attention_workspace_bytes(case["T"], case["heads"]))
        st.update(q=q, k=k, out=torch.empty((case["T"],), dtype=torch.float32, device="cuda"),
                  ws=torch.empty((max(n, 256),), dtype=torch.uint8, device="cuda"))
    elif case["kind"] == "factor":
        K = case["K"]
        st.update(x=_calibration(case["n"], K, _gen(seed)), hess=torch.empty((K, K), dtype=torch.float32, device="cuda"),
                  u=torch.empty((K, K), dtype=torch.float32, device="cuda"),
                  ws=torch.empty((int(B.lib.dymoe_gptq_factor_workspace_bytes(K)),), dtype=torch.uint8, device="cuda"))
    elif case["kind"] == "sweep":
        N, K, b = case["N"], case["K"], case["bits"]
        w, u = _sweep_inputs(case, seed)
        st.update(w=w, u=u, out=(torch.empty((N, K * b // 8), dtype=torch.uint8, device="cuda"),
                                 torch.empty((N, K // GROUP), dtype=torch.float16, device="cuda"),
                                 torch.empty((N, K // GROUP), dtype=torch.float16, device="cuda")),
                  ws=torch.empty((int(B.lib.dymoe_gptq_workspace_bytes(N, K)),), dtype=torch.uint8, device="cuda"))
    else:
        H, F, E = case["H"], case["F"], case["E"]
        h0, routers, w = _stack_inputs(case, seed)
        pool = HostExpertPool(H, F, E, E, lambda i: [m[i].view(torch.int16).cpu().numpy().view("uint16") for m in w])
        pool.add_quantised(ctx, "cuda:0", formats=(4, 2))
        counts, bits = _stack_tiers(case)
        st.update(h0=h0, stack=ResidentDecodeStack(ctx, H, F, E, case["k"], routers, pool, counts, bits,
                                                   alpha=STACK_ALPHA, graph=False))
    return st


def run(state):
    case, ctx = state["case"], state["ctx"]
    if case["kind"] == "layer":
        ly = state["layer"]
        y = ly.step(state["x"], state["wg"], state["bias"], state["store"], quantize=case["quantize"])
        return {"y": y, "idx": ly.idx, "gate": ly.gate, "bits": ly.bits, "load": ly.load}
    if case["kind"] == "attention":
        return {"score": ctx.token_score_attention(state["q"], state["k"], causal=case["causal"], out=state["out"],
                                                   workspace=state["ws"])}
    if case["kind"] == "factor":
        hess = ctx.gptq_hessian(state["x"], out=state["hess"])
        return {"hess": hess, "u": ctx.gptq_factor(hess, out=state["u"], workspace=state["ws"])}
    if case["kind"] == "sweep":
        codes, scale, zero = ctx.gptq_quantize_pack(state["w"], state["u"], case["bits"], out=state["out"],
                                                    workspace=state["ws"])
        return {"codes": codes, "scale": scale, "zero": zero}
    s = state["stack"]
    return {"h": s.step(state["h0"]), "idx": s.idx, "gate": s.gate, "bits": s.bits}


# ------------------------------------------------------------------------------------------------- accounts and limits

def _routed(T, k, E, counts, bits):
    """Expected number of distinct experts T tokens reach when routing is even, and the widths of that many experts
    from the top of the ranking down (who is asked for ranks high)."""
    active = E * (1.0 - (1.0 - k / E) ** T)
    widths = [b for c, b in zip(counts, bits) for b in [b] * c]
    whole = int(active)
    return [(b, 1.0) for b in widths[:whole]] + ([(widths[whole], active - whole)] if whole < E else [])


def work(case):
    kind = case["kind"]
    if kind == "layer":
        T, H, F, E, k = (case[n] for n in ("T", "H", "F", "E", "k"))
        counts, bits = _tiers(case)
        per = 3.0 * H * F
        total = (T + E) * H * 2.0 + T * H * (4.0 if case["out"] == "f32" else 2.0)
        for b, share in _routed(T, k, E, counts, bits):
            # quantising on first use reads the bf16 source and writes the codes
            read = 2.0 + BYTES_PER_WEIGHT[b] if case["quantize"] and b != 16 else BYTES_PER_WEIGHT[b]
            total += share * per * read
        return {"bytes": total, "flops": 6.0 * T * k * H * F + 2.0 * T * H * E}
    if kind == "attention":
        T, nh, nkv, d = case["T"], case["heads"], case["kv_heads"], case["d"]
        # the logits once: every probability needs its row's sum, which a second pass over the logits may use
        return {"bytes": 2.0 * T * (nh + nkv) * d + 4.0 * T, "flops": 2.0 * nh * T * T * d * (0.5 if case["causal"] else 1.0)}
    if kind == "factor":
        n, K = case["n"], case["K"]
        return {"bytes": 2.0 * n * K + 8.0 * K * K, "flops": 1.0 * n * K * K + 2.0 * K ** 3 / 3.0}
    if kind == "sweep":
        N, K, b = case["N"], case["K"], case["bits"]
        return {"bytes": N * K * (2.0 + BYTES_PER_WEIGHT[b]) + 2.0 * K * K, "flops": 1.0 * N * K * K}
    L, H, F, E, k = (case[n] for n in ("L", "H", "F", "E", "k"))
    counts, bits = _stack_tiers(case)
    total = 0.0
    for c in counts:
        total += E * H * 2.0 + sum(s * BYTES_PER_WEIGHT[b] * 3.0 * H * F for b, s in _routed(1, k, E, c, bits))
    return {"bytes": total, "flops": L * (6.0 * k * H * F + 2.0 * H * E)}


def tolerance(case):
    # Each bound is about four times the error against exact() that was measured over the listed and drawn cases.
    kind = case["kind"]
    if kind == "layer":
        # 16-bit intermediate and weights of 11 bits on the way to the matrix cores, bf16 rounding of y; whole
        # numbers only where two logits or two experts' importances are a rounding apart
        return {"rel": 8e-3, "max": 0.1, "differ": 2e-3}                # measured 3.4e-4 (fp32 out) to 1.9e-3 (bf16)
    if kind == "attention":
        return {"rel": 8e-7}                                            # measured 1.8e-7
    if kind == "factor":
        # fp32 Cholesky of a matrix whose condition number is about a thousand: measured 1e-5 to 2.5e-4
        return {"rel": 1e-3}
    if kind == "sweep":
        return "exact"      # the codes are defined by an exact sequence of binary32 operations
    # a bf16 rounding of the hidden state in every layer travels through those behind it: measured 4.1e-3
    return {"rel": 1.6e-2, "max": 0.2, "differ": 2e-3}


# ------------------------------------------------------------------------------------------------------ 64-bit results

def _dequantised(w, bits):
    """The plain quantiser's definition (binary32, one rounding per step) and the values its codes stand for, fp64."""
    if bits == 16:
        return w.double()
    v = w.float().view(*w.shape[:-1], w.shape[-1] // GROUP, GROUP)
    lo, hi = v.amin(-1, keepdim=True), v.amax(-1, keepdim=True)
    top = float(2 ** bits - 1)
    zero, scale = lo.half().float(), ((hi - lo) / top).half().float()
    inv = torch.where(scale > 0, 1.0 / scale, torch.zeros_like(scale))
    q = torch.clamp(torch.round((v - zero) * inv), 0.0, top)
    return (q.double() * scale.double() + zero.double()).view(w.shape)


def _route64(x, wg, bias, k):
    logit = x.double() @ wg.double().T
    if bias is not None:
        logit = logit + bias.double()
    probs = torch.softmax(logit, dim=1)
    idx = torch.sort(logit, dim=1, descending=True, stable=True).indices[:, :k]
    gate = probs.gather(1, idx)
    return probs, idx, gate / gate.sum(1, keepdim=True)


def _assign(importance, load, counts, bits):
    imp, ld = importance.tolist(), load.tolist()
    order = sorted(range(len(imp)), key=lambda e: (-imp[e], -ld[e], e))
    widths = [b for c, b in zip(counts, bits) for b in [b] * c]
    out = [0] * len(imp)
    for pos, e in enumerate(order):
        out[e] = widths[pos]
    return out


def _ffn64(x, idx, gate, widths, w_of):
    y = torch.zeros((x.shape[0], x.shape[1]), dtype=torch.float64, device="cuda")
    for e, b in enumerate(widths):
        if b == 0:
            continue
        tok, slot = torch.where(idx == e)
        if tok.numel() == 0:
            continue
        xe = x[tok].double()
        a = xe @ _dequantised(w_of(e, 0), b).T
        a = a * torch.sigmoid(a) * (xe @ _dequantised(w_of(e, 1), b).T)
        y.index_add_(0, tok, gate[tok, slot].unsqueeze(1) * (a @ _dequantised(w_of(e, 2), b).T))
    return y


def _layer64(case, seed):
    T, E, k = case["T"], case["E"], case["k"]
    x, wg, bias, w = _layer_inputs(case, seed)
    counts, bits = _tiers(case)
    probs, idx, gate = _route64(x, wg, bias, k)
    load = torch.bincount(idx.reshape(-1), minlength=E)
    if case["phase"] == "prefill":
        heavy = torch.sort(x.double().norm(dim=1), descending=True, stable=True).indices[:_k_hh(case)]
        imp = torch.bincount(idx[heavy].reshape(-1), minlength=E)
    else:
        imp = probs.mean(0)
    widths = _assign(imp, load, counts, bits)
    y = _ffn64(x, idx, gate, widths, lambda e, m: w[m][e])
    return {"y": y, "idx": idx.int(), "gate": gate, "bits": torch.tensor(widths, dtype=torch.uint8), "load": load.int()}


def _attention64(case, seed):
    q, k = _attention_inputs(case, seed)
    T, nh, nkv, d = case["T"], case["heads"], case["kv_heads"], case["d"]
    score = torch.zeros((T,), dtype=torch.float64, device="cuda")
    keep = torch.ones((T, T), dtype=torch.bool, device="cuda").tril() if case["causal"] else None
    for h in range(nh):
        logit = q[:, h].double() @ k[:, h // (nh // nkv)].double().T.contiguous() / math.sqrt(d)
        if keep is not None:
            logit = logit.masked_fill(~keep, -math.inf)
        score += torch.softmax(logit, dim=1).sum(0)
    return {"score": score / (nh * T)}


def _sweep64(case, seed):
    """Scale and zero of every group from the compensated values; the codes follow binary32 roundings and have no
    64-bit counterpart."""
    w, u = _sweep_inputs(case, seed)
    u, v = u.double(), w.double()
    N, K, top = case["N"], case["K"], float(2 ** case["bits"] - 1)
    scale = torch.empty((N, K // GROUP), dtype=torch.float64, device="cuda")
    zero = torch.empty_like(scale)
    for g in range(K // GROUP):
        a, b = GROUP * g, GROUP * (g + 1)
        blk, err = v[:, a:b].clone(), torch.empty((N, GROUP), dtype=torch.float64, device="cuda")
        lo, hi = blk.amin(1), blk.amax(1)
        m, s = lo.half().double(), ((hi - lo) / top).half().double()
        inv = torch.where(s > 0, 1.0 / s, torch.zeros_like(s))
        scale[:, g], zero[:, g] = s, m
        for c in range(GROUP):
            dq = torch.clamp(torch.round((blk[:, c] - m) * inv), 0.0, top) * s + m
            err[:, c] = (blk[:, c] - dq) / u[a + c, a + c]
            if c + 1 < GROUP:
                blk[:, c + 1:] -= err[:, c:c + 1] * u[a + c, a + c + 1:b]
        if b < K:
            v[:, b:] -= err @ u[a:b, b:]
    return {"codes": None, "scale": scale, "zero": zero}


def _stack64(case, seed):
    h, routers, w = _stack_inputs(case, seed)
    L, E = case["L"], case["E"]
    counts, bits = _stack_tiers(case)
    out = {"idx": [], "gate": [], "bits": []}
    for l in range(L):
        probs, idx, gate = _route64(h, routers[l], None, case["k"])
        load = torch.bincount(idx.reshape(-1), minlength=E)
        widths = _assign(probs[0], load, counts[l], bits)
        y = _ffn64(h, idx, gate, widths, lambda e, m: w[m][(l * E + e) % E])
        v = h.double() + STACK_ALPHA * y
        h = (v / v.square().mean(1, keepdim=True).sqrt()).bfloat16()      # a layer hands on bf16
        out["idx"].append(idx.int())
        out["gate"].append(gate)
        out["bits"].append(torch.tensor(widths, dtype=torch.uint8))
    return {"h": h.double(), "idx": torch.stack(out["idx"]), "gate": torch.stack(out["gate"]), "bits": torch.stack(out["bits"])}


def exact(case, seed):
    kind = case["kind"]
    if kind == "layer":
        return _layer64(case, seed)
    if kind == "attention":
        return _attention64(case, seed)
    if kind == "factor":
        x = _calibration(case["n"], case["K"], _gen(seed)).double()
        hess = x.T @ x
        return {"hess": hess, "u": _factor64(hess.float())}
    if kind == "sweep":
        return _sweep64(case, seed)
    return _stack64(case, seed)
