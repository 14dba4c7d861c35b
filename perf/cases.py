"""The work that programs on top of this package have it do, as a list of cases to time and compare.

Every case goes through the entry points of the package (`paper_2506_11449_amd`), with buffers, workspace and prepared
operands held by the caller as a training loop or a server holds them.  Sizes are those of the benchmark's workloads
(`synth.WORKLOADS`, the stack step) and of the tests, and draws over the same ranges."""
import torch

import paper_2506_11449_amd as dd
from paper_2506_11449_amd import synth
from paper_2506_11449_amd.stack import StackStep

TEMPERATURE = 0.5


def listed():
    return [
        # The tiny configuration (smoke test, debugging, unit tests of a training loop): re-selection and the three products
        # in fp32, where only latency and the number of launches count.
        _case("step", "tiny_step_f32", 64, 64, 8, 16, "f32"),
        # A server answering for one image (197 tokens): one wide layer on operands prepared when the weights were loaded.
        _case("infer", "one_image_infer", 768, 3072, 307, 197, "bf16"),
        # Inference on a trained mask whose offsets lie in runs (the small-world structure), on the kernels that skip
        # empty blocks; the ViT-Base MLP at 128 images.
        dict(_case("clustered", "clustered_infer", 768, 3072, 307, 128 * 197, "bf16"), runs=5),
        # Training step of a ViT-Base attention projection at 64 images, diagonals re-selected each step.
        _case("step", "attn_step", 768, 768, 77, 64 * 197, "bf16"),
        # Training step of the widest configured layer: ViT-Large fc1 at 80 % sparsity, 128 images.
        _case("step", "wide_step", 1024, 4096, 819, 128 * 197, "bf16"),
        # The benchmark's step on one block of the ViT-Base stack at 256 images: the largest work.
        {"kind": "stack", "name": "stack_block", "tokens": 256 * 197, "sparsity": 90},
        # Training with the differentiable selection (soft TopK weights and their gradients), attention projection.
        _case("soft", "soft_step", 768, 768, 77, 64 * 197, "bf16"),
        # Training in fp32 (gradient checks, runs where bf16 is not trusted): attention projection at 16 images.
        _case("step", "f32_step", 768, 768, 77, 16 * 197, "f32"),
        # Widths that are no multiple of any tile, an odd token count: a narrow layer feeding a 1000-way head.
        _case("step", "ragged_step", 320, 1000, 100, 5005, "bf16"),
        # Extreme sparsity (a handful of diagonals per layer, 99.6 %).
        _case("step", "few_diagonals_step", 1024, 1024, 4, 128 * 197, "bf16"),
        # Query, key and value projections that share their input, as one group.
        dict(_case("shared", "qkv_step", 768, 768, 77, 64 * 197, "bf16"), sets=3),
        # The heuristic update of the active set, once per update interval: magnitudes, drop, grow.
        dict(_case("heur", "heuristic_update", 3072, 768, 307, 0, "bf16"), drop=92),
    ]


def _case(kind, name, M, N, K, T, dtype):
    return {"kind": kind, "name": name, "in": M, "out": N, "K": K, "tokens": T, "dtype": dtype}


def _log(rng, lo, hi):
    """An integer between lo and hi, uniform over the logarithm."""
    return min(hi, max(lo, round(lo * (hi / lo) ** rng.random())))


def draw(rng):
    kind = rng.choice(["step", "step_f32", "step_ragged", "step_few", "infer", "clustered", "soft", "shared", "heur", "stack"])
    wide = lambda: 128 * _log(rng, 1, 32)  # the widths the bf16 layers come in: 128 ... 4096
    pair = lambda: rng.choice([lambda w: (w, w), lambda w: (w, min(4 * w, 4096)), lambda w: (min(4 * w, 4096), w)])(wide())
    density = lambda D: synth.num_diagonals(D, rng.choice([60, 70, 80, 85, 90, 95]))
    tokens = lambda lo, hi: _log(rng, lo, hi)
    if kind == "stack":
        return {"kind": "stack", "tokens": tokens(4 * 197, 200 * 197), "sparsity": rng.choice([80, 90, 95])}
    if kind == "step_f32":
        M, N = _log(rng, 48, 1024), _log(rng, 48, 1024)
        if rng.random() < 0.7:
            M, N = -(-M // 32) * 32, -(-N // 32) * 32
        case = _case("step", "", M, N, density(max(M, N)), tokens(16, 6304), "f32")
    elif kind == "step_ragged":
        M, N = _log(rng, 48, 1536), _log(rng, 48, 1536)
        if rng.random() < 0.7:
            M, N = -(-M // 8) * 8, -(-N // 8) * 8
        case = _case("step", "", M, N, density(max(M, N)), tokens(50, 12608), "bf16")
    elif kind == "step_few":
        w = 128 * _log(rng, 4, 16)
        M, N = rng.choice([(w, w), (w, 2 * w), (2 * w, w)])
        case = _case("step", "", M, N, rng.randint(1, 8), tokens(1000, 25216), "bf16")
    elif kind == "heur":
        M, N = pair()
        K = density(max(M, N))
        case = dict(_case("heur", "", M, N, K, 0, rng.choice(["bf16", "f32"])), drop=max(1, min(K, max(M, N) - K) * rng.randint(5, 50) // 100))
    elif kind == "infer":
        M, N = pair()
        case = _case("infer", "", M, N, density(max(M, N)), tokens(1, 12608), "bf16")
    elif kind == "clustered":
        M, N = 128 * _log(rng, 4, 32), 128 * _log(rng, 4, 32)
        K = density(max(M, N))
        case = dict(_case("clustered", "", M, N, K, tokens(197, 25216), "bf16"), runs=rng.randint(1, 8))
    else:
        M, N = pair()
        case = _case(kind, "", M, N, density(max(M, N)), tokens(64, 12608 if kind != "step" else 25216), "bf16")
        if kind == "shared":
            case["sets"] = rng.randint(2, 4)
    # no dearer than the stack: bounds on the dense and on the sparse multiply-adds (fp32 and odd widths cost more of those)
    dense = case["tokens"] * case["in"] * case["out"] * case.get("sets", 1)
    sparse = case["tokens"] * case["K"] * min(case["in"], case["out"])
    over = max(dense / 1.5e11, sparse / {"step_f32": 6e8, "step_ragged": 2e9}.get(kind, 1e15), 1.0)
    case["tokens"] = int(case["tokens"] / over)
    del case["name"]
    return case


# ---- inputs: drawn on the device from the seed alone ----

def _dtype(case):
    return torch.float32 if case["dtype"] == "f32" else torch.bfloat16


def _generator(seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    return gen


def _normal(shape, std, dtype, gen):
    return (torch.randn(shape, device="cuda", generator=gen) * std).to(dtype)


def _offsets(D, K, gen):
    return torch.sort(torch.randperm(D, device="cuda", generator=gen)[:K])[0].to(torch.int32)


def _inputs(case, seed):
    """What the call reads: activations N(0, 1), values N(0, 0.02^2), scores N(0, 1), offsets uniform without repetition
    (or in runs)."""
    gen = _generator(seed)
    M, N, K, T, dtype = case["in"], case["out"], case["K"], case["tokens"], _dtype(case)
    D, L = max(M, N), min(M, N)
    S = case.get("sets", 0)
    a = {"values": _normal(((S, K, L) if S else (K, L)), 0.02, dtype, gen)}
    if case["kind"] in ("step", "soft"):
        a["scores"] = _normal((1, D), 1.0, torch.float32, gen)
    elif S:
        a["offsets"] = torch.stack([_offsets(D, K, gen) for _ in range(S)])
    elif case["kind"] == "clustered":
        a["offsets"] = torch.from_numpy(synth.draw_offsets_clustered(D, K, case["runs"], seed=int(seed))).cuda()
    else:
        a["offsets"] = _offsets(D, K, gen)
    if case["kind"] == "heur":
        a["random"] = torch.rand((D,), device="cuda", generator=gen)
        return a
    a["X"] = _normal((T, M), 1.0, dtype, gen)
    if case["kind"] in ("step", "soft", "shared"):
        a["dY"] = _normal(((S, T, N) if S else (T, N)), 1.0, dtype, gen)
    return a


def _stack(case, seed):
    return StackStep(blocks=1, tokens=case["tokens"], sets_attn=4, sets_mlp=1, score_sets=1, seed=int(seed),
                     device_inputs=True, distinct_sets=True, sparsity_percent=case["sparsity"])


def prepare(case, seed):
    if case["kind"] == "stack":
        return {"case": case, "stack": _stack(case, seed)}
    s = _inputs(case, seed)
    M, N, K, T, dtype = case["in"], case["out"], case["K"], case["tokens"], _dtype(case)
    new = lambda shape, d: torch.empty(shape, dtype=d, device="cuda")
    s.update(case=case, ws=dd.Workspace())
    kind = case["kind"]
    if kind in ("infer", "clustered"):
        s["prepared"] = dd.dd_prepare(s["offsets"], s["values"], M, N)  # once, when the weights are loaded
        s["Y"] = new((T, N), dtype)
    elif kind == "shared":
        s["prepared"] = dd.dd_prepare_shared(s["offsets"], s["values"], M, N)  # the buffer; refilled every step
        s["Y"], s["dX"] = new((case["sets"], T, N), dtype), new((T, M), dtype)
    elif kind in ("step", "soft"):
        s["selected"] = new((1, K), torch.int32)
        s["Y"], s["dX"], s["dV"] = new((T, N), dtype), new((T, M), dtype), new((K, min(M, N)), torch.float32)
        # operands are shared between the products where the matrix cores run them, as the stack step does
        s["matrix"] = case["dtype"] == "bf16" and M % 128 == 0 and N % 128 == 0 and K > 16
        s["prepared"] = dd.dd_prepare(torch.arange(K, dtype=torch.int32, device="cuda"), s["values"], M, N) if s["matrix"] else None
    if kind == "soft":
        D = max(M, N)
        s["alpha"], s["dalpha"], s["dscores"] = new((1, D), torch.float32), new((D,), torch.float32), new((1, D), torch.float32)
    return s


def run(s):
    case = s["case"]
    if case["kind"] == "stack":
        st = s["stack"]
        st.step()
        out = {"offsets_" + k: v for k, v in st.select_out.items()}
        for g in st.groups.values():
            out.update({g.name + "_Y": g.Y, g.name + "_dX": g.dX, g.name + "_dV": g.dValues})
        return out
    M, N, K, kind, ws = case["in"], case["out"], case["K"], case["kind"], s["ws"]
    if kind == "infer":
        return {"Y": dd.dd_fwd(s["X"], None, None, N, Y=s["Y"], prepared=s["prepared"])}
    if kind == "clustered":
        return {"Y": dd.dd_fwd(s["X"], s["offsets"], None, N, Y=s["Y"], prepared=s["prepared"], algo=dd.DD_ALGO_BLOCKS)}
    if kind == "heur":
        magnitudes = dd.dd_diag_magnitude(s["values"])
        new, source = dd.dd_diagheur_update(max(M, N), s["offsets"], magnitudes, s["random"], case["drop"], ws=ws)
        return {"magnitudes": magnitudes, "offsets": new, "source": source}
    if kind == "shared":
        dd.dd_prepare_shared(s["offsets"], s["values"], M, N, prepared=s["prepared"])
        dd.dd_fwd_shared(s["X"], s["prepared"], Y=s["Y"])
        dd.dd_bwd_input_shared(s["dY"], s["prepared"], dX=s["dX"])
        dV = [dd.dd_bwd_weight(s["X"], s["dY"][i], s["offsets"][i], ws=ws) for i in range(case["sets"])]
        return {"Y": s["Y"], "dX": s["dX"], "dV": dV}
    if kind == "soft":
        offsets = s["selected"][0]
        dd.dd_select_soft(s["scores"], K, TEMPERATURE, offsets_out=s["selected"], alpha_tilde=s["alpha"])
        if s["matrix"]:
            dd.dd_prepare_scaled(offsets, s["alpha"][0], s["values"], M, N, prepared=s["prepared"])
            dd.dd_fwd(s["X"], None, None, N, Y=s["Y"], prepared=s["prepared"])
            dd.dd_bwd_input(s["dY"], None, None, M, dX=s["dX"], prepared=s["prepared"])
        else:
            effective = dd.dd_scale_values(offsets, s["alpha"][0], s["values"])
            dd.dd_fwd(s["X"], offsets, effective, N, Y=s["Y"], ws=ws)
            dd.dd_bwd_input(s["dY"], offsets, effective, M, dX=s["dX"], ws=ws)
        dd.dd_bwd_weight_scaled(s["X"], s["dY"], offsets, s["alpha"][0], s["values"], dV=s["dV"], d_alpha_tilde=s["dalpha"], ws=ws)
        dd.dd_soft_topk_bwd(s["scores"], K, TEMPERATURE, s["dalpha"].view(1, -1), d_scores=s["dscores"])
        return {"offsets": s["selected"], "alpha": s["alpha"], "Y": s["Y"], "dX": s["dX"], "dV": s["dV"], "dscores": s["dscores"]}
    offsets = s["selected"][0]
    if s["matrix"]:
        dd.dd_select_prepare(s["scores"][0], s["values"], M, N, offsets_out=offsets, prepared=s["prepared"])
        dd.dd_fwd(s["X"], None, None, N, Y=s["Y"], prepared=s["prepared"])
    else:
        dd.dd_select_diagonals(s["scores"], K, offsets_out=s["selected"], ws=ws)
        dd.dd_fwd(s["X"], offsets, s["values"], N, Y=s["Y"], ws=ws)
    dd.dd_bwd(s["X"], s["dY"], offsets, s["values"], dX=s["dX"], dValues=s["dV"], ws=ws, prepared=s["prepared"])
    return {"offsets": s["selected"], "Y": s["Y"], "dX": s["dX"], "dV": s["dV"]}


# ---- what the path cannot do without ----

def _products_work(M, N, K, T, size, S=1, fwd_only=False):
    L = min(M, N)
    if fwd_only:
        return {"bytes": size * (T * (M + N) + K * L) + 4 * K, "flops": 2.0 * T * K * L}
    # X and values in once, dY in, Y and dX out, dV out; a group has one X and one dX
    return {"bytes": size * (2 * T * M + 2 * S * T * N + S * K * L) + 4 * S * (K * L + K + max(M, N)),
            "flops": 3 * 2.0 * S * T * K * L}


def work(case):
    if case["kind"] == "stack":
        T, S = case["tokens"], case["sparsity"]
        total = {"bytes": 0, "flops": 0.0}
        for M, N, layers in ((768, 768, 4), (768, 3072, 1), (3072, 768, 1)):
            w = _products_work(M, N, synth.num_diagonals(max(M, N), S), T, 2)
            total = {k: total[k] + layers * w[k] for k in total}
        return total
    M, N, K, T = case["in"], case["out"], case["K"], case["tokens"]
    D, L = max(M, N), min(M, N)
    size = 4 if case["dtype"] == "f32" else 2
    if case["kind"] == "heur":
        return {"bytes": size * K * L + 4 * (D + 5 * K), "flops": float(K * L)}
    if case["kind"] in ("infer", "clustered"):
        return _products_work(M, N, K, T, size, fwd_only=True)
    w = _products_work(M, N, K, T, size, S=case.get("sets", 1))
    if case["kind"] == "soft":
        w["bytes"] += 4 * 2 * D
    return w


def tolerance(case):
    """About four times what two correct paths differ by (the matrix-core kernels against the vector kernels, the diagonals
    given in another order, the tokens in reverse), measured on the listed cases: fp32 results 7e-7 (largest element
    4e-6); results rounded to bf16 up to 4e-5 with K = 819 (a few roundings turned the other way, each one unit in the
    last place, 7.8e-3 of the element)."""
    if case["kind"] == "heur":
        return {"rel": 5e-7, "max": 2e-6}   # sums of absolute values; the chosen sets are whole numbers
    if case.get("dtype") == "f32":
        return {"rel": 3e-6, "max": 1.6e-5}
    return {"rel": 2e-4, "max": 3.2e-2}


# ---- the same in 64 bits, by dense matrix products ----

def _dense(M, N, offsets, values):
    D, L = max(M, N), min(M, N)
    o = offsets.long() % D
    p = torch.arange(L, device=o.device)
    q = (p[None, :] + o[:, None]) % D
    pp = p[None, :].expand_as(q)
    W = torch.zeros((M, N), dtype=torch.float64, device=o.device)
    W.index_put_((pp, q) if M <= N else (q, pp), values.double(), accumulate=True)
    return W, (pp, q) if M <= N else (q, pp)


def _topk(scores, K):
    order = torch.sort(scores.double(), dim=-1, descending=True, stable=True)[1]
    return torch.sort(order[..., :K], dim=-1)[0]


def _exact_products(M, N, offsets, values, X, dY):
    W, at = _dense(M, N, offsets, values)
    X, dY = X.double(), dY.double()
    return X @ W, dY @ W.t().contiguous(), (X.t().contiguous() @ dY)[at]


def exact(case, seed):
    if case["kind"] == "stack":
        st = _stack(case, seed)
        out = {"offsets_" + k: None for k in st.select_out}
        for g in st.groups.values():
            offsets = _topk(st.scores[g.select][0], g.K)[g.select_row0:g.select_row0 + g.n_layers]
            each = [_exact_products(g.M, g.N, offsets[j], g.values[j], g.X[j % g.sets], g.dY[j % g.sets]) for j in range(g.n_layers)]
            out.update({g.name + "_Y": [e[0] for e in each], g.name + "_dX": [e[1] for e in each],
                        g.name + "_dV": torch.stack([e[2] for e in each])})
        return out
    a = _inputs(case, seed)
    M, N, K, kind = case["in"], case["out"], case["K"], case["kind"]
    if kind == "heur":
        return {"magnitudes": a["values"].double().abs().sum(1), "offsets": None, "source": None}
    if kind in ("infer", "clustered"):
        return {"Y": a["X"].double() @ _dense(M, N, a["offsets"], a["values"])[0]}
    if kind == "shared":
        each = [_exact_products(M, N, a["offsets"][i], a["values"][i], a["X"], a["dY"][i]) for i in range(case["sets"])]
        return {"Y": torch.stack([e[0] for e in each]), "dX": sum(e[1] for e in each), "dV": [e[2] for e in each]}
    offsets = _topk(a["scores"], K)[0]
    if kind == "step":
        Y, dX, dV = _exact_products(M, N, offsets, a["values"], a["X"], a["dY"])
        return {"offsets": None, "Y": Y, "dX": dX, "dV": dV}
    p = torch.softmax(a["scores"].double() / TEMPERATURE, dim=-1)
    alpha = torch.clamp(K * p, max=1.0)
    weight = alpha[0][offsets][:, None]
    Y, dX, dV = _exact_products(M, N, offsets, a["values"].double() * weight, a["X"], a["dY"])
    dalpha = torch.zeros_like(alpha)
    dalpha[0][offsets] = (dV * a["values"].double()).sum(1)
    open_ = torch.where(K * p < 1, dalpha, torch.zeros_like(dalpha))
    dscores = K / TEMPERATURE * p * (open_ - (open_ * p).sum())
    return {"offsets": None, "alpha": alpha, "Y": Y, "dX": dX, "dV": dV * weight, "dscores": dscores}
