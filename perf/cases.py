"""The work that users of this library have it do, as measurable cases.

A case is a dict of plain values; `prepare` makes what a program holds before the call (activations, masks,
registered weights, output buffers), `run` makes one pass through the public entry points
(`FMoE.layer_forward`, the single steps of it, `FMoEStack.forward`).  The layer shapes are those of the
library's own workloads: `tiny` (d 128, 8 experts of 256), `small` (d 1280, 64 experts of 896 and two shared),
`medium` (d 2048, 64 experts of 1408 and two shared), `wide` (d 2048, 128 experts of 768).
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

from paper_2511_17885_amd import binding

# d_model, experts, d_ffn, shared experts, top-k for text, router bias deviation, mixture components of the visual
# tokens, tokens per image tile (0: one mixture for the whole image), window
SHAPES = {
    "tiny": (128, 8, 256, 0, 2, 0.0, 16, 0, 4),
    "small": (1280, 64, 896, 2, 6, 1.0, 96, 0, 3),
    "medium": (2048, 64, 1408, 2, 6, 1.0, 192, 0, 3),
    "wide": (2048, 128, 768, 0, 8, 1.5, 64, 256, 5),
}
BATCH_VISUAL = "4864,1024,1536,1536,2048,1792,5120,3072"   # the library's ragged batch
LAYERS = 12        # depth of the stack cases
FULL_LAYERS = 2    # its first layers activate k_text experts for every token; the next one prunes


def _case(name, path, shape, visual, text, *, dtype="bf16", k_visual, retention=1.0, window=None, gamma=0.0,
          alpha=1.0, attention=False, residual=True):
    c = {"path": path, "shape": shape, "dtype": dtype, "visual": visual, "text": text, "k_visual": k_visual,
         "retention": retention, "window": SHAPES[shape][8] if window is None else window, "gamma": gamma,
         "alpha": alpha, "attention": attention, "residual": residual}
    return c if name is None else dict(c, name=name)


def listed():
    return [
        # A handful of text tokens, one of each of eight conversations, through one layer: the weights of a few
        # dozen experts stream past eight rows.
        _case("text_8x1_medium", "layer", "medium", "0,0,0,0,0,0,0,0", "1,1,1,1,1,1,1,1", k_visual=3),
        # The smallest configuration, in fp32: what a test-bed or a reference run calls; nothing but latency.
        _case("tiny_f32", "layer", "tiny", "48", "16", dtype="f32", k_visual=1, retention=0.75, residual=False),
        # One small picture and a short question, odd sizes.
        _case("picture_416_small", "layer", "small", "389", "27", k_visual=3, retention=0.5),
        # One picture of ordinary size.
        _case("image_1600_small", "layer", "small", "1536", "64", k_visual=3, retention=0.5),
        # The same with everything the method has: attention term in the drop order and window merging, 75 % kept.
        _case("image_1600_small_merge", "layer", "small", "1536", "64", k_visual=3, retention=0.75, gamma=0.05,
              alpha=0.5, attention=True),
        # The same in the fp32 storage type, used to check a bf16 deployment against.
        _case("image_1600_small_f32", "layer", "small", "1536", "64", dtype="f32", k_visual=3, retention=0.5),
        # A large picture, half of its tokens kept.
        _case("image_4096_medium", "layer", "medium", "3840", "256", k_visual=3, retention=0.5),
        # A picture in 31 tiles.
        _case("tiles_8192_wide", "layer", "wide", "7936", "256", k_visual=4, retention=0.5),
        # The five steps called one by one (a caller with its own scheduling between them), three ragged sequences.
        _case("steps_5003_wide", "steps", "wide", "1801,257,2603", "113,31,198", k_visual=4, retention=0.75),
        # A packed batch of eight prompts, every token at full activation, nothing pruned: the layers below l_v.
        _case("batch_22016_medium_full", "layer", "medium", BATCH_VISUAL, "128," * 7 + "128", k_visual=6),
        # The same batch through a stack of twelve layers: full activation in the first two, then three experts
        # per visual token, half of the visual tokens dropped once.
        _case("stack_22016_medium", "stack", "medium", BATCH_VISUAL, "128," * 7 + "128", k_visual=3, retention=0.5),
    ]


def _spread(rng, total, parts):
    """`total` tokens over `parts` sequences, ragged."""
    w = [math.exp(rng.uniform(-1.0, 1.0)) for _ in range(parts)]
    n = [max(1, int(total * v / sum(w))) for v in w]
    return ",".join(str(v) for v in n)


def draw(rng):
    path = rng.choice(["layer"] * 7 + ["steps"] * 2 + ["stack"])
    shape = rng.choice(["tiny", "small", "small", "medium", "medium", "wide", "wide"])
    dtype = "f32" if shape == "tiny" or (shape == "small" and rng.random() < 0.3) else "bf16"
    if path == "stack":        # packed prompts
        shape, dtype, lo, hi = rng.choice(["small", "medium"]), "bf16", 4096, 18000
    else:
        lo, hi = 1, (3000 if dtype == "f32" else 20000)
    total = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    seqs = min(total, rng.choice([1, 1, 2, 3, 5, 8]))
    if total < 48:             # text turns
        visual, text = ",".join("0" * seqs), _spread(rng, total, seqs)
    else:
        share = rng.uniform(0.02, 0.2)
        visual, text = _spread(rng, total * (1.0 - share), seqs), _spread(rng, max(1.0, total * share), seqs)
    k = SHAPES[shape][4]
    retention = rng.choice([0.25, 0.5, 0.75, 1.0]) if total >= 48 else 1.0
    merge = path == "layer" and retention < 1.0 and rng.random() < 0.25
    attention = path == "layer" and retention < 1.0 and (merge or rng.random() < 0.25)
    return _case(None, path, shape, visual, text, dtype=dtype, k_visual=rng.randint(1, k), retention=retention,
                 window=rng.randint(2, 7), gamma=0.05 if merge else 0.0, alpha=0.5 if attention else 1.0,
                 attention=attention, residual=rng.random() < 0.7)


def _lens(text):
    return [int(v) for v in text.split(",")]


def _sequence_tokens(rng, g, n_visual, n_text, d, components, tile):
    """[visual, text] rows of one sequence: visual tokens from a mixture whose component runs over 1..16
    neighbours (adjacent patches are alike), text tokens on their own."""
    parts, done = [], 0
    while done < n_visual:
        n = min(tile, n_visual - done) if tile else n_visual
        runs = rng.integers(1, 17, size=n)
        comp = np.repeat(rng.integers(0, components, size=n), runs)[:n]
        centres = torch.randn((components, d), generator=g, device="cuda")
        parts.append(centres[torch.from_numpy(comp).cuda()] + 0.3 * torch.randn((n, d), generator=g, device="cuda"))
        done += n
    parts.append(torch.randn((n_text, d), generator=g, device="cuda"))
    return torch.cat(parts)


def _weights(case, g, down_std):
    """Router matrix, router bias (or None), gate / up / down projections of the experts and of the shared ones."""
    d, E, F, shared, _, bias_std, _, _, _ = SHAPES[case["shape"]]
    td = torch.float32 if case["dtype"] == "f32" else torch.bfloat16

    def w(*shape, std=0.02):
        return torch.empty(shape, dtype=td, device="cuda").normal_(0.0, std, generator=g)

    bias = torch.randn(E, generator=g, device="cuda") * bias_std if bias_std > 0.0 else None
    sh = [w(shared, F, d), w(shared, F, d), w(shared, d, F, std=down_std)] if shared else [None] * 3
    return [w(E, d), bias, w(E, F, d), w(E, F, d), w(E, d, F, std=down_std), *sh]


def _layer(case, g, down_std):
    d, E, F, shared, k, _, _, _, _ = SHAPES[case["shape"]]
    m = binding.FMoE(d_model=d, n_experts=E, d_ffn=F, n_shared=shared, d_ffn_shared=F if shared else 0, k_text=k,
                     k_visual=case["k_visual"], dtype=case["dtype"])
    m.set_weights(*_weights(case, g, down_std), release_packed=True)
    return m


def _inputs(case, g, rng):
    """Packed rows, modality mask, sequence offsets and the attention importance (or None)."""
    d, _, _, _, _, _, components, tile, _ = SHAPES[case["shape"]]
    nv, nt = _lens(case["visual"]), _lens(case["text"])
    td = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    x = torch.cat([_sequence_tokens(rng, g, a, b, d, components, tile) for a, b in zip(nv, nt)]).to(td).contiguous()
    vis = torch.from_numpy(np.concatenate([np.repeat([1, 0], [a, b]) for a, b in zip(nv, nt)]).astype(np.uint8)).cuda()
    cu = torch.from_numpy(np.concatenate([[0], np.cumsum(np.add(nv, nt))]).astype(np.int32)).cuda()
    # attention importance of every token: non-negative, long-tailed
    attn = torch.empty(x.shape[0], device="cuda").exponential_(1.0, generator=g) if case["attention"] else None
    return x, vis, cu, attn


def _generators(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed * 7919 + 17)
    return g, np.random.Generator(np.random.PCG64(seed))


def prepare(case, seed):
    d, k = SHAPES[case["shape"]][0], SHAPES[case["shape"]][4]
    g, rng = _generators(seed)
    nv, nt = _lens(case["visual"]), _lens(case["text"])
    x, vis, cu, attn = _inputs(case, g, rng)
    td = x.dtype
    T, B = x.shape[0], len(nv)
    params = None
    if case["retention"] < 1.0:
        params = binding.prune_params(retention=case["retention"], window=case["window"], alpha=case["alpha"],
                                      gamma=case["gamma"])
    kept = binding.kept_count(nv, nt, case["retention"])
    s = {"case": case, "x": x, "vis": vis, "cu": cu, "params": params, "attn": attn, "n": kept, "nv": nv, "nt": nt,
         "out": torch.empty((T, d), dtype=td, device="cuda"),
         "kept": torch.empty(T, dtype=torch.int32, device="cuda"),
         "new_cu": torch.empty(B + 1, dtype=torch.int32, device="cuda"),
         "vis_out": torch.empty(T, dtype=torch.uint8, device="cuda")}
    if case["path"] == "stack":
        # depth-scaled down projections keep the residual stream of a stack without normalisation at O(1)
        layers = [_layer(case, g, 0.02 / math.sqrt(2 * LAYERS)) for _ in range(LAYERS)]
        sched = [(k, k) if l < FULL_LAYERS else (k, case["k_visual"]) for l in range(LAYERS)]
        s["stack"] = binding.FMoEStack(layers, sched, prune_schedule={FULL_LAYERS: params} if params is not None else None)
    else:
        s["layer"] = _layer(case, g, 0.02)
        s["layer"].workspace(T, B)
    torch.cuda.current_stream().synchronize()
    return s


def run(state):
    case, x, vis, cu, n = state["case"], state["x"], state["vis"], state["cu"], state["n"]
    if case["path"] == "stack":
        out, kept, new_cu, vis_out = state["stack"].forward(x, vis, cu, state["nv"], state["nt"], out=state["out"],
                                                            kept_idx=state["kept"], new_cu=state["new_cu"],
                                                            want_mask=True)
        return {"out": out, "kept": kept, "new_cu": new_cu, "visual": vis_out}
    m = state["layer"]
    if case["path"] == "layer":
        out, kept, new_cu, vis_out = m.layer_forward(x, vis, cu, state["params"], attn=state["attn"],
                                                     add_residual=case["residual"], out=state["out"],
                                                     kept_idx=state["kept"], new_cu=state["new_cu"],
                                                     is_visual_out=state["vis_out"])
        return {"out": out[:n], "kept": kept[:n], "new_cu": new_cu, "visual": vis_out[:n]}
    probs, idx, gate = m.route(x, vis)
    if state["params"] is not None:
        kept, new_cu, _ = m.prune(state["params"], probs, vis, cu)
    else:
        kept, new_cu = None, cu
    offs, perm, inv = m.permute(idx, kept, n)
    y, y_shared = m.expert_ffn(x, kept, n, offs, perm)
    out = m.combine(y, y_shared, inv, gate, kept, n, residual=x if case["residual"] else None)
    r = {"probs": probs, "experts": idx, "gates": gate, "new_cu": new_cu, "offsets": offs, "inv": inv, "out": out}
    if kept is not None:
        r["kept"] = kept[:n]
    return r


@functools.lru_cache(maxsize=None)
def _experts_touched(shape, n_visual, n_text, k_visual, k_text):
    """Experts that at least one kept token is routed to: mean over draws of the router's logits with the inputs' own
    distribution (a mixture component's logit, the deviation inside a component, the bias)."""
    d, E, _, _, _, bias_std, components, tile, _ = SHAPES[shape]
    rng, got = np.random.default_rng(1), []
    n_visual, n_text = min(n_visual, 4096), min(n_text, 1024)
    components = min(components * (max(1, n_visual // tile) if tile else 1), max(1, n_visual // 8))
    for _ in range(4):
        std, bias = 0.02 * math.sqrt(d), rng.standard_normal(E) * bias_std
        hit = np.zeros(E, bool)
        if n_visual and k_visual:
            z = rng.standard_normal((components, E))[rng.integers(0, components, n_visual)]
            z = bias + std * (z + 0.3 * rng.standard_normal((n_visual, E)))
            hit[np.argpartition(-z, k_visual - 1)[:, :k_visual]] = True
        if n_text and k_text:
            z = bias + std * rng.standard_normal((n_text, E))
            hit[np.argpartition(-z, k_text - 1)[:, :k_text]] = True
        got.append(int(hit.sum()))
    return sum(got) / len(got)


def work(case):
    d, E, F, shared, k, _, _, _, _ = SHAPES[case["shape"]]
    es = 4 if case["dtype"] == "f32" else 2
    nv, nt = _lens(case["visual"]), _lens(case["text"])
    text = sum(nt)
    stack = case["path"] == "stack"
    vis_in, total_bytes, flops = sum(nv), 0.0, 0.0
    for l in range(LAYERS if stack else 1):
        kv = k if stack and l < FULL_LAYERS else case["k_visual"]
        vis_out = vis_in
        if case["retention"] < 1.0 and l == (FULL_LAYERS if stack else 0):
            vis_out = sum(binding.kept_visual_lens(nv, case["retention"]))
        rows = text * k + vis_out * kv
        n = text + vis_out
        flops += 2.0 * (vis_in + text) * d * E + 6.0 * rows * d * F + 6.0 * n * d * F * shared
        total_bytes += es * 3.0 * d * F * (_experts_touched(case["shape"], vis_out, text, kv, k) + shared)   # weights
        total_bytes += es * d * E                                                                            # router
        vis_in = vis_out
    total_bytes += es * d * (sum(nv) + text + vis_in + text) + 5.0 * (sum(nv) + text)   # input, output, masks, lists
    if case["path"] == "steps":    # the steps hand over through the caller's tensors
        n_in, n, rows = sum(nv) + text, vis_in + text, text * k + vis_in * case["k_visual"]
        total_bytes += 4.0 * E * n_in * (2 if case["retention"] < 1.0 else 1) + 8.0 * k * (2 * n_in + 3 * n)
        total_bytes += 2.0 * es * d * (rows + shared * n)
    return {"bytes": total_bytes, "flops": flops}


def tolerance(case):
    # Against fp64 with the router's own decisions the listed layers are off by rel 2e-3, max 9e-3 (bf16) and rel
    # 4e-7, max 2e-6 (fp32): four times that.  Decisions (experts, kept tokens) are reproducible and stay the same.
    return {"rel": 2e-6, "max": 1e-5} if case["dtype"] == "f32" else {"rel": 8e-3, "max": 4e-2}


def _kept(case, P, attn, x):
    """Kept token indices and the layer input after merging: the drop rule and the window merging (token means
    rescaled to the window's largest norm) on fp64 routing probabilities."""
    W, r, alpha = case["window"], case["retention"], case["alpha"]
    gamma = float(np.float32(case["gamma"]))    # a C float in the parameters
    keep, xm, start = np.ones(P.shape[0], bool), x, 0
    for n_visual, n_text in zip(_lens(case["visual"]), _lens(case["text"])):
        n = (n_visual + W - 1) // W
        if n:
            rows = torch.zeros((n * W, P.shape[1]), dtype=torch.float64, device=P.device)
            rows[:n_visual] = P[start:start + n_visual]
            rows = rows.view(n, W, -1)
            size = torch.full((n,), W, device=P.device)
            size[-1] = n_visual - (n - 1) * W
            mean = rows.sum(1) / size[:, None]
            norms = rows.norm(dim=2) * mean.norm(dim=1)[:, None]
            cos = torch.where(norms > 0, (rows * mean[:, None]).sum(2) / norms.clamp_min(1e-300), 0.0)
            C = (cos.sum(1) / size).cpu().numpy()
            size = size.cpu().numpy()
            C[size == 1] = 1.0
            A = np.zeros(n)
            if attn is not None:
                A = np.pad(attn[start:start + n_visual].double().cpu().numpy(), (0, n * W - n_visual)).reshape(n, W).sum(1)
                A = A / A.max() if A.max() > 0 else A
                C = alpha * C - (1.0 - alpha) * A
            eta = max(1, min(n_visual, int(math.floor(r * n_visual + 0.5))))
            u, left, merged = n_visual - eta, int(math.floor(eta * gamma)), np.zeros(n, bool)
            for i in np.lexsort((np.arange(n), -C)):
                if left == 0:
                    break
                if 2 <= size[i] <= u + 1:
                    t = start + i * W
                    if xm is x:
                        xm = x.clone()
                    m = x[t:t + size[i]].double()
                    top, m = m.norm(dim=1).max(), m.mean(0)
                    xm[t] = (m * (top / m.norm())).to(x.dtype)
                    keep[t + 1:t + size[i]] = False
                    merged[i], u, left = True, u - (size[i] - 1), left - 1
            for i in np.lexsort((np.arange(n), -C, A)):
                if u == 0:
                    break
                if not merged[i]:
                    cut = min(u, size[i])
                    keep[start + i * W + size[i] - cut:start + i * W + size[i]] = False
                    u -= cut
        start += n_visual + n_text
    return torch.from_numpy(np.flatnonzero(keep)).cuda(), xm


def exact(case, seed):
    """The floating outputs in 64 bits.  Near-ties can be decided differently from the fp32 routing probabilities;
    down a stack those differences travel, so the stack has none."""
    if case["path"] == "stack":
        return None
    d, E, F, shared, k, _, _, _, _ = SHAPES[case["shape"]]
    g, rng = _generators(seed)
    x, vis, _, attn = _inputs(case, g, rng)
    router, bias, w_gate, w_up, w_down, s_gate, s_up, s_down = _weights(case, g, 0.02)
    kmax = max(k, case["k_visual"])

    def route(v, visual):
        z = v.double() @ router.double().T
        P = torch.softmax(z if bias is None else z + bias.double(), dim=1)
        p, e = P.topk(kmax, dim=1)
        live = torch.arange(kmax, device=v.device)[None, :] < torch.where(visual.bool(), case["k_visual"], k)[:, None]
        p = p * live
        return P, p / p.sum(1, keepdim=True), torch.where(live, e, -1)

    def ffn(v, a, b, c):
        return (torch.nn.functional.silu(v @ a.double().T) * (v @ b.double().T)) @ c.double().T

    P, gates, experts = route(x, vis)
    kept, xm = torch.arange(x.shape[0], device=x.device), x
    if case["retention"] < 1.0:
        kept, xm = _kept(case, P, attn, x)
    v, gk, ek = xm[kept], gates[kept], experts[kept]
    if xm is not x:
        _, gk, ek = route(v, vis[kept])
    v = v.double()
    out = v.clone() if case["residual"] else torch.zeros_like(v)
    for i in range(shared):
        out += ffn(v, s_gate[i], s_up[i], s_down[i])
    for e in range(E):
        row, slot = (ek == e).nonzero(as_tuple=True)
        if len(row):
            out[row] += gk[row, slot, None] * ffn(v[row], w_gate[e], w_up[e], w_down[e])
    if case["path"] == "layer":
        return {"out": out}
    return {"probs": P, "gates": gates, "out": out}
