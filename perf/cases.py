"""The framework's path as its users run it, case by case: what is timed and compared when a kernel changes.

Every case goes through the public entry points of ``paper_2609_00891_amd``:

* ``build``     single-layer maps from calibration batches: ``cb_stats_zero``, one ``cb_stats_accumulate``
                (or ``cb_stats_accumulate_rope``) per batch, ``cb_ridge_solve``;
* ``centered``  the same fit from centered moments, in one pass about a pilot's means or in two passes;
* ``probe``     layer selection: a centered fit and its R^2 for every (target layer, source layer, head, K/V);
* ``attn``      attention-aligned calibration weights: ``cb_attn_sensitivity`` and ``cb_attn_weights``;
* ``apply``     a sender's cache mapped into the receiver's, with or without the rotary transforms, by
                single-layer (k = 1) or multi-layer maps;
* ``k_stats``   multi-layer moments of a calibration batch (k selected source layers per map);
* ``k_solve``   the wide ridge systems of those moments, in a caller's workspace or without one.

Geometries are the repository's own: Qwen3-14B -> 32B shaped caches (40 x 8 x 128 -> 64 x 8 x 128), the
mismatched pair (26 x 8 x 96 -> 40 x 4 x 128), the tiny one (1 x 2 x 64), and slices of them by target layer
(how the work is sharded over GPUs).
"""
import math

import numpy as np
import torch

import paper_2609_00891_amd as cb

LAM = 1e-2                                  # relative ridge of every workload
SRC_THETA, TGT_THETA = 1e4, 1e6
FLAGS = cb.CB_LAMBDA_RELATIVE | cb.CB_RIDGE_BIAS_UNPENALIZED

QWEN = dict(L_s=40, H_s=8, d_s=128, L_t=64, H_t=8, d_t=128)
MISMATCH = dict(L_s=26, H_s=8, d_s=96, L_t=40, H_t=4, d_t=128)
TINY = dict(L_s=1, H_s=2, d_s=64, L_t=1, H_t=2, d_t=64)


def listed():
    return [
        # the smallest build (4 maps, 1,024 tokens): launches and latency
        dict(name="build_tiny", kind="build", **TINY, seqs=4, seq_len=256, batches=1, rope="none", token_major=False),
        # a build streamed one 2,048-token calibration sequence per call, then all 1,024 systems
        dict(name="build_seq", kind="build", **QWEN, seqs=1, seq_len=2048, batches=4, rope="none", token_major=False),
        # a large resident calibration batch whose keys carry rotary positions on both sides
        dict(name="build_batch_rope", kind="build", **QWEN, seqs=16, seq_len=2048, batches=1, rope="both",
             token_major=False),
        # centered fit between models of different head widths, ragged sequences, one pass about a pilot
        dict(name="centered_mismatch", kind="centered", **MISMATCH, seqs=6, seq_len=1531, form="one_pass"),
        # layer selection for a slice of 16 target layers against all 40 source layers
        dict(name="probe_16_layers", kind="probe", **dict(QWEN, L_t=16), seqs=4, seq_len=1024),
        # attention-aligned weights of four 1,024-token sequences, 32 boundaries, every fourth position
        dict(name="attn_weights", kind="attn", L_t=64, H_t=8, d_t=128, group=8, bounds=32, seqs=4, seq_len=1024,
             stride=4),
        # the online handoff of one short prompt, decode-ready (both rotary transforms)
        dict(name="apply_prompt", kind="apply", **QWEN, k=1, seqs=1, seq_len=777, rope="both", token_major=False),
        # the handoff of one 32,768-token context
        dict(name="apply_long", kind="apply", **QWEN, k=1, seqs=1, seq_len=32768, rope="none", token_major=False),
        # the k = 8 construction's moments from a batch of eight 1,024-token sequences, every fourth token
        dict(name="k8_stats", kind="k_stats", **QWEN, k=8, seqs=8, seq_len=1024, stride=4),
        # one GPU's share of the k = 8 systems when eight GPUs build (8 target layers)
        dict(name="k8_solve_shard", kind="k_solve", n=128, k=8, d_t=128, workspace=True),
        # k = 8 systems of four target layers where nothing may be allocated
        dict(name="k8_solve_noalloc", kind="k_solve", n=64, k=8, d_t=128, workspace=False),
        # the k = 8 handoff of a ragged prompt, decode-ready
        dict(name="k8_apply_prompt", kind="apply", **QWEN, k=8, seqs=1, seq_len=1500, rope="target",
             token_major=False),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _slice(rng, g, lo=2):
    """A geometry with some of its target layers (a shard by target layer)."""
    return dict(g, L_t=min(g["L_t"], _log(rng, lo, g["L_t"]))) if g["L_t"] > lo else dict(g)


def draw(rng):
    kind = rng.choice(["build", "centered", "probe", "attn", "apply", "apply", "k_stats", "k_solve", "k_apply"])
    if kind == "build":
        g = _slice(rng, rng.choice([QWEN, MISMATCH, TINY]))
        rope = rng.choice(["none", "both", "source"]) if g["d_s"] == g["d_t"] else "none"
        return dict(kind="build", **g, seqs=_log(rng, 1, 8), seq_len=_log(rng, 40, 2500), batches=rng.randint(1, 3),
                    rope=rope, token_major=rng.random() < 0.3)
    if kind == "centered":
        g = _slice(rng, rng.choice([QWEN, MISMATCH]))
        return dict(kind="centered", **g, seqs=_log(rng, 2, 10), seq_len=_log(rng, 60, 2200),
                    form=rng.choice(["one_pass", "two_pass"]))
    if kind == "probe":
        g = rng.choice([QWEN, MISMATCH])
        g = dict(g, L_s=rng.randint(4, g["L_s"]), L_t=rng.randint(2, 10))
        return dict(kind="probe", **g, seqs=_log(rng, 1, 4), seq_len=_log(rng, 100, 1100))
    if kind == "attn":
        return dict(kind="attn", L_t=_log(rng, 4, 64), H_t=rng.choice([4, 8]), d_t=rng.choice([64, 128]),
                    group=rng.choice([2, 4, 8]), bounds=rng.randint(6, 32), seqs=rng.randint(1, 4),
                    seq_len=_log(rng, 100, 1100), stride=rng.choice([1, 4]))
    if kind == "apply":
        g = _slice(rng, rng.choice([QWEN, MISMATCH]))
        rope = rng.choice(["none", "both", "target"]) if g["d_s"] != 96 else rng.choice(["none", "target"])
        return dict(kind="apply", **g, k=1, seqs=rng.randint(1, 4), seq_len=_log(rng, 20, 8000), rope=rope,
                    token_major=rng.random() < 0.3)
    if kind == "k_stats":
        g = _slice(rng, QWEN)
        return dict(kind="k_stats", **g, k=rng.randint(2, 8), seqs=_log(rng, 1, 8), seq_len=_log(rng, 100, 1024),
                    stride=rng.choice([1, 4]))
    if kind == "k_solve":
        return dict(kind="k_solve", n=_log(rng, 4, 64), k=rng.randint(2, 8), d_t=128, workspace=rng.random() < 0.5)
    g = _slice(rng, QWEN)
    return dict(kind="apply", **g, k=rng.randint(2, 8), seqs=rng.randint(1, 2), seq_len=_log(rng, 20, 700),
                rope=rng.choice(["none", "both", "target"]), token_major=rng.random() < 0.3)


# ---------------------------------------------------------------- inputs

def _gen(seed, salt):
    return torch.Generator(device="cuda").manual_seed((int(seed) * 1000003 + salt) & ((1 << 62) - 1))


def _src_layer(c, l):
    """round(l (L_s - 1) / (L_full - 1)) for target layer l of the model the slice is taken from."""
    full = 64 if c["d_s"] == 128 else 40 if c["d_s"] == 96 else 1
    n = max(full, c["L_t"]) - 1
    return (2 * l * (c["L_s"] - 1) + n) // (2 * n) if n > 0 else 0


def _window(c, l):
    """The k consecutive source layers centred on the target layer's, clipped to the source model."""
    start = min(max(_src_layer(c, l) - c["k"] // 2, 0), c["L_s"] - c["k"])
    return list(range(start, start + c["k"]))


def _heads(c, h):
    return h * (c["H_s"] // c["H_t"])


def _head_map(c):
    """Maps in the order (target layer, K/V, target head); with k, the source layers of each."""
    rows = []
    for l in range(c["L_t"]):
        layers = _window(c, l) if c.get("k", 1) > 1 else _src_layer(c, l)
        rows += [(l, h, z, layers, _heads(c, h), l * c["H_t"] + h) for z in range(2) for h in range(c["H_t"])]
    tl, th, kv, sl, sh, wr = zip(*rows)
    out = dict(tgt_layer=tl, tgt_head=th, kv=kv, src_head=sh, weight_row=wr)
    out["src_layers" if c.get("k", 1) > 1 else "src_layer"] = sl
    return {k: np.asarray(v, dtype=np.int32) for k, v in out.items()}


def _probe_map(c):
    rows = [(l, h, z, j, _heads(c, h), l * c["H_t"] + h)
            for l in range(c["L_t"]) for j in range(c["L_s"]) for z in range(2) for h in range(c["H_t"])]
    names = ("tgt_layer", "tgt_head", "kv", "src_layer", "src_head", "weight_row")
    return {k: np.asarray(v, dtype=np.int32) for k, v in zip(names, zip(*rows))}


def _empty_cache(L, B, H, T, d, token_major=False):
    """[layer][2][seq][head][tok][d]; token_major: the heads of a token lie side by side."""
    if token_major:
        return torch.empty((L, 2, B, T, H, d), dtype=torch.bfloat16, device="cuda").transpose(3, 4)
    return torch.empty((L, 2, B, H, T, d), dtype=torch.bfloat16, device="cuda")


def _angles(theta, d, T, pos0):
    f = theta ** (-2.0 * torch.arange(d // 2, dtype=torch.float64, device="cuda") / d)
    a = (pos0 + torch.arange(T, dtype=torch.float64, device="cuda"))[:, None] * f
    return torch.cos(a), torch.sin(a)


def _turn(x, cs, inverse=False):
    """Half-split rotary transform of rows x [..., T, d] (any float type)."""
    c, s = (v.to(x.dtype) for v in cs)
    s = -s if inverse else s
    a, b = x.chunk(2, dim=-1)
    return torch.cat([a * c - b * s, b * c + a * s], dim=-1)


POS0 = 5                                     # position of a sequence's first token where keys carry rotary positions


def _source(c, B, seed, means=0.0, turned=False):
    """Per-channel lognormal scales with four x20 outlier channels per (layer, K/V, head); `means`: channel means
    of that many scales."""
    L, H, d, T = c["L_s"], c["H_s"], c["d_s"], c["seq_len"]
    x = _empty_cache(L, B, H, T, d, c.get("token_major", False))
    g = _gen(seed, 1)
    cs = _angles(SRC_THETA, d, T, POS0) if turned else None
    for l in range(L):
        s = torch.exp(torch.randn((2, 1, H, 1, d), generator=g, device="cuda"))
        out = torch.rand((2, 1, H, 1, d), generator=g, device="cuda").argsort(dim=-1) < 4
        s = torch.where(out, 20 * s, s)
        v = torch.randn((2, B, H, T, d), generator=g, device="cuda") * s
        if means:
            v += means * s * torch.randn((2, 1, H, 1, d), generator=g, device="cuda")
        if turned:
            v[0] = _turn(v[0], cs)
        x[l] = v
    return x


def _target(c, B, src, layers_of, seed, turned=False):
    """Planted affine targets y = x A + b + 0.1 N(0, 1) from the source layers of each target layer."""
    L, H, d, T = c["L_t"], c["H_t"], c["d_t"], c["seq_len"]
    y = _empty_cache(L, B, H, T, d, c.get("token_major", False))
    g = _gen(seed, 2)
    heads = torch.tensor([_heads(c, h) for h in range(H)], device="cuda")
    back = _angles(SRC_THETA, c["d_s"], T, POS0) if turned else None
    cs = _angles(TGT_THETA, d, T, POS0) if turned else None
    for l in range(L):
        ls = layers_of(l)
        x = torch.cat([src[j].index_select(2, heads).float() for j in ls], dim=-1)       # [2, B, H, T, k d_s]
        if turned:
            x[0] = _turn(x[0], back, inverse=True)
        p = x.shape[-1]
        A = torch.randn((2, H, p, d), generator=g, device="cuda") / math.sqrt(p)
        v = torch.bmm(x.transpose(1, 2).reshape(2 * H, B * T, p), A.reshape(2 * H, p, d))
        v = v.reshape(2, H, B, T, d).transpose(1, 2)
        v = v + torch.randn((2, 1, H, 1, d), generator=g, device="cuda")
        v = v + 0.1 * torch.randn(v.shape, generator=g, device="cuda")
        if turned:
            v[0] = _turn(v[0], cs)
        y[l] = v
    return y


def _weights(c, B, seed):
    """[row][seq * T + tok] fp32, skewed and decaying along the sequence, mean one per (row, sequence)."""
    R, T = c["L_t"] * c["H_t"], c["seq_len"]
    z = torch.randn((R, B, T), generator=_gen(seed, 3), device="cuda")
    w = torch.exp(z) / torch.sqrt(torch.arange(T, device="cuda") + 1.0)
    return (w / w.mean(dim=2, keepdim=True)).reshape(R, B * T)


def _table(theta, d, n_pos):
    t = torch.empty((n_pos, d // 2, 2), dtype=torch.float32, device="cuda")
    cb.cb_rope_table(theta, d, n_pos, t)
    return t


def _ropes(c):
    """(source spec, target spec) of a case's rope option, None where a side is not turned."""
    n = POS0 + c["seq_len"]
    src = cb.rope_spec(_table(SRC_THETA, c["d_s"], n), 0, POS0) if c["rope"] in ("both", "source") else None
    tgt = cb.rope_spec(_table(TGT_THETA, c["d_t"], n), 0, POS0) if c["rope"] in ("both", "target") else None
    return src, tgt


def _f32(*shape):
    return torch.empty(shape, dtype=torch.float32, device="cuda")


def _f64(*shape):
    return torch.empty(shape, dtype=torch.float64, device="cuda")


def prepare(case, seed):
    c = case
    return {"case": c, **_PREPARE[c["kind"]](c, seed)}


def _geoms(c):
    return (c["L_s"], c["H_s"], c["d_s"]), (c["L_t"], c["H_t"], c["d_t"])


def _prepare_build(c, seed):
    B, T, n, P = c["seqs"], c["seq_len"], 2 * c["L_t"] * c["H_t"], c["d_s"] + 1
    turned = c["rope"] != "none"
    src = _source(c, B * c["batches"], seed, turned=turned)
    tgt = _target(c, B * c["batches"], src, lambda l: [_src_layer(c, l)], seed, turned=turned)
    return dict(src=src, tgt=tgt, w=_weights(c, B * c["batches"], seed), ropes=_ropes(c),
                plan=cb.cb_plan_create(_head_map(c), *_geoms(c), B * T), G=_f32(n, P, P), C=_f32(n, P, c["d_t"]),
                maps=_f32(n, P, c["d_t"]), info=torch.empty(n, dtype=torch.int32, device="cuda"))


def _prepare_centered(c, seed, plan=None, n=None):
    B, T, ds, dt = c["seqs"], c["seq_len"], c["d_s"], c["d_t"]
    n = n or 2 * c["L_t"] * c["H_t"]
    src = _source(c, B, seed, means=30.0)
    tgt = _target(c, B, src, lambda l: [_src_layer(c, l)], seed)
    return dict(src=src, tgt=tgt, w=_weights(c, B, seed),
                plan=plan or cb.cb_plan_create(_head_map(c), *_geoms(c), B * T), sums=_f64(n, 1 + ds + dt),
                shift=_f64(n, 1 + ds + dt), A=_f32(n, ds, ds), B=_f32(n, ds, dt), maps=_f32(n, ds + 1, dt),
                info=torch.empty(n, dtype=torch.int32, device="cuda"))


def _prepare_probe(c, seed):
    n = 2 * c["L_t"] * c["H_t"] * c["L_s"]
    plan = cb.cb_plan_create(_probe_map(c), *_geoms(c), c["seqs"] * c["seq_len"])
    return dict(_prepare_centered(c, seed, plan, n), sq=_f64(n, c["d_s"] + c["d_t"]), r2=_f64(n))


def _boundaries(c):
    b = np.rint(np.geomspace(12, c["seq_len"] - 1, c["bounds"])).astype(np.int64)
    return np.unique(b).astype(np.int32)


def _prepare_attn(c, seed):
    L, H, d, B, T, G = c["L_t"], c["H_t"], c["d_t"], c["seqs"], c["seq_len"], c["group"]
    kv = _source(dict(L_s=L, H_s=H, d_s=d, seq_len=T), B, seed)
    b = _boundaries(c)
    g = _gen(seed, 4)
    q = torch.empty((L, B, len(b), H * G, d), dtype=torch.bfloat16, device="cuda")
    for l in range(L):
        scale = 2.0 / kv[l, 0].float().square().mean(dim=(0, 2, 3)).sqrt()            # scores of deviation 2
        v = torch.randn((B, len(b), H * G, d), generator=g, device="cuda")
        q[l] = v * scale.repeat_interleave(G)[:, None]
    R = 2 * L * H
    return dict(kv=kv, q=q, bounds=b, r=_f32(R, B * T), w=_f32(R, B * T), alpha=_f32(R))


def _prepare_apply(c, seed):
    B, T, k, n = c["seqs"], c["seq_len"], c["k"], 2 * c["L_t"] * c["H_t"]
    p = k * c["d_s"]
    maps = torch.randn((n, p + 1, c["d_t"]), generator=_gen(seed, 5), device="cuda")
    maps[:, :p] /= math.sqrt(p)
    plan = cb.cb_plan_create(_head_map(c), *_geoms(c), B * T) if k == 1 else \
        cb.cb_plan_create_multi(_head_map(c), *_geoms(c), 1)
    out = _empty_cache(c["L_t"], B, c["H_t"], T, c["d_t"], c["token_major"])
    return dict(src=_source(c, B, seed, turned=c["rope"] == "both"), maps=maps, plan=plan, ropes=_ropes(c), out=out)


def _prepare_k_stats(c, seed):
    B, n, P = c["seqs"], 2 * c["L_t"] * c["H_t"], c["k"] * c["d_s"] + 1
    src = _source(c, B, seed)
    tgt = _target(c, B, src, lambda l: _window(c, l), seed)
    return dict(src=src, tgt=tgt, w=_weights(c, B, seed),
                plan=cb.cb_plan_create_multi(_head_map(c), *_geoms(c), c["stride"]), G=_f32(n, P, P),
                C=_f32(n, P, c["d_t"]))


def _prepare_k_solve(c, seed):
    """Moments G = X^T X, C = X^T Y of scaled features, one system at a time."""
    n, dt = c["n"], c["d_t"]
    P, rows, g = c["k"] * 128 + 1, 2048, _gen(seed, 6)
    G, C = _f32(n, P, P), _f32(n, P, dt)
    for m in range(n):
        s = torch.exp(torch.randn(P - 1, generator=g, device="cuda"))
        x = torch.randn((rows, P), generator=g, device="cuda")
        x[:, :-1] *= s
        x[:, -1] = 1.0
        y = x @ (torch.randn((P, dt), generator=g, device="cuda") / math.sqrt(P))
        y += 0.1 * torch.randn((rows, dt), generator=g, device="cuda")
        v = x.t() @ x
        G[m] = torch.triu(v) + torch.triu(v, 1).t()                # exactly symmetric, as the moments are
        C[m] = x.t() @ y
    ws = None
    if c["workspace"]:
        ws = torch.empty(cb.cb_ridge_solve_workspace_bytes(P, dt, n), dtype=torch.uint8, device="cuda")
    return dict(G=G, C=C, ws=ws, maps=_f32(n, P, dt), info=torch.empty(n, dtype=torch.int32, device="cuda"))


_PREPARE = dict(build=_prepare_build, centered=_prepare_centered, probe=_prepare_probe, attn=_prepare_attn,
                apply=_prepare_apply, k_stats=_prepare_k_stats, k_solve=_prepare_k_solve)


# ---------------------------------------------------------------- one pass

def run(state):
    return _RUN[state["case"]["kind"]](state, state["case"])


def _run_build(s, c):
    B, T = c["seqs"], c["seq_len"]
    cb.cb_stats_zero(s["plan"], s["G"], s["C"])
    for b in range(c["batches"]):
        src, tgt = s["src"][:, :, b * B:(b + 1) * B], s["tgt"][:, :, b * B:(b + 1) * B]
        w = s["w"][:, b * B * T:(b + 1) * B * T]
        if c["rope"] == "none":
            cb.cb_stats_accumulate(s["plan"], src, tgt, w, s["G"], s["C"])
        else:
            cb.cb_stats_accumulate_rope(s["plan"], src, tgt, w, s["G"], s["C"], src_rope=s["ropes"][0],
                                        tgt_rope=s["ropes"][1])
    cb.cb_ridge_solve(s["G"], s["C"], LAM, FLAGS, s["maps"], s["info"])
    return {k: s[k] for k in ("G", "C", "maps", "info")}


def _run_centered(s, c):
    plan, src, tgt, w = s["plan"], s["src"], s["tgt"], s["w"]
    cb.cb_stats_zero_centered(plan, s["sums"], s["A"], s["B"])
    if c["form"] == "one_pass":
        T = c["seq_len"]
        s["shift"].zero_()
        cb.cb_stats_means(plan, src[:, :, :1], tgt[:, :, :1], w[:, :T], s["shift"])       # pilot: one sequence
        cb.cb_stats_accumulate_shifted(plan, src, tgt, w, s["shift"], s["sums"], s["A"], s["B"])
        cb.cb_stats_shift_finish(plan, s["shift"], s["sums"], s["A"], s["B"])
    else:
        cb.cb_stats_means(plan, src, tgt, w, s["sums"])
        cb.cb_stats_accumulate_centered(plan, src, tgt, w, s["sums"], s["A"], s["B"])
    cb.cb_ridge_solve_centered(s["sums"], s["A"], s["B"], LAM, cb.CB_LAMBDA_RELATIVE, s["maps"], s["info"])
    return {k: s[k] for k in ("sums", "A", "B", "maps", "info")}


def _run_probe(s, c):
    plan = s["plan"]
    cb.cb_stats_zero_centered(plan, s["sums"], s["A"], s["B"], s["sq"])
    cb.cb_stats_means(plan, s["src"], s["tgt"], s["w"], s["sums"], s["sq"])
    cb.cb_stats_accumulate_centered(plan, s["src"], s["tgt"], s["w"], s["sums"], s["A"], s["B"])
    cb.cb_ridge_solve_centered(s["sums"], s["A"], s["B"], LAM, cb.CB_LAMBDA_RELATIVE, s["maps"], s["info"])
    cb.cb_probe_r2(s["sums"], s["sq"], s["A"], s["B"], s["maps"], s["r2"])
    return {k: s[k] for k in ("sums", "sq", "A", "B", "maps", "info", "r2")}


def _run_attn(s, c):
    cb.cb_attn_sensitivity(s["kv"], s["q"], s["bounds"], c["stride"], s["r"])
    cb.cb_attn_weights(s["r"], c["seqs"], c["seq_len"], c["stride"], c["d_t"], s["w"], s["alpha"])
    return {k: s[k] for k in ("r", "w", "alpha")}


def _run_apply(s, c):
    if c["rope"] == "none":
        cb.cb_apply(s["plan"], s["maps"], s["src"], s["out"])
    else:
        cb.cb_apply_rope(s["plan"], s["maps"], s["src"], s["out"], tgt_rope=s["ropes"][1], src_rope=s["ropes"][0])
    return s["out"]


def _run_k_stats(s, c):
    cb.cb_stats_zero(s["plan"], s["G"], s["C"])
    cb.cb_stats_accumulate(s["plan"], s["src"], s["tgt"], s["w"], s["G"], s["C"])
    return {k: s[k] for k in ("G", "C")}


def _run_k_solve(s, c):
    if c["workspace"]:
        cb.cb_ridge_solve_ws(s["G"], s["C"], LAM, FLAGS, s["maps"], s["info"], s["ws"])
    else:
        cb.cb_ridge_solve_noalloc(s["G"], s["C"], LAM, FLAGS, s["maps"], s["info"])
    return {k: s[k] for k in ("maps", "info")}


_RUN = dict(build=_run_build, centered=_run_centered, probe=_run_probe, attn=_run_attn, apply=_run_apply,
            k_stats=_run_k_stats, k_solve=_run_k_solve)


# ---------------------------------------------------------------- what a pass cannot do without

def _solve_work(n, P, dt):
    """Cholesky and two substitutions; moments read, maps written."""
    return n * (P ** 3 / 3 + 2 * P * P * dt), 4 * n * (P * P + 2 * P * dt)


def work(case):
    c, kind = case, case["kind"]
    if kind == "k_solve":
        flops, nbytes = _solve_work(c["n"], c["k"] * 128 + 1, c["d_t"])
        return {"bytes": nbytes, "flops": flops}
    N = c["seqs"] * c["seq_len"] * c.get("batches", 1)
    n = 2 * c["L_t"] * c["H_t"]
    if kind == "attn":
        rows = len(_boundaries(c)) * c["group"]
        keys = int((_boundaries(c).astype(np.int64) + 1).sum()) * c["group"] * c["seqs"] * c["L_t"] * c["H_t"]
        nbytes = 2 * n * N * c["d_t"] + 2 * c["seqs"] * c["L_t"] * c["H_t"] * rows * c["d_t"] + 2 * 4 * n * N
        return {"bytes": nbytes, "flops": 2 * 3 * keys * c["d_t"]}
    if kind == "probe":
        blocks, n = 2 * c["L_s"] * c["H_t"], n * c["L_s"]
    elif c.get("k", 1) > 1:
        blocks = 2 * c["H_t"] * len({j for l in range(c["L_t"]) for j in _window(c, l)})
    else:
        blocks = 2 * c["H_t"] * len({_src_layer(c, l) for l in range(c["L_t"])})
    ds, dt = c["d_s"], c["d_t"]
    n_tgt, rows = 2 * c["L_t"] * c["H_t"], c["L_t"] * c["H_t"]
    if kind == "apply":
        P = c["k"] * ds + 1
        return {"bytes": 2 * N * (blocks * ds + n * dt) + 4 * n * P * dt, "flops": 2 * N * n * P * dt}
    if kind == "k_stats":
        P, R = c["k"] * ds + 1, c["seqs"] * -(-c["seq_len"] // c["stride"])
        return {"bytes": R * (2 * blocks * ds + 2 * n * dt + 4 * rows) + 4 * n * (P * P + P * dt),
                "flops": 2 * R * n * (P * (P + 1) / 2 + P * dt)}
    P = ds + 1
    flops, nbytes = _solve_work(n, P, dt)
    return {"bytes": N * (2 * blocks * ds + 2 * n_tgt * dt + 4 * rows) + nbytes + 4 * n * (P * P + P * dt),
            "flops": flops + 2 * N * n * (P * (P + 1) / 2 + P * dt)}


def tolerance(case):
    """Relative Frobenius errors; fp32 sums of exact bf16 products with weights or coefficients as two bf16 terms."""
    kind = case["kind"]
    if kind == "apply":
        return {"rel": 5e-4, "max": 0.02}                # a last-place difference of a bf16 value here and there
    if kind == "attn":
        return {"rel": 3e-5, "max": 3e-3}
    if kind == "k_solve":
        return {"rel": 1.5e-7, "max": 1e-5}              # fp64 inside, results rounded to fp32
    if kind == "build" and case["rope"] != "none":
        return {"rel": 6e-5, "max": 6e-3}                # de-rotated rows: a last-place difference of a bf16 value
    if kind == "k_stats":
        return {"rel": 6e-6, "max": 1e-3}
    return {"rel": 2e-5, "max": 2e-3}


# ---------------------------------------------------------------- the same in 64 bits

def _solve64(M, C):
    """M^-1 C by block Gauss-Jordan elimination, fp64 (M [n, P, P] positive definite)."""
    n, P, _ = M.shape
    A = torch.cat([M, C], dim=2)
    for b0 in range(0, P, 64):
        b1 = min(P, b0 + 64)
        D = torch.cat([A[:, b0:b1, b0:b1], torch.eye(b1 - b0, dtype=A.dtype, device=A.device).expand(n, -1, -1)], dim=2)
        for k in range(b1 - b0):
            row = D[:, k] / D[:, k, k, None]
            col = D[:, :, k].clone()
            D -= col[:, :, None] * row[:, None, :]
            D[:, k] = row
        rows = torch.bmm(D[:, :, b1 - b0:].contiguous(), A[:, b0:b1].contiguous())
        col = A[:, :, b0:b1].clone()
        col[:, b0:b1] = 0.0
        A[:, b0:b1] = rows
        A = torch.baddbmm(A, col, rows, alpha=-1.0)
    return A[:, :, P:].contiguous()


def _rows64(cache, l, z, h):
    """Rows [B T, d] of one (layer, K/V, head) in fp64."""
    return cache[l, z, :, h].reshape(-1, cache.shape[-1]).double()


def _turned_back(cache, spec, theta):
    """The cache with its keys' rotary transform removed in fp64 and rounded once to bf16."""
    if spec is None:
        return cache
    out = cache.clone()
    cs = _angles(theta, cache.shape[-1], cache.shape[4], POS0)
    for l in range(cache.shape[0]):
        out[l, 0] = _turn(cache[l, 0].double(), cs, inverse=True).to(torch.bfloat16)
    return out


def _moments64(c, src, tgt, w, layers_of, stride=1):
    """(G, C) of the augmented feature for the maps in head-map order."""
    T, dt = c["seq_len"], c["d_t"]
    keep = (torch.arange(w.shape[1], device="cuda") % T) % stride == 0
    G, C = [], []
    for l in range(c["L_t"]):
        X, Y, W = [], [], []
        for z in range(2):
            for h in range(c["H_t"]):
                x = torch.cat([_rows64(src, j, z, _heads(c, h)) for j in layers_of(l)], dim=1)[keep]
                X.append(torch.cat([x, torch.ones_like(x[:, :1])], dim=1))
                Y.append(_rows64(tgt, l, z, h)[keep])
                W.append(w[l * c["H_t"] + h].double()[keep])
        X, Y = torch.stack(X), torch.stack(Y)
        XW = (X * torch.stack(W)[:, :, None]).transpose(1, 2).contiguous()
        G.append(torch.bmm(XW, X))
        C.append(torch.bmm(XW, Y))
    return torch.cat(G), torch.cat(C)


def _ridge64(G, C):
    n, P, _ = G.shape
    lam = float(np.float32(LAM)) * G.diagonal(dim1=1, dim2=2).sum(dim=1) / P
    D = torch.eye(P, dtype=torch.float64, device="cuda")
    D[-1, -1] = 0.0
    return _solve64(G + lam[:, None, None] * D, C)


def _exact_build(c, s):
    src, tgt = (_turned_back(s["src"], s["ropes"][0], SRC_THETA), _turned_back(s["tgt"], s["ropes"][1], TGT_THETA))
    G, C = _moments64(c, src, tgt, s["w"], lambda l: [_src_layer(c, l)])
    return {"G": G, "C": C, "maps": _ridge64(G, C), "info": None}


def _centered64(c, s, layers_of):
    """sums, A, B, maps and the squares' sums of the maps (target layer, source layer of layers_of, K/V, head)."""
    res = {k: [] for k in ("sums", "sq", "A", "B", "maps", "r2")}
    lam = float(np.float32(LAM))
    for l in range(c["L_t"]):
        for j in layers_of(l):
            X, Y, W = [], [], []
            for z in range(2):
                for h in range(c["H_t"]):
                    X.append(_rows64(s["src"], j, z, _heads(c, h)))
                    Y.append(_rows64(s["tgt"], l, z, h))
                    W.append(s["w"][l * c["H_t"] + h].double())
            X, Y, W = torch.stack(X), torch.stack(Y), torch.stack(W)[:, :, None]
            S = W.sum(dim=1)
            sx, sy = (W * X).sum(dim=1), (W * Y).sum(dim=1)
            res["sums"].append(torch.cat([S, sx, sy], dim=1))
            res["sq"].append(torch.cat([(W * X * X).sum(dim=1), (W * Y * Y).sum(dim=1)], dim=1))
            mx, my = sx / S, sy / S
            U, V = X - mx[:, None], Y - my[:, None]
            UW = (U * W).transpose(1, 2).contiguous()
            A, B = torch.bmm(UW, U), torch.bmm(UW, V)
            d = A.shape[1]
            lm = lam * (A.diagonal(dim1=1, dim2=2).sum(dim=1) + S[:, 0] * (mx * mx).sum(dim=1) + S[:, 0]) / (d + 1)
            M = _solve64(A + lm[:, None, None] * torch.eye(d, dtype=torch.float64, device="cuda"), B)
            b = my - torch.bmm(mx[:, None], M)[:, 0]
            rss = (W * (V - torch.bmm(U, M)) ** 2).sum(dim=(1, 2))
            res["r2"].append(1.0 - rss / (W * V * V).sum(dim=(1, 2)))
            res["A"].append(A)
            res["B"].append(B)
            res["maps"].append(torch.cat([M, b[:, None]], dim=1))
    return {k: torch.cat(v) for k, v in res.items()}


def _exact_centered(c, s):
    v = _centered64(c, s, lambda l: [_src_layer(c, l)])
    return {"sums": v["sums"], "A": v["A"], "B": v["B"], "maps": v["maps"], "info": None}


def _exact_probe(c, s):
    return dict(_centered64(c, s, lambda l: range(c["L_s"])), info=None)


def _exact_attn(c, s):
    L, H, d, B, T, G, st = c["L_t"], c["H_t"], c["d_t"], c["seqs"], c["seq_len"], c["group"], c["stride"]
    b = torch.tensor(s["bounds"].astype(np.int64), device="cuda")
    nb, i = len(s["bounds"]), torch.arange(T, device="cuda")
    seen = (i[None] <= b[:, None])                                     # [nb, T]
    inE = (i[None] < b[:, None]) & (i[None] % st == 0)
    r = torch.zeros((2 * L * H, B * T), dtype=torch.float64, device="cuda")
    for l in range(L):
        for h in range(H):
            k, v = s["kv"][l, 0, :, h].double(), s["kv"][l, 1, :, h].double()            # [B, T, d]
            q = s["q"][l, :, :, h * G:(h + 1) * G].double().reshape(B, nb * G, d)
            sc = torch.bmm(q, k.transpose(1, 2).contiguous()).reshape(B, nb, G, T) / math.sqrt(d)
            a = torch.softmax(sc.masked_fill(~seen[None, :, None], float("-inf")), dim=-1)
            o = torch.bmm(a.reshape(B, nb * G, T), v)
            a2 = a * a
            vo = (v * v).sum(-1)[:, None] - 2 * torch.bmm(o, v.transpose(1, 2).contiguous()) + (o * o).sum(-1)[..., None]
            pk = (a2 * vo.reshape(B, nb, G, T) * ((q * q).sum(-1) / d).reshape(B, nb, G, 1)).sum(2) * inE
            pv = a2.sum(2) * inE
            for z, p in ((0, pk), (1, pv)):
                m = p.sum(-1, keepdim=True)
                r[(l * 2 + z) * H + h] = torch.where(m > 0, p / m, torch.zeros_like(p)).sum(1).reshape(-1)
    keep = (torch.arange(B * T, device="cuda") % T) % st == 0
    v = r[:, keep]
    n = v.shape[1]
    mean = v.mean(dim=1, keepdim=True)
    v = torch.where(mean > 0, v / mean, torch.ones_like(v))
    cv2 = ((v - 1) ** 2).mean(dim=1)
    tau = min(n, 2 * d)
    alpha = torch.where(cv2 > 0, torch.sqrt((n / tau - 1) / cv2).clamp(max=1.0), torch.ones_like(cv2))
    w = torch.zeros_like(r)
    w[:, keep] = 1 + alpha[:, None] * (v - 1)
    return {"r": r, "w": w, "alpha": alpha}


def _exact_apply(c, s):
    k, n = c["k"], 2 * c["L_t"] * c["H_t"]
    src = _turned_back(s["src"], s["ropes"][0], SRC_THETA)
    B, T, H, dt = c["seqs"], c["seq_len"], c["H_t"], c["d_t"]
    out = torch.empty((c["L_t"], 2, B, H, T, dt), dtype=torch.float64, device="cuda")
    cs = _angles(TGT_THETA, dt, T, POS0)
    for l in range(c["L_t"]):
        for z in range(2):
            for h in range(H):
                m = (l * 2 + z) * H + h
                layers = _window(c, l) if k > 1 else [_src_layer(c, l)]
                x = torch.cat([_rows64(src, j, z, _heads(c, h)) for j in layers], dim=1)
                W = s["maps"][m].double()
                y = (x @ W[:-1] + W[-1]).reshape(B, T, dt)
                out[l, z, :, h] = _turn(y, cs) if z == 0 and s["ropes"][1] is not None else y
    return out


def _exact_k_stats(c, s):
    G, C = _moments64(c, s["src"], s["tgt"], s["w"], lambda l: _window(c, l), c["stride"])
    return {"G": G, "C": C}


def _exact_k_solve(c, s):
    return {"maps": _ridge64(s["G"].double(), s["C"].double()), "info": None}


_EXACT = dict(build=_exact_build, centered=_exact_centered, probe=_exact_probe, attn=_exact_attn, apply=_exact_apply,
              k_stats=_exact_k_stats, k_solve=_exact_k_solve)


def exact(case, seed):
    """What run() returns for these inputs in 64 bits, by plain torch."""
    return _EXACT[case["kind"]](case, prepare(case, seed))
