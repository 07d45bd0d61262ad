"""The work this library is used for, as a list of measurable cases.

A user of the library holds Q, K, V of one global-attention layer on the GPU, a plan of the scene's
geometry and a workspace, and calls layer_forward once per layer and scene; or calls the stages one by
one where it wants the intermediate tensors; or calls the attention over ragged per-head sequences on
its own.  Scenes go from two small frames (where launches and latency count) to 200 frames of 37 x 37
patches.  The method has no backward pass: it accelerates inference.

Inputs are seeded tensors with the shape and the structure of the activations the method is made for
(neighbouring patches and consecutive frames are similar), by the recipe of synth/vggt_tokens.py, drawn
on the GPU so that they are quick to make: a smooth field per scene, shifted by a few patches and
perturbed per frame, five special tokens, one random projection to Q, K and V, one rounding to bf16.
"""
import math
import random

import torch

import paper_2511_21317_amd as httm

D_MODEL = 1024
D_HEAD = 64

# What a case of kind "layer" or "stages" may leave out.
_DEFAULTS = {"n_special": 5, "H": 16, "variant": "headwise", "anchor": False, "chunked": False,
             "outlier_frac": 0.0, "dst_frac": 0.0, "log2_keys": True, "max_shift": 1}


def listed():
    return [
        # two small frames: the smallest scene, a call of a few launches (latency)
        _layer("layer_2_frames", S=2, Hp=16, Wp=16, b=4, T=2, rho_q=0.5, rho_kv=0.5),
        # a handful of full-size frames: an interactive reconstruction
        _layer("layer_8_frames", S=8, Hp=37, Wp=37, b=4, T=2, rho_q=0.5, rho_kv=0.5),
        # a short clip with a 16:9-like grid
        _layer("layer_32_frames", S=32, Hp=21, Wp=37, b=4, T=4, rho_q=0.75, rho_kv=0.75),
        # a long clip in small blocks (64 tokens)
        _layer("layer_100_frames", S=100, Hp=37, Wp=37, b=4, T=4, rho_q=0.8, rho_kv=0.8, max_shift=2),
        # the longest clip, in 256-token blocks with nine tenths merged
        _layer("layer_200_frames", S=200, Hp=37, Wp=37, b=8, T=4, rho_q=0.9, rho_kv=0.9),
        # the same clip with a tenth of the queries kept out of the merging as outliers
        _layer("layer_200_frames_outliers", S=200, Hp=37, Wp=37, b=8, T=4, rho_q=0.9, rho_kv=0.9, outlier_frac=0.1),
        # the paper's own configuration: runs of 128 tokens x 30 frames, 90 % / 70 %, outliers kept
        _layer("layer_200_frames_paper", S=200, Hp=37, Wp=37, b=128, T=30, rho_q=0.9, rho_kv=0.7, chunked=True,
               outlier_frac=0.1),
        # nothing divides anything: ragged windows in space and time, different ratios for Q and K / V,
        # anchored first frame, keys without the logit scale (the kernel with per-row shifts)
        _layer("layer_odd_plain_keys", S=37, Hp=19, Wp=27, b=5, T=3, rho_q=0.6, rho_kv=0.35, anchor=True,
               log2_keys=False, n_special=4),
        # the unmerged layer: the same attention over all tokens, what the merged one is compared with
        _layer("layer_8_frames_unmerged", S=8, Hp=37, Wp=37, b=4, T=2, rho_q=0.0, rho_kv=0.0, variant="none"),
        # the general src / dst rule of the method (25 % dst tokens, the most similar src tokens merge)
        _layer("layer_32_frames_top_r", S=32, Hp=37, Wp=37, b=8, T=4, rho_q=0.6, rho_kv=0.6, dst_frac=0.25),
        # the stages one by one, with every intermediate tensor and the similarities in the caller's hands
        _layer("stages_48_frames", kind="stages", S=48, Hp=28, Wp=37, b=7, T=5, rho_q=0.8, rho_kv=0.7),
        # attention alone over sequences of another length for every head, queries and keys apart
        {"name": "attention_ragged", "kind": "attention", "H": 16, "m_q": 5500, "m_k": 9000, "spread": 0.5,
         "log2_keys": False},
    ]


def _layer(name, kind="layer", **kw):
    case = {"name": name, "kind": kind}
    case.update(_DEFAULTS)
    case.update(kw)
    return case


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng: random.Random):
    """One more case of the same ranges: 2 to 200 frames of 16 x 16 to 37 x 37 patches in blocks of 16 to
    3840 tokens, 35 % to 90 % merged, with the options in the shares in which the list has them."""
    while True:
        pick = rng.random()
        if pick < 0.15:
            c = {"kind": "attention", "H": rng.choice([8, 12, 16]), "m_q": _log_uniform(rng, 250, 12000),
                 "m_k": _log_uniform(rng, 250, 12000), "spread": rng.choice([0.0, 0.3, 0.5]),
                 "log2_keys": rng.random() < 0.6}
        else:
            c = dict(_DEFAULTS)
            c["kind"] = "stages" if pick < 0.25 else "layer"
            c["S"] = _log_uniform(rng, 2, 200)
            c["Hp"], c["Wp"] = rng.randint(16, 37), rng.randint(16, 37)
            c["n_special"] = rng.choice([5, 5, 5, 4, 1])
            c["H"] = rng.choice([16, 16, 16, 8, 12])
            c["max_shift"] = rng.choice([1, 2])
            c["log2_keys"] = rng.random() < 0.8
            c["rho_q"] = round(rng.uniform(0.5, 0.9), 2)
            c["rho_kv"] = c["rho_q"] if rng.random() < 0.5 else round(rng.uniform(0.35, 0.9), 2)
            option = rng.random()
            if option < 0.2 and c["kind"] == "layer":
                c["outlier_frac"] = round(rng.uniform(0.03, 0.12), 2)
            elif option < 0.35:
                c["anchor"] = True
            elif option < 0.45:
                c["dst_frac"] = 0.25
            elif option < 0.5 and c["kind"] == "layer":
                c["variant"] = "none"
                c["rho_q"] = c["rho_kv"] = 0.0
            shape = rng.random()
            if shape < 0.25:
                c["chunked"], c["b"], c["T"] = True, rng.choice([64, 100, 128]), rng.choice([12, 20, 30])
            elif shape < 0.6:
                c["b"], c["T"] = 4, rng.choice([1, 2, 3, 4])
            else:
                c["b"], c["T"] = rng.choice([5, 6, 7, 8]), rng.choice([2, 3, 4, 5, 6])
        if work(c)["flops"] <= 1.0e13:      # below the largest listed case (1.9e13)
            return c


def _geom(case):
    return httm.make_geom(case["S"], case["Hp"], case["Wp"], case["b"], case["T"], case["rho_q"], case["rho_kv"],
                          H=case["H"], n_special=case["n_special"], variant=case["variant"],
                          anchor_first_frame=case["anchor"], outlier_frac=case["outlier_frac"],
                          chunked_blocks=case["chunked"], dst_frac=case["dst_frac"], log2_keys=case["log2_keys"])


# ---- inputs ------------------------------------------------------------------------------------------

def _circular_blur(n, sigma, device):
    """[n, n] matrix of a Gaussian filter that wraps around, cut off at four sigma."""
    radius = int(4 * sigma + 0.5)
    m = torch.zeros((n, n), dtype=torch.float64)
    rows = torch.arange(n)
    for d in range(-radius, radius + 1):
        m[rows, (rows + d) % n] += math.exp(-0.5 * (d / sigma) ** 2)
    return (m / m.sum(dim=1, keepdim=True)).to(device=device, dtype=torch.float32)


def _tokens(S, Hp, Wp, n_special, H, max_shift, seed):
    """q, k, v [H, N, 64] bf16 in the caller's token order (see the top of this file)."""
    dev = torch.device("cuda")
    rng = random.Random(seed)
    gen = torch.Generator(device=dev)
    gen.manual_seed(rng.getrandbits(62))
    field = torch.randn((Hp, Wp * D_MODEL), generator=gen, device=dev)
    field = (_circular_blur(Hp, 2.0, dev) @ field).view(Hp, Wp, D_MODEL)
    field = field.transpose(0, 1).reshape(Wp, Hp * D_MODEL)
    field = (_circular_blur(Wp, 2.0, dev) @ field).view(Wp, Hp, D_MODEL).transpose(0, 1).contiguous()
    field = field / field.reshape(-1, D_MODEL).std(dim=0)
    special = torch.randn((n_special, D_MODEL), generator=gen, device=dev)
    weight = torch.randn((D_MODEL, 3 * H * D_HEAD), generator=gen, device=dev) / math.sqrt(D_MODEL)
    tpf = n_special + Hp * Wp
    out = torch.empty((3, H, S * tpf, D_HEAD), dtype=torch.bfloat16, device=dev)
    for f in range(S):
        shift = (rng.randint(-max_shift, max_shift), rng.randint(-max_shift, max_shift))
        x = torch.cat([special, torch.roll(field, shift, dims=(0, 1)).view(Hp * Wp, D_MODEL)])
        x += 0.1 * torch.randn(x.shape, generator=gen, device=dev)
        out[:, :, f * tpf:(f + 1) * tpf] = (x @ weight).view(tpf, 3, H, D_HEAD).permute(1, 2, 0, 3)
    return out[0], out[1], out[2]


def _head_lengths(m, H, spread):
    """Lengths around m, from m * (1 - spread / 2) for the first head to m * (1 + spread / 2) for the last."""
    return [max(1, round(m * (1.0 + spread * (h / max(1, H - 1) - 0.5)))) for h in range(H)]


def _offsets(lengths):
    off = [0]
    for n in lengths:
        off.append(off[-1] + n)
    return off


def prepare(case, seed):
    H = case["H"]
    if case["kind"] == "attention":
        # merged tokens of a scene, packed with another length for every head
        len_q = _head_lengths(case["m_q"], H, case["spread"])
        len_k = _head_lengths(case["m_k"], H, -case["spread"])
        frames = -(-max(len_q + len_k) // (20 * 20 + 5))
        q, k, v = _tokens(frames, 20, 20, 5, H, 1, seed)
        q = torch.cat([q[h, :n] for h, n in enumerate(len_q)])
        k, v = (torch.cat([t[h, :n] for h, n in enumerate(len_k)]) for t in (k, v))
        if case["log2_keys"]:
            k = (k.float() * httm.LOG2_KEY_SCALE).to(torch.bfloat16)
        return {"case": case, "q": q, "k": k, "v": v, "o": torch.empty_like(q), "q_off": _offsets(len_q),
                "k_off": _offsets(len_k),
                "scratch": torch.empty(httm.attention_scratch_bytes(H), dtype=torch.uint8, device="cuda")}
    q, k, v = _tokens(case["S"], case["Hp"], case["Wp"], case["n_special"], H, case["max_shift"], seed)
    plan = httm.Plan(_geom(case))
    out = torch.empty((plan.N, H * D_HEAD), dtype=torch.bfloat16, device="cuda")
    st = {"case": case, "q": q, "k": k, "v": v, "plan": plan, "out": out}
    if case["kind"] == "layer":
        st["workspace"] = httm.alloc_workspace(plan)
        return st
    bf, dev = torch.bfloat16, "cuda"
    st["q_m"] = torch.empty((H, plan.M_q, D_HEAD), dtype=bf, device=dev)
    st["o_m"] = torch.empty_like(st["q_m"])
    st["k_m"] = torch.empty((H, plan.M_k, D_HEAD), dtype=bf, device=dev)
    st["v_m"] = torch.empty_like(st["k_m"])
    for name, dtype in (("assign_q", torch.int32), ("assign_k", torch.int32), ("score_q", torch.float32),
                        ("score_k", torch.float32)):
        st[name] = torch.empty((H, plan.N), dtype=dtype, device=dev)
    for name in ("q_r", "k_r", "v_r", "o_r", "o_hn"):
        st[name] = torch.empty_like(q)
    st["q_off"] = [h * plan.M_q for h in range(H + 1)]
    st["k_off"] = [h * plan.M_k for h in range(H + 1)]
    return st


# ---- one pass ------------------------------------------------------------------------------------------

def run(state):
    st, case = state, state["case"]
    if case["kind"] == "layer":
        return httm.layer_forward(st["plan"], st["q"], st["k"], st["v"], st["out"], st["workspace"])
    if case["kind"] == "attention":
        if case["log2_keys"]:
            return httm.attention_log2(st["q"], st["k"], st["v"], st["o"], st["q_off"], st["k_off"],
                                       scratch=st["scratch"])
        return httm.attention(st["q"], st["k"], st["v"], st["o"], st["q_off"], st["k_off"], 0.125,
                              scratch=st["scratch"])
    # the stages: reorder, match and merge, attention (without scratch memory), unmerge, inverse reorder
    plan = st["plan"]
    for a, b in (("q", "q_r"), ("k", "k_r"), ("v", "v_r")):
        httm.reorder(plan, st[a], st[b], 0)
    httm.match_merge(plan, st["q_r"], st["k_r"], st["v_r"], st["q_m"], st["k_m"], st["v_m"], st["assign_q"],
                     st["assign_k"], st["score_q"], st["score_k"])
    if case["log2_keys"]:
        httm.attention_log2(st["q_m"], st["k_m"], st["v_m"], st["o_m"], st["q_off"], st["k_off"])
    else:
        httm.attention(st["q_m"], st["k_m"], st["v_m"], st["o_m"], st["q_off"], st["k_off"])
    httm.unmerge(plan, st["o_m"], st["assign_q"], st["o_r"], fuse_inverse_reorder=False)
    httm.reorder(plan, st["o_r"], st["o_hn"], 1)
    return {n: st[n] for n in ("q_r", "k_r", "v_r", "q_m", "k_m", "v_m", "assign_q", "assign_k", "score_q", "score_k",
                               "o_m", "o_r", "o_hn")}


# ---- what a pass cannot do without -----------------------------------------------------------------------

def work(case):
    row, H = D_HEAD * 2, case["H"]
    if case["kind"] == "attention":
        len_q = _head_lengths(case["m_q"], H, case["spread"])
        len_k = _head_lengths(case["m_k"], H, -case["spread"])
        return {"bytes": 2 * row * (sum(len_q) + sum(len_k)),
                "flops": 4 * D_HEAD * sum(a * b for a, b in zip(len_q, len_k))}
    g = _geom(case)
    s = httm.geom_sizes(g)
    N, M_q, M_k = int(s.N), int(s.M_q), int(s.M_k)
    nbytes = 4 * H * N * row                                    # q, k, v in, the output out
    if case["kind"] == "stages":
        # reordered copies in and out, merged tensors, assignments and similarities, two more copies of the output
        nbytes = H * (N * row * (6 + 3 + 1 + 2) + row * 2 * (2 * M_q + 2 * M_k) + N * 4 * 5)
    flops = 4 * H * (M_q * M_k + int(s.outlier_cap) // H * M_k) * D_HEAD
    if case["variant"] == "headwise":
        t = httm.geom_tables(g)
        n = t["block_n"].astype("int64")
        for k in (t["block_kq"].astype("int64"), t["block_kk"].astype("int64")):
            dst = (n * case["dst_frac"]).astype("int64") if case["dst_frac"] > 0 else k
            flops += int(2 * H * D_HEAD * (dst * (n - dst)).sum())   # every src token against every dst token
    return {"bytes": int(nbytes), "flops": int(flops)}


def tolerance(case):
    """Outputs in bf16 through two products with bf16 operands: 1.7e-3 to 2.1e-3 of the norm against the
    same path with means, products and softmax in 64 bits.  Whole numbers are cluster indices, of which
    those may differ whose two best similarities agree to the precision in which they are compared:
    3e-6 of them against sums in another order, 2.4e-4 in blocks of more than 512 tokens, whose
    similarities are compared in 19 bits."""
    if case["kind"] == "stages":
        big = case["T"] * (case["b"] if case["chunked"] else case["b"] ** 2) > 512
        return {"rel": 8e-3, "differ": 1e-3 if big else 2e-5}
    return {"rel": 8e-3}
