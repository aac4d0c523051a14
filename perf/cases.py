"""What a program that uses this library has it do, as measurable cases.

A case names a kind of call (one MMDiT block, its MLP half, joint attention, a full denoise step,
a TeaCache step that reuses its residual, the sampler update with its log-density, the reward
statistics) and its sizes. `listed` holds the sizes that stand for real use; `draw` gives others of
the same ranges. Sizes follow the configurations of `seeded_inputs.py`: hidden 3072 with 24 heads of
128 at 512x512 (32x32 latent tokens, 256 text tokens) and 1280x1280 (80x80, 512), the small ragged
shapes and the fp32 model. Values are synthetic: weights and biases N(0, 0.02), activations,
conditioning and noise N(0, 1), rewards U(0, 1).
"""
from __future__ import annotations

import math
import zlib

import torch

from paper_2606_19004_amd import ditstep

DT = {"bf16": torch.bfloat16, "f32": torch.float32}
LATENT = 64            # 16 latent channels x 2x2 patch
T, T_NEXT = 0.62, 0.57
TEACACHE_T = 0.60      # the gated step's timestep, after a computed step at T
TEACACHE_BLOCKS = 2


def _model(kind, hidden, head_dim, grid, n_txt, batch, dtype="bf16", blocks=1, rope=True, noise=0.7):
    return {"kind": kind, "hidden": hidden, "head_dim": head_dim, "grid_h": grid[0], "grid_w": grid[1],
            "n_txt": n_txt, "batch": batch, "dtype": dtype, "blocks": blocks, "rope": rope, "noise": noise}


def listed():
    cases = {
        # rewards of 64 prompt groups of 16 seeds, top and bottom 4 kept: the end of every rollout, one
        # small call that lives on its launches
        "reward_64x16": {"kind": "reward", "groups": 64, "n": 16, "k": 4},
        # the sampler's SDE update of 16 latents of a 512x512 image and the log-density of the step
        # taken, as a policy-gradient rollout stores it
        "sampler_512_k16": {"kind": "sampler", "batch": 16, "n": 1024 * LATENT, "noise": 0.7},
        # the tiny fp32 model, one whole deterministic (Euler) step of two seeds: the smallest step, bound
        # by launches
        "step_tiny_f32": _model("step", 256, 64, (8, 8), 16, 2, "f32", noise=0.0),
        # one block of a small model in fp32, the type that reference runs and debugging use
        "block_f32_768": _model("block", 768, 64, (32, 32), 64, 2, "f32"),
        # a small ragged bf16 block (grid 11x13, 37 text tokens, heads of 64)
        "block_ragged_d64": _model("block", 320, 64, (11, 13), 37, 2),
        # one seed at 512x512: interactive use and the last seeds of a group, weights read for few rows
        "block_512_k1": _model("block", 3072, 128, (32, 32), 256, 1),
        # eight seeds of a group at 512x512
        "block_512_k8": _model("block", 3072, 128, (32, 32), 256, 8),
        # four seeds at 1280x1280, where attention over 6912 tokens weighs most
        "block_1280_k4": _model("block", 3072, 128, (80, 80), 512, 4),
        # a sequence-parallel rank's share at 1280x1280, eight seeds: the MLP half on its 1600 + 128
        # tokens ...
        "mlp_slice_1280_k8": _model("mlp", 3072, 128, (40, 40), 128, 8, rope=False),
        # ... and joint attention of its 6 heads over the whole sequence
        "attn_headslice_1280_k8": {"kind": "attn", "batch": 8, "heads": 6, "seq": 6912, "head_dim": 128,
                                   "dtype": "bf16"},
        # a step that TeaCache lets reuse the cached residual: half or more of the steps of a long
        # exploration run
        "teacache_skip_512_k16": _model("teacache", 3072, 128, (32, 32), 256, 16, blocks=TEACACHE_BLOCKS),
        # the headline workload: a whole denoise step of a 16-seed group through 8 blocks at 512x512, SDE
        "step_512_k16": _model("step", 3072, 128, (32, 32), 256, 16, blocks=8),
    }
    return [{"name": n, **c} for n, c in cases.items()]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case. Every kind but the smallest ones (reward, sampler) is drawn over its model sizes."""
    cap = max(work(c)["flops"] for c in listed())
    while True:
        kind = rng.choice(["reward", "sampler", "step", "block", "block", "block", "mlp", "attn", "teacache"])
        if kind == "reward":
            n = _log_int(rng, 2, 1024)
            return {"kind": kind, "groups": _log_int(rng, 1, 512), "n": n, "k": rng.randint(0, min(n, 64))}
        if kind == "sampler":
            return {"kind": kind, "batch": rng.randint(1, 32), "n": LATENT * _log_int(rng, 64, 6400),
                    "noise": rng.choice([0.3, 0.7, 1.0])}
        if kind == "attn":
            c = {"kind": kind, "batch": rng.randint(1, 8), "heads": rng.randint(1, 24),
                 "seq": _log_int(rng, 64, 6912), "head_dim": rng.choice([64, 128]),
                 "dtype": rng.choice(["bf16", "bf16", "f32"])}
            if c["dtype"] == "f32":
                c["seq"] = min(c["seq"], 1500)
        else:
            f32 = rng.random() < 0.25
            head_dim = rng.choice([64, 128, 128])
            hidden = head_dim * _log_int(rng, 2, (1024 if f32 else 3072) // head_dim)
            side = 40 if f32 else 80
            grid = (_log_int(rng, 6, side), _log_int(rng, 6, side))
            c = _model(kind, hidden, head_dim, grid, _log_int(rng, 13, 512), _log_int(rng, 1, 2 if f32 else 16),
                       "f32" if f32 else "bf16",
                       blocks=rng.randint(1, 4) if kind == "step" else TEACACHE_BLOCKS if kind == "teacache" else 1,
                       rope=kind != "mlp", noise=rng.choice([0.0, 0.7]))
            # the library's limit on one activation buffer
            rows = c["batch"] * (grid[0] * grid[1] + c["n_txt"])
            if rows * 4 * hidden * (4 if f32 else 2) >= 2 ** 31:
                continue
        if work(c)["flops"] < cap:
            return c


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
class _Draws:
    """Named seeded draws on the GPU; each tensor depends on its name and the seed alone."""

    def __init__(self, seed):
        self.seed = seed

    def _gen(self, name):
        return torch.Generator(device="cuda").manual_seed((self.seed * 1000003 + zlib.crc32(name.encode())) & 0x7FFFFFFF)

    def normal(self, name, shape, dtype=torch.float32, std=1.0):
        return torch.empty(shape, dtype=dtype, device="cuda").normal_(0.0, std, generator=self._gen(name))

    def uniform(self, name, shape):
        return torch.empty(shape, dtype=torch.float32, device="cuda").uniform_(0.0, 1.0, generator=self._gen(name))


def _shape(case):
    D, n_img = case["hidden"], case["grid_h"] * case["grid_w"]
    return D, 4 * D, n_img, case["n_txt"], case["batch"]


def _block_weights(case, dr, i):
    D, F, _, _, _ = _shape(case)
    shapes = {"mod": (6 * D, D), "qkv": (3 * D, D), "out": (D, D), "mlp1": (F, D), "mlp2": (D, F)}
    dt = DT[case["dtype"]]
    out = []
    for s in ("img", "txt"):
        w = {}
        for n, shp in shapes.items():
            w[n + "_w"] = dr.normal(f"b{i}.{s}.{n}_w", shp, dt, 0.02)
            w[n + "_b"] = dr.normal(f"b{i}.{s}.{n}_b", shp[:1], dt, 0.02)
        out.append(w)
    return out


def _step_weights(case, dr):
    D, dt = case["hidden"], DT[case["dtype"]]
    shapes = {"t1": (D, 256), "t2": (D, D), "in": (D, LATENT), "fmod": (2 * D, D), "fout": (LATENT, D)}
    w = {}
    for n, shp in shapes.items():
        w[n + "_w"] = dr.normal(n + "_w", shp, dt, 0.02)
        w[n + "_b"] = dr.normal(n + "_b", shp[:1], dt, 0.02)
    return w


def _activations(case, dr):
    D, _, n_img, n_txt, B = _shape(case)
    dt = DT[case["dtype"]]
    return {"temb": dr.normal("temb", (B, D)), "x_img": dr.normal("x_img", (B, n_img, D), dt),
            "x_txt": dr.normal("x_txt", (B, n_txt, D), dt)}


def _latents(case, dr):
    _, _, n_img, n_txt, B = _shape(case)
    return {"latent": dr.normal("latent", (B, n_img, LATENT)),
            "x_txt": dr.normal("x_txt", (B, n_txt, case["hidden"]), DT[case["dtype"]]),
            "noise": dr.normal("noise", (B, n_img, LATENT)) if case["noise"] > 0 else None}


def _config(case):
    D, F, n_img, n_txt, _ = _shape(case)
    return ditstep.block_config(D, D // case["head_dim"], case["head_dim"], F, n_img, n_txt, case["grid_h"],
                                case["grid_w"], rope=case["rope"], dtype=case["dtype"])


def prepare(case, seed):
    dr, kind = _Draws(seed), case["kind"]
    st = {"case": case}
    if kind == "reward":
        g, n, k = case["groups"], case["n"], case["k"]
        st["rewards"] = dr.uniform("rewards", (g, n))
        st["out"] = {"mean": torch.empty(g, device="cuda"), "std": torch.empty(g, device="cuda"),
                     "adv": torch.empty(g, n, device="cuda"),
                     "order": torch.empty(g, n, dtype=torch.int32, device="cuda"),
                     "selected": torch.empty(g, k, dtype=torch.int32, device="cuda")}
        st["status"] = torch.empty(1, dtype=torch.int32, device="cuda")
        return st
    if kind == "sampler":
        shp = (case["batch"], case["n"])
        st["x_prev"], st["v"], st["noise"] = dr.normal("x", shp), dr.normal("v", shp), dr.normal("noise", shp)
        st["x"] = st["x_prev"].clone()   # the trajectory keeps the latent before the step
        st["logp"] = torch.empty(case["batch"], dtype=torch.float64, device="cuda")
        return st
    if kind == "attn":
        B, H, S, d = case["batch"], case["heads"], case["seq"], case["head_dim"]
        st["qkv"] = dr.normal("qkv", (B, S, 3, H, d), DT[case["dtype"]])   # the packed layout of a QKV projection
        st["o"] = torch.empty(B, S, H, d, dtype=DT[case["dtype"]], device="cuda")
        return st
    cfg = _config(case)
    st["cfg"], B = cfg, case["batch"]
    if kind in ("block", "mlp"):
        st.update(_activations(case, dr))
        st["w"] = ditstep.block_weights(*_block_weights(case, dr, 0))
        st["ws"] = ditstep.workspace(ditstep.dit_block_workspace_bytes(cfg, B))
        return st
    st.update(_latents(case, dr))
    st["sw"] = ditstep.step_weights(_step_weights(case, dr))
    st["blocks"] = [ditstep.block_weights(*_block_weights(case, dr, i)) for i in range(case["blocks"])]
    st["v"] = torch.empty_like(st["latent"])
    st["ws"] = ditstep.workspace(ditstep.dit_denoise_workspace_bytes(cfg, B, LATENT))
    if kind == "teacache":
        # a run in progress: the first step has computed the blocks and filled the cache
        st["cache"] = ditstep.workspace(ditstep.dit_teacache_cache_bytes(cfg, B))
        st["state"] = ditstep.teacache_state(1e30)
        ditstep.dit_denoise_step_teacache(cfg, st["sw"], st["blocks"], T, TEACACHE_T, case["noise"], st["latent"],
                                          st["x_txt"], st["noise"], st["v"], st["state"], st["cache"], st["ws"])
    return st


def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "reward":
        ditstep.group_reward_stats_async(st["rewards"], st["status"], k_select=case["k"], **st["out"])
        return {**st["out"], "status": st["status"]}
    if kind == "sampler":
        ditstep.flow_step(st["x"], st["v"], st["noise"], T, T_NEXT, case["noise"])
        ditstep.flow_logprob(st["x_prev"], st["v"], st["x"], T, T_NEXT, case["noise"], st["logp"])
        return {"x": st["x"], "logp": st["logp"]}
    if kind == "attn":
        B, H, S, d = case["batch"], case["heads"], case["seq"], case["head_dim"]
        qkv = st["qkv"]
        ditstep.joint_attention(qkv[:, :, 0], qkv[:, :, 1], qkv[:, :, 2], st["o"], B, H, S, d,
                                (S * 3 * H * d, 3 * H * d, d), (S * H * d, H * d, d), dtype=case["dtype"])
        return st["o"]
    if kind == "block":
        ditstep.dit_block_forward(st["cfg"], st["w"], st["temb"], st["x_img"], st["x_txt"], st["ws"])
        return {"x_img": st["x_img"], "x_txt": st["x_txt"]}
    if kind == "mlp":
        ditstep.dit_block_mlp(st["cfg"], st["w"], st["temb"], st["x_img"], st["x_txt"], st["ws"])
        return {"x_img": st["x_img"], "x_txt": st["x_txt"]}
    if kind == "step":
        ditstep.dit_denoise_step(st["cfg"], st["sw"], st["blocks"], T, T_NEXT, case["noise"], st["latent"],
                                 st["x_txt"], st["noise"], st["v"], st["ws"])
        return {"latent": st["latent"], "v": st["v"]}
    ran, rel = ditstep.dit_denoise_step_teacache(st["cfg"], st["sw"], st["blocks"], TEACACHE_T, T_NEXT, case["noise"],
                                                 st["latent"], st["x_txt"], st["noise"], st["v"], st["state"],
                                                 st["cache"], st["ws"])
    return {"latent": st["latent"], "v": st["v"], "ran": int(ran), "rel": rel}


# ---------------------------------------------------------------------------
# necessary work
# ---------------------------------------------------------------------------
def work(case):
    kind = case["kind"]
    if kind == "reward":
        g, n, k = case["groups"], case["n"], case["k"]
        return {"bytes": 4 * g * (3 * n + k + 2), "flops": g * n * (6 + 2 * max(1, math.ceil(math.log2(n))))}
    if kind == "sampler":
        # flow_step reads x, v, noise and writes x; the log-density reads the earlier latent besides
        return {"bytes": 20 * case["batch"] * case["n"], "flops": 15 * case["batch"] * case["n"]}
    es = 2 if case["dtype"] == "bf16" else 4
    if kind == "attn":
        e = case["batch"] * case["heads"] * case["seq"] * case["head_dim"]
        return {"bytes": 4 * e * es, "flops": 4 * e * case["seq"]}
    D, F, n_img, n_txt, B = _shape(case)
    m, S = B * (n_img + n_txt), n_img + n_txt
    mod_w, half_w = 12 * D * D, 4 * D * F            # elements of both streams
    attn_w = 8 * D * D
    mlp = {"bytes": es * (mod_w + half_w + 2 * m * D), "flops": 4 * m * D * F + 2 * B * mod_w}
    block = {"bytes": mlp["bytes"] + es * attn_w, "flops": mlp["flops"] + 8 * m * D * D + 4 * B * S * S * D}
    if kind == "mlp":
        return mlp
    if kind == "block":
        return block
    lat = B * n_img * LATENT
    ends_w = D * (256 + D + LATENT + 2 * D + LATENT)
    ends = {"bytes": es * (ends_w + B * n_txt * D) + 4 * lat * (4 if case["noise"] > 0 else 3),
            "flops": 4 * lat * D + 2 * B * ends_w}
    if kind == "step":
        return {"bytes": ends["bytes"] + case["blocks"] * es * (mod_w + attn_w + half_w),
                "flops": ends["flops"] + case["blocks"] * block["flops"]}
    # a reused residual: the image stream's modulation of block 0, h_prev read and written, the fp32 residual read
    a = B * n_img * D
    return {"bytes": ends["bytes"] - es * B * n_txt * D + es * (2 * D * D + 2 * a) + 4 * a,
            "flops": ends["flops"] + 4 * B * D * D + 30 * a}


def tolerance(case):
    """About four times the distance from 64 bits that the present kernels show: sums of 32-bit values
    2e-7 (a whole fp32 model 4e-7 after one block, more after four), one bf16 rounding of the output and
    those inside attention 2.3e-3, a bf16 block 3.3e-3, a step through eight bf16 blocks 7.5e-3."""
    kind = case["kind"]
    if kind in ("reward", "sampler"):
        return {"rel": 1e-6}
    if case["dtype"] == "f32":
        return {"rel": 5e-6 if kind in ("step", "teacache") else 2e-6}
    return {"rel": {"attn": 1e-2, "block": 1.3e-2, "mlp": 1.3e-2}.get(kind, 3e-2)}


# ---------------------------------------------------------------------------
# the same outputs in 64 bits
# ---------------------------------------------------------------------------
def _f64(t):
    return t.to(torch.float64)


def _linear(x, w, b):
    """x W^T + b in 64 bits, rows in pieces so that no temporary outgrows the card."""
    w64, b64 = _f64(w), _f64(b)
    rows = x.reshape(-1, x.shape[-1])
    out = torch.cat([r @ w64.t() + b64 for r in rows.split(8192)])
    return out.reshape(*x.shape[:-1], w.shape[0])


def _silu(x):
    return x / (1.0 + torch.exp(-x))


def _ln(x, shift, scale, eps=1e-6):
    mu = x.mean(-1, keepdim=True)
    xc = x - mu
    var = (xc * xc).mean(-1, keepdim=True)
    return xc / torch.sqrt(var + eps) * (1.0 + scale) + shift


def _gelu(z):
    return 0.5 * z * (1.0 + torch.tanh(math.sqrt(2.0 / math.pi) * (z + 0.044715 * z ** 3)))


def _rope(x, case):
    """x [B][N_i][H][d]: head dims [0, d/2) rotate by the grid row, [d/2, d) by the column, pairs (2i, 2i+1)."""
    d, gh, gw = case["head_dim"], case["grid_h"], case["grid_w"]
    m = d // 2
    freq = 1e4 ** (-torch.arange(0, m, 2, dtype=torch.float64, device="cuda") / m)
    tok = torch.arange(gh * gw, device="cuda")
    ang = torch.cat([(tok // gw)[:, None] * freq, (tok % gw)[:, None] * freq], 1)[None, :, None, :]
    a, b = x[..., 0::2], x[..., 1::2]
    out = torch.empty_like(x)
    out[..., 0::2] = a * torch.cos(ang) - b * torch.sin(ang)
    out[..., 1::2] = a * torch.sin(ang) + b * torch.cos(ang)
    return out


def _attention(q, k, v):
    """[B][S][H][d] in 64 bits, one (sample, head) and at most 4096 queries at a time."""
    B, S, H, d = q.shape
    o = torch.empty_like(q)
    for b in range(B):
        for h in range(H):
            kt, vv = k[b, :, h].t().contiguous(), v[b, :, h].contiguous()
            for i in range(0, S, 4096):
                p = torch.softmax(q[b, i:i + 4096, h].contiguous() @ kt / math.sqrt(d), dim=-1)
                o[b, i:i + 4096, h] = p @ vv
    return o


def _mlp64(x, mod, w):
    D = x.shape[-1]
    h = _ln(x, mod[..., 3 * D:4 * D], mod[..., 4 * D:5 * D])
    out = []
    for xr, hr, g in zip(x, h, mod[..., 5 * D:]):   # one sample at a time
        out.append(xr + g * _linear(_gelu(_linear(hr, w["mlp1_w"], w["mlp1_b"])), w["mlp2_w"], w["mlp2_b"]))
    return torch.stack(out)


def _block64(case, ws, temb, x_img, x_txt, mlp_only=False):
    x = [x_img, x_txt]
    D, H, d = case["hidden"], case["hidden"] // case["head_dim"], case["head_dim"]
    mods = [_linear(_silu(temb), w["mod_w"], w["mod_b"])[:, None, :] for w in ws]
    if not mlp_only:
        qkv = []
        for s in range(2):
            h = _ln(x[s], mods[s][..., :D], mods[s][..., D:2 * D])
            y = _linear(h, ws[s]["qkv_w"], ws[s]["qkv_b"]).reshape(*x[s].shape[:2], 3, H, d)
            q, k, v = y[:, :, 0], y[:, :, 1], y[:, :, 2]
            if s == 0 and case["rope"]:
                q, k = _rope(q, case), _rope(k, case)
            qkv.append((q, k, v))
        q, k, v = (torch.cat([t, i], 1) for i, t in zip(*qkv))   # text tokens first
        o = _attention(q, k, v)
        n_txt = x_txt.shape[1]
        for s, os in enumerate((o[:, n_txt:], o[:, :n_txt])):
            x[s] = x[s] + mods[s][..., 2 * D:3 * D] * _linear(os.reshape(x[s].shape), ws[s]["out_w"], ws[s]["out_b"])
    return tuple(_mlp64(x[s], mods[s], ws[s]) for s in range(2))


def _f32(x):
    return float(torch.tensor(x, dtype=torch.float32))


def _flow64(x, v, noise, t, t_next, a):
    t, t_next, a = _f32(t), _f32(t_next), _f32(a)
    h = t_next - t
    if a == 0.0:
        return x + h * v
    sigma = a * math.sqrt(t / (1.0 - t))
    return x + h * (v + sigma ** 2 / (2 * t) * (x + (1 - t) * v)) + sigma * math.sqrt(-h) * noise


def _temb64(t, sw, B):
    f = 1e4 ** (-torch.arange(128, dtype=torch.float64, device="cuda") / 128)
    e = torch.cat([torch.cos(1000 * _f32(t) * f), torch.sin(1000 * _f32(t) * f)]).expand(B, 256)
    return _linear(_silu(_linear(e, sw["t1_w"], sw["t1_b"])), sw["t2_w"], sw["t2_b"])


def _final64(x, temb, sw):
    D = x.shape[-1]
    m = _linear(_silu(temb), sw["fmod_w"], sw["fmod_b"])[:, None, :]
    return _linear(_ln(x, m[..., :D], m[..., D:]), sw["fout_w"], sw["fout_b"])


def _step64(case, dr, sw, lat, x_txt, noise, t, t_next):
    """(latent', v, residual of the block stack)"""
    temb = _temb64(t, sw, case["batch"])
    x_in = _linear(lat, sw["in_w"], sw["in_b"])
    x, xt = x_in, x_txt
    for i in range(case["blocks"]):
        ws = _block_weights(case, dr, i)
        x, xt = _block64(case, ws, temb, x, xt)
    v = _final64(x, temb, sw)
    return _flow64(lat, v, noise, t, t_next, case["noise"]), v, x - x_in


def exact(case, seed):
    dr, kind = _Draws(seed), case["kind"]
    if kind == "reward":
        r = _f64(dr.uniform("rewards", (case["groups"], case["n"])))
        n, k = case["n"], case["k"]
        mu = r.mean(1, keepdim=True)
        sd = torch.sqrt(((r - mu) ** 2).mean(1, keepdim=True))
        adv = torch.where(sd > 0, (r - mu) / (sd + _f32(1e-4)), torch.zeros_like(r))
        order = torch.sort(r, dim=1, descending=True, stable=True).indices.to(torch.int32)
        sel = torch.cat([order[:, :(k + 1) // 2], order[:, n - k // 2:]], 1)
        return {"mean": mu[:, 0], "std": sd[:, 0], "adv": adv, "order": order, "selected": sel,
                "status": torch.zeros(1, dtype=torch.int32, device="cuda")}
    if kind == "sampler":
        shp = (case["batch"], case["n"])
        x, v, e = (_f64(dr.normal(n, shp)) for n in ("x", "v", "noise"))
        xn = _flow64(x, v, e, T, T_NEXT, case["noise"])
        t, h, a = _f32(T), _f32(T_NEXT) - _f32(T), _f32(case["noise"])
        var = a * a * t / (1 - t) * -h
        r = xn - _flow64(x, v, 0.0, T, T_NEXT, case["noise"])
        return {"x": xn, "logp": -(r * r).sum(1) / (2 * var) - 0.5 * case["n"] * math.log(2 * math.pi * var)}
    if kind == "attn":
        B, H, S, d = case["batch"], case["heads"], case["seq"], case["head_dim"]
        qkv = dr.normal("qkv", (B, S, 3, H, d), DT[case["dtype"]])
        return _attention(*(_f64(qkv[:, :, i]) for i in range(3)))
    if kind in ("block", "mlp"):
        a = _activations(case, dr)
        xi, xt = _block64(case, _block_weights(case, dr, 0), _f64(a["temb"]), _f64(a["x_img"]), _f64(a["x_txt"]),
                          mlp_only=kind == "mlp")
        return {"x_img": xi, "x_txt": xt}
    sw, lt = _step_weights(case, dr), _latents(case, dr)
    lat, x_txt = _f64(lt["latent"]), _f64(lt["x_txt"])
    noise = _f64(lt["noise"]) if lt["noise"] is not None else 0.0
    if kind == "step":
        lat, v, _ = _step64(case, dr, sw, lat, x_txt, noise, T, T_NEXT)
        return {"latent": lat, "v": v}
    # the computed step of `prepare`, then the step that reuses its residual
    D, B = case["hidden"], case["batch"]
    w0 = _block_weights(case, dr, 0)[0]

    def modulated(latent, t):
        m = _linear(_silu(_temb64(t, sw, B)), w0["mod_w"], w0["mod_b"])[:, None, :]
        return _ln(_linear(latent, sw["in_w"], sw["in_b"]), m[..., :D], m[..., D:2 * D])

    h_prev = modulated(lat, T)
    lat, _, residual = _step64(case, dr, sw, lat, x_txt, noise, T, TEACACHE_T)
    rel = float((modulated(lat, TEACACHE_T) - h_prev).abs().sum() / h_prev.abs().sum())
    v = _final64(_linear(lat, sw["in_w"], sw["in_b"]) + residual, _temb64(TEACACHE_T, sw, B), sw)
    return {"latent": _flow64(lat, v, noise, TEACACHE_T, T_NEXT, case["noise"]), "v": v, "ran": 0, "rel": rel}
