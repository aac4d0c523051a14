"""The velocity head, in one pass and as LayerNorm and a GEMM, and the fused TeaCache distance at the edges of their
row and k splits.

Head: the 8 waves of the one pass share a row's 32-deep k steps, so widths run from one step per two waves (64) to
the largest (4096, with a residual), with equal and unequal shares; rows of one and several 16-row tiles, the last
partial, tiles that span samples; weights at the 8-byte alignment that is enough elsewhere. The reference is
float64 from the same bf16 inputs; h is rounded to bf16 once (2^-9 per element, random), which over a
sum of products stays below 2^-8 of the output's size: 1e-2 of max|v|.

Distance: two steps far apart in t, so that |h - h_prev| is of h's size; the roundings of h to bf16
(relative 2^-9 each) then move the ratio by less than 2 * 2^-9 / 0.3 = 1.3e-2."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def d():
    from paper_2606_19004_amd import ditstep
    return ditstep


def weights(hidden, latent, dtype, g, skew=0):
    shapes = {"t1": (hidden, 256), "t2": (hidden, hidden), "in": (hidden, latent), "fmod": (2 * hidden, hidden),
              "fout": (latent, hidden)}
    w = {}
    for n, shp in shapes.items():
        for s, full in (("_w", shp), ("_b", shp[:1])):
            flat = torch.randn(int(np.prod(full)) + skew, generator=g, device="cuda") * 0.02
            w[n + s] = flat.to(dtype)[skew:].view(full)
    return w


def ln(x, shift, scale):
    xc = x - x.mean(-1, keepdim=True)
    return xc / torch.sqrt((xc * xc).mean(-1, keepdim=True) + 1e-6) * (1 + scale) + shift


def lin(x, w, b):
    return x @ w.double().t() + b.double()


@pytest.mark.parametrize("hidden,latent,b,n,skew", [(64, 64, 1, 1, 0), (128, 64, 3, 5, 4), (320, 128, 2, 17, 0),
                                                    (512, 64, 1, 16, 0), (1088, 64, 2, 33, 4), (2176, 64, 1, 31, 0),
                                                    (3072, 64, 2, 40, 4), (4096, 64, 1, 18, 0), (4032, 64, 1, 7, 0)])
def test_final_head(d, hidden, latent, b, n, skew):
    g = torch.Generator(device="cuda").manual_seed(hidden + n)
    c = d.block_config(hidden, hidden // 64, 64, 4 * hidden, n, 0, 1, n)
    sw = weights(hidden, latent, torch.bfloat16, g, skew)
    x = torch.randn(b, n, hidden, generator=g, device="cuda").to(torch.bfloat16)
    temb = torch.randn(b, hidden, generator=g, device="cuda")
    v = torch.full((b, n, latent), 7.0, device="cuda")
    d.dit_final_layer(c, d.step_weights(sw), temb, x, v, d.workspace(d.dit_denoise_workspace_bytes(c, b, latent)))
    t64 = temb.double()
    m = lin(t64 / (1 + torch.exp(-t64)), sw["fmod_w"], sw["fmod_b"])[:, None]
    want = lin(ln(x.double(), m[..., :hidden], m[..., hidden:]), sw["fout_w"], sw["fout_b"])
    assert (v.double() - want).abs().max() <= 1e-2 * want.abs().max()


# both sides of the choice between one pass and two kernels: width, workgroups, output features, tiles that span samples
@pytest.mark.parametrize("hidden,latent,b,n,one_pass", [(320, 128, 2, 48, True), (512, 64, 3, 32, True), (1024, 64, 2, 40, True),
                                                        (1088, 64, 4, 416, True), (1792, 64, 4, 401, True), (1024, 192, 1, 700, True),
                                                        (1088, 64, 2, 32, False), (1856, 64, 4, 416, False), (3072, 64, 2, 32, False),
                                                        (4096, 64, 2, 48, False), (1024, 1024, 2, 333, False),
                                                        (256, 512, 3, 2000, False), (64, 1024, 4, 1000, False),
                                                        (1024, 64, 16, 1024, True), (1024, 64, 16, 1023, False)])
def test_final_head_choice(d, hidden, latent, b, n, one_pass):
    g = torch.Generator(device="cuda").manual_seed(hidden + n)
    c = d.block_config(hidden, hidden // 64, 64, 4 * hidden, n, 0, 1, n)
    sw = weights(hidden, latent, torch.bfloat16, g)
    x = torch.randn(b, n, hidden, generator=g, device="cuda").to(torch.bfloat16)
    temb = torch.randn(b, hidden, generator=g, device="cuda")
    v = torch.full((b, n, latent), 7.0, device="cuda")
    x0 = x.clone()
    d.dit_profile_begin()
    d.dit_final_layer(c, d.step_weights(sw), temb, x, v, d.workspace(d.dit_denoise_workspace_bytes(c, b, latent)))
    assert {s["name"] for s in d.dit_profile_end()} == {"final_gemv"} | ({"final_head"} if one_pass else {"ln_modulate", "gemm_final"})
    assert torch.equal(x, x0)
    t64 = temb.double()
    m = lin(t64 / (1 + torch.exp(-t64)), sw["fmod_w"], sw["fmod_b"])[:, None]
    want = lin(ln(x.double(), m[..., :hidden], m[..., hidden:]), sw["fout_w"], sw["fout_b"])
    assert (v.double() - want).abs().max() <= 1e-2 * want.abs().max()


# A step that reuses its residual. The block adds gate1 out_b + gate2 mlp2_b (its other weights are zero), so the
# residual is known; it is of x's size. x is rounded to bf16 after each addition and once with the residual (2^-9
# each, random), h once more: below 2^-8 of the output's size together, as above.
@pytest.mark.parametrize("hidden,latent,b,n,one_pass", [(64, 64, 3, 5, True), (320, 64, 2, 33, True), (512, 64, 2, 48, True),
                                                        (1088, 64, 2, 16, True), (2048, 64, 2, 48, True), (2048, 64, 3, 33, True),
                                                        (3072, 64, 2, 48, True), (3072, 64, 2, 33, True), (4096, 64, 2, 32, True),
                                                        (4096, 64, 3, 7, True), (320, 128, 2, 40, True), (3072, 128, 2, 33, False)])
def test_reused_residual(d, hidden, latent, b, n, one_pass):
    g = torch.Generator(device="cuda").manual_seed(hidden + n)
    bf = torch.bfloat16
    c = d.block_config(hidden, hidden // 64, 64, 64, n, 0, 1, n)
    sw = weights(hidden, latent, bf, g)
    sw["t2_w"] *= 20.0                                      # a temb of ordinary size
    sw["in_w"] *= 6.0
    blk = {k: torch.zeros(s, dtype=bf, device="cuda")
           for k, s in {"qkv_w": (3 * hidden, hidden), "qkv_b": (3 * hidden,), "out_w": (hidden, hidden), "mlp1_w": (64, hidden),
                        "mlp1_b": (64,), "mlp2_w": (hidden, 64)}.items()}
    blk["mod_w"], blk["mod_b"] = ((torch.randn(*s, generator=g, device="cuda") * 0.02).to(bf) for s in ((6 * hidden, hidden), (6 * hidden,)))
    blk["out_b"], blk["mlp2_b"] = (torch.randn(hidden, generator=g, device="cuda").to(bf) for _ in range(2))
    blk["mod_b"].view(6, hidden)[[2, 5]] += 1.0             # gates about 1
    bw, swt = d.block_weights(blk, blk), d.step_weights(sw)
    st, cache = d.teacache_state(1e30), d.workspace(d.dit_teacache_cache_bytes(c, b))
    ws = d.workspace(d.dit_denoise_workspace_bytes(c, b, latent))
    v = torch.zeros(b, n, latent, device="cuda")

    def cond(t):
        temb = torch.empty(b, hidden, device="cuda")
        d.dit_timestep_embed(c, swt, torch.full((b,), t, device="cuda"), temb, ws)
        t64 = temb.double()
        return (t64 / (1 + torch.exp(-t64)))[:, None]

    s1, s2 = cond(0.9), cond(0.3)
    m1 = lin(s1, blk["mod_w"], blk["mod_b"]).view(b, 1, 6, hidden)
    resid = m1[:, :, 2] * blk["out_b"].double() + m1[:, :, 5] * blk["mlp2_b"].double()
    lat = [torch.randn(b, n, latent, generator=g, device="cuda") for _ in range(2)]
    x2 = lin(lat[1].double(), sw["in_w"], sw["in_b"])
    ran, _ = d.dit_denoise_step_teacache(c, swt, [bw], 0.9, 0.85, 0.0, lat[0], None, None, v, st, cache, ws)
    assert ran
    d.dit_profile_begin()
    ran, _ = d.dit_denoise_step_teacache(c, swt, [bw], 0.3, 0.25, 0.0, lat[1], None, None, v, st, cache, ws)
    names = {s["name"] for s in d.dit_profile_end()}
    assert not ran and ("final_head" in names) == one_pass and ("gemm_final" in names) == (not one_pass)
    fm = lin(s2, sw["fmod_w"], sw["fmod_b"])
    want = lin(ln(x2 + resid, fm[..., :hidden], fm[..., hidden:]), sw["fout_w"], sw["fout_b"])
    assert (v.double() - want).abs().max() <= 1e-2 * want.abs().max()


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("hidden,b,n", [(64, 1, 1), (576, 2, 9), (1088, 1, 30), (2176, 2, 5), (4096, 1, 11), (128, 3, 1100)])
def test_teacache_distance_widths(d, dtype, hidden, b, n):
    g = torch.Generator(device="cuda").manual_seed(hidden)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    c = d.block_config(hidden, hidden // 64, 64, 64, n, 0, 1, n, dtype=dtype)
    sw = weights(hidden, 64, tdt, g)
    sw["t2_w"] *= 20.0                                      # a temb of ordinary size
    blk = {k: (torch.randn(s, generator=g, device="cuda") * 0.02).to(tdt)
           for k, s in {"mod_w": (6 * hidden, hidden), "mod_b": (6 * hidden,), "qkv_w": (3 * hidden, hidden),
                        "qkv_b": (3 * hidden,), "out_w": (hidden, hidden), "out_b": (hidden,), "mlp1_w": (64, hidden),
                        "mlp1_b": (64,), "mlp2_w": (hidden, 64), "mlp2_b": (hidden,)}.items()}
    bw, swt = d.block_weights(blk, blk), d.step_weights(sw)
    st, cache = d.teacache_state(1e30), d.workspace(d.dit_teacache_cache_bytes(c, b))
    ws = d.workspace(d.dit_denoise_workspace_bytes(c, b, 64))

    def modulated(lat, t):
        temb = torch.empty(b, hidden, device="cuda")
        d.dit_timestep_embed(c, swt, torch.full((b,), t, device="cuda"), temb, ws)
        t64 = temb.double()
        m = lin(t64 / (1 + torch.exp(-t64)), blk["mod_w"], blk["mod_b"])[:, None]
        return ln(lin(lat.double(), sw["in_w"], sw["in_b"]), m[..., :hidden], m[..., hidden:2 * hidden])

    h = []
    for t in (0.9, 0.3):
        lat = torch.randn(b, n, 64, generator=g, device="cuda")
        h.append(modulated(lat, t))
        _, rel = d.dit_denoise_step_teacache(c, swt, [bw], t, t - 0.1, 0.0, lat, None, None, None, st, cache, ws)
    want = ((h[1] - h[0]).abs().sum() / h[0].abs().sum()).item()
    assert want > 0.3
    assert abs(rel - want) <= (1.3e-2 if dtype == "bf16" else 1e-5) * want
