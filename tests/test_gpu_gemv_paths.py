"""The MFMA GEMV over its choices of kernel: batches of one to several 16-sample passes (rows past the batch
are left out of the loads), widths from one k step per wave to many, few and many weight matrices.

The input is taken as two bf16 parts, x = hi + lo to 2^-16 relative, the sums are fp32: an output is off by at
most 2^-16 sum|w x| (and K 2^-24 sum|w x| for the sums, less in practice), sqrt(K) ~ 20 to 64 times the typical
size of the result itself at these widths: 64 * 2^-16 = 1e-3 of max|out| bounds it, 1e-4 is typical."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def d():
    from paper_2606_19004_amd import ditstep
    return ditstep


def randn(g, *shape, std=1.0, dtype=torch.float32):
    return torch.empty(shape, dtype=dtype, device="cuda").normal_(0.0, std, generator=g)


def step_weights(g, hidden, latent=64):
    bf = torch.bfloat16
    w = {}
    for n, shp in {"t1": (hidden, 256), "t2": (hidden, hidden), "in": (hidden, latent), "fmod": (2 * hidden, hidden),
                   "fout": (latent, hidden)}.items():
        w[n + "_w"], w[n + "_b"] = randn(g, *shp, std=0.02, dtype=bf), randn(g, shp[0], std=0.02, dtype=bf)
    return w


@pytest.mark.parametrize("hidden", [64, 192, 1088, 3072, 4096])
@pytest.mark.parametrize("b", [1, 2, 5, 8, 9, 16, 17, 33])
def test_timestep_embed_batches(d, hidden, b):
    g = torch.Generator(device="cuda").manual_seed(hidden + b)
    c = d.block_config(hidden, hidden // 64, 64, 64, 1, 0, 1, 1)
    sw = step_weights(g, hidden)
    t = torch.rand(b, generator=g, device="cuda")
    temb = torch.full((b, hidden), 5.0, device="cuda")
    d.dit_timestep_embed(c, d.step_weights(sw), t, temb, d.workspace(d.dit_denoise_workspace_bytes(c, b, 64)))
    f = 1e4 ** (-torch.arange(128, dtype=torch.float64, device="cuda") / 128)
    arg = 1000.0 * t.double()[:, None] * f
    h = torch.cat([torch.cos(arg), torch.sin(arg)], 1) @ sw["t1_w"].double().t() + sw["t1_b"].double()
    want = (h / (1 + torch.exp(-h))) @ sw["t2_w"].double().t() + sw["t2_b"].double()
    assert (temb.double() - want).abs().max() <= 1e-3 * want.abs().max()


# A step (all modulations in one launch, inputs split by the launch before) against its parts called one by
# one (two weight matrices per launch, a split of their own). The parts differ in the order of fp32 sums
# only, which bf16 storage rounds away or turns into single-ulp differences: 2e-2 of max|v|.
# 4096 x 4 blocks: enough rows for whole-K waves; more than 16 samples: no chained start
@pytest.mark.parametrize("hidden,blocks,b,n_txt", [(128, 3, 1, 5), (128, 9, 4, 0), (320, 2, 17, 3), (1024, 5, 7, 4),
                                                   (4096, 4, 1, 2), (4096, 4, 16, 1)])
def test_step_equals_its_parts(d, hidden, blocks, b, n_txt):
    bf = torch.bfloat16
    g = torch.Generator(device="cuda").manual_seed(hidden * blocks + b)
    gh, gw = 3, 4
    n = gh * gw
    c = d.block_config(hidden, hidden // 64, 64, 64, n, n_txt, gh, gw)
    sw = d.step_weights(step_weights(g, hidden))
    shapes = {"mod": (6 * hidden, hidden), "qkv": (3 * hidden, hidden), "out": (hidden, hidden), "mlp1": (64, hidden),
              "mlp2": (hidden, 64)}
    bw = []
    for _ in range(blocks):
        pair = []
        for _ in range(2):
            w = {}
            for k, shp in shapes.items():
                w[k + "_w"], w[k + "_b"] = randn(g, *shp, std=0.02, dtype=bf), randn(g, shp[0], std=0.02, dtype=bf)
            pair.append(w)
        bw.append(d.block_weights(*pair))
    lat, xt = randn(g, b, n, 64), randn(g, b, n_txt, hidden, dtype=bf)
    ws = d.workspace(d.dit_denoise_workspace_bytes(c, b, 64))
    v, lat1 = torch.zeros_like(lat), lat.clone()
    d.dit_denoise_step(c, sw, bw, 0.5, 0.4, 0.0, lat1, xt, None, v, ws)
    temb, x, xt1, v2 = torch.zeros(b, hidden, device="cuda"), torch.zeros(b, n, hidden, dtype=bf, device="cuda"), xt.clone(), torch.zeros_like(v)
    d.dit_timestep_embed(c, sw, torch.full((b,), 0.5, device="cuda"), temb, ws)
    d.dit_patch_embed(c, sw, lat, x, ws)
    for w in bw:
        d.dit_block_forward(c, w, temb, x, xt1, ws)
    d.dit_final_layer(c, sw, temb, x, v2, ws)
    assert torch.isfinite(v).all()
    assert (v - v2).abs().max() <= 2e-2 * v2.abs().max()
    assert np.isfinite(lat1.cpu().numpy()).all()


# fp32: SiLU folded into the GEMV for few samples, a launch of its own past that (kernels of the second layer's
# input: 0 or 1 beside the sinusoid). fp32 sums of up to 1088 terms: 1e-5 of max|temb|
@pytest.mark.parametrize("hidden,b,apart", [(64, 2, 0), (64, 3, 1), (128, 4, 0), (512, 4, 0), (576, 2, 0), (576, 3, 1),
                                            (512, 5, 1), (1088, 1, 0), (1088, 2, 1), (1088, 17, 1)])
def test_timestep_embed_f32_silu(d, hidden, b, apart):
    g = torch.Generator(device="cuda").manual_seed(hidden + b)
    c = d.block_config(hidden, hidden // 64, 64, 64, 1, 0, 1, 1, dtype="f32")
    sw = {k: v.float() for k, v in step_weights(g, hidden).items()}
    t = torch.rand(b, generator=g, device="cuda")
    temb = torch.full((b, hidden), 5.0, device="cuda")
    d.dit_profile_begin()
    d.dit_timestep_embed(c, d.step_weights(sw), t, temb, d.workspace(d.dit_denoise_workspace_bytes(c, b, 64)))
    launches = {s["name"]: s["launches"] for s in d.dit_profile_end()}
    assert launches == {"small_elementwise": 1 + apart, "timestep_gemv": 2}
    f = 1e4 ** (-torch.arange(128, dtype=torch.float64, device="cuda") / 128)
    arg = 1000.0 * t.double()[:, None] * f
    h = torch.cat([torch.cos(arg), torch.sin(arg)], 1) @ sw["t1_w"].double().t() + sw["t1_b"].double()
    want = (h / (1 + torch.exp(-h))) @ sw["t2_w"].double().t() + sw["t2_b"].double()
    assert (temb.double() - want).abs().max() <= 1e-5 * want.abs().max()
