"""The fp32 matrix-instruction kernels at the edges of their tiles.

GEMM (through the patch embedding, the ABI's plain GEMM): integer operands make every partial sum an
integer below 2^24, so fp32 results are exact in any order and are compared bit for bit, on both tile
shapes (32 x 32 with K split over four waves, 64 x 64) with ragged rows and one to many k slices.

Attention against float64: the score of a query and a key is a d-term fp32 sum, off by at most
(d + 2) 2^-24 sum|q k| scale; with N(0, 1) inputs sum|q k| scale stays below 12 at d = 128, so
probabilities (and with them the output, a convex combination of v) are off by at most 1e-4 of max|v|
in the worst case. Typical errors are a hundred times smaller; 1e-5 separates them from a wrong tile."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def d():
    from paper_2606_19004_amd import ditstep
    return ditstep


# (grid_h, grid_w, batch, hidden, K): one row; both sides of a 32- and a 64-row tile; 2, 6 and 20 k
# slices; enough tiles for the 64 x 64 kernel (3 and 20 slices of 32, last row tile partial)
@pytest.mark.parametrize("gh,gw,b,hidden,k", [(1, 1, 1, 64, 64), (1, 31, 1, 128, 64), (1, 33, 1, 64, 192), (5, 13, 1, 64, 640),
                                              (7, 9, 3, 320, 64), (50, 41, 4, 1024, 64), (31, 33, 8, 1024, 640)])
def test_gemm_f32_integer_operands_exact(d, gh, gw, b, hidden, k):
    g = torch.Generator(device="cuda").manual_seed(7)
    n = gh * gw
    c = d.block_config(hidden, hidden // 64, 64, 4 * hidden, n, 0, gh, gw, dtype="f32")
    lat = torch.randint(-3, 4, (b, n, k), generator=g, device="cuda").float()
    sw = {nm: torch.zeros(shp, device="cuda") for nm, shp in
          {"t1_w": (hidden, 256), "t1_b": (hidden,), "t2_w": (hidden, hidden), "t2_b": (hidden,), "in_w": (hidden, k),
           "in_b": (hidden,), "fmod_w": (2 * hidden, hidden), "fmod_b": (2 * hidden,), "fout_w": (k, hidden),
           "fout_b": (k,)}.items()}
    sw["in_w"] = torch.randint(-3, 4, (hidden, k), generator=g, device="cuda").float()
    sw["in_b"] = torch.randint(-3, 4, (hidden,), generator=g, device="cuda").float()
    x = torch.full((b, n, hidden), 0.5, device="cuda")
    d.dit_patch_embed(c, d.step_weights(sw), lat, x, d.workspace(256))
    want = lat.double().reshape(-1, k) @ sw["in_w"].double().t() + sw["in_b"].double()
    assert torch.equal(x.double().reshape(-1, hidden), want)


@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("seq", [1, 15, 16, 17, 32, 33, 63, 64, 65, 130])
def test_attention_f32_tile_edges(d, hd, seq):
    b, h = 2, 3
    g = torch.Generator(device="cuda").manual_seed(seq + hd)
    qkv = torch.randn(b, seq, 3, h, hd, generator=g, device="cuda")
    o = torch.full((b, h, seq, hd), 9.0, device="cuda")      # head-major output: other strides than the input's
    d.joint_attention(qkv[:, :, 0], qkv[:, :, 1], qkv[:, :, 2], o, b, h, seq, hd,
                      (seq * 3 * h * hd, 3 * h * hd, hd), (h * seq * hd, hd, seq * hd), dtype="f32")
    q, k, v = (t.permute(0, 2, 1, 3).double().cpu().numpy() for t in qkv.unbind(2))
    s = q @ k.swapaxes(-1, -2) / np.sqrt(hd)
    p = np.exp(s - s.max(-1, keepdims=True))
    want = (p / p.sum(-1, keepdims=True)) @ v
    assert np.max(np.abs(o.cpu().numpy() - want)) <= 1e-5 * np.max(np.abs(v))


@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("seq", [1, 17, 33, 47, 64])
def test_attention_f32_infinite_value_in_the_last_key(d, hd, seq):
    """An infinite value stays in its own column, also where the last tile of keys is not full: every query gives
    the last key a positive probability (scores of unit size), so that column is inf and the others are finite."""
    b, h = 1, 2
    g = torch.Generator(device="cuda").manual_seed(seq + hd)
    qkv = torch.randn(b, seq, 3, h, hd, generator=g, device="cuda") * 0.1
    clean = qkv.clone()
    qkv[:, -1, 2, :, 5] = float("inf")
    o = [torch.zeros(b, seq, h, hd, device="cuda") for _ in range(2)]
    for x, out in zip((qkv, clean), o):
        d.joint_attention(x[:, :, 0], x[:, :, 1], x[:, :, 2], out, b, h, seq, hd, (seq * 3 * h * hd, 3 * h * hd, hd),
                          (seq * h * hd, h * hd, hd), dtype="f32")
    assert torch.isposinf(o[0][..., 5]).all()
    keep = [e for e in range(hd) if e != 5]
    assert torch.equal(o[0][..., keep], o[1][..., keep])


@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("size,scale", [(1e20, 1e-30), (1e-36, 3e38), (1e-36, -3e38)])
def test_attention_f32_scale_of_any_size(d, hd, size, scale):
    """Scores that fit fp32 while the unscaled products, or the scale in the exponential's base, do not. Large q and k
    give scores some 1e10 apart (one key takes all); at 1e-36 sum|q k| scale is below 300, off by at most
    (d + 2) 2^-24 of that = 2.3e-3, which moves the output by less than twice that of max|v|."""
    b, h, seq = 1, 2, 37
    g = torch.Generator(device="cuda").manual_seed(hd)
    q, k, v = (torch.randn(b, seq, h, hd, generator=g, device="cuda") for _ in range(3))
    q, k = q * size, k * (size if size > 1 else 1e-2)
    o = torch.zeros(b, seq, h, hd, device="cuda")
    d.joint_attention(q, k, v, o, b, h, seq, hd, (seq * h * hd, h * hd, hd), (seq * h * hd, h * hd, hd), scale=scale, dtype="f32")
    qd, kd, vd = (t.permute(0, 2, 1, 3).double() for t in (q, k, v))
    p = torch.softmax(qd @ kd.transpose(-1, -2) * scale, -1)
    want = (p @ vd).permute(0, 2, 1, 3)
    assert (o.double() - want).abs().max() <= (1e-5 if size > 1 else 4.6e-3) * v.abs().max()


@pytest.mark.parametrize("hd", [64, 128])
def test_attention_f32_scores_near_the_largest_float(d, hd):
    """Scores up to 3e38, which no factor above 1.13 leaves finite: the largest takes all, exactly."""
    b, h, seq = 1, 2, 37
    g = torch.Generator(device="cuda").manual_seed(hd)
    q, k = (torch.zeros(b, seq, h, hd, device="cuda") for _ in range(2))
    v = torch.randn(b, seq, h, hd, generator=g, device="cuda")
    q[..., 0] = 1e19
    k[..., 0] = (torch.randperm(seq, generator=g, device="cuda").float() * (6e19 / 36) - 3e19)[None, :, None]
    o = torch.zeros(b, seq, h, hd, device="cuda")
    d.joint_attention(q, k, v, o, b, h, seq, hd, (seq * h * hd, h * hd, hd), (seq * h * hd, h * hd, hd), scale=1.0, dtype="f32")
    assert torch.equal(o, v[:, k[0, :, 0, 0].argmax()][:, None].expand_as(o))


def test_gemm_f32_rows_past_2_gib_of_a_tile(d):
    """An MLP so wide that the 32 rows of a down-projection tile span 2 GiB: everything is zero but the last element
    of the last row, GELU(8) = 8 exactly in fp32."""
    hidden, mlp = 64, 16777216 + 64
    c = d.block_config(hidden, 1, 64, mlp, 1, 0, 1, 1, dtype="f32")
    w = {k: torch.zeros(shp, device="cuda") for k, shp in
         {"mod_w": (6 * hidden, hidden), "mod_b": (6 * hidden,), "qkv_w": (3 * hidden, hidden), "qkv_b": (3 * hidden,),
          "out_w": (hidden, hidden), "out_b": (hidden,), "mlp1_w": (mlp, hidden), "mlp1_b": (mlp,), "mlp2_w": (hidden, mlp),
          "mlp2_b": (hidden,)}.items()}
    w["mod_b"][5 * hidden:] = 1.0                             # gate2
    w["mlp1_b"][-1] = 8.0
    w["mlp2_w"][-1, -1] = 1.0
    x = torch.zeros(1, 1, hidden, device="cuda")
    d.dit_block_mlp(c, d.block_weights(w, w), torch.zeros(1, hidden, device="cuda"), x, None,
                    d.workspace(d.dit_block_workspace_bytes(c, 1)))
    want = torch.zeros(hidden, device="cuda")
    want[-1] = 8.0
    assert torch.equal(x.view(-1), want)
