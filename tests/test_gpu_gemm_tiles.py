"""Every bf16 GEMM tile shape at its edges, with integer operands whose results are exact in any order.

Through the patch embedding (plain GEMM): rows and features around the tile edges and one to many 64-deep k-tiles.
Which tile a size takes is the library's choice, so test_tile_exact names it for every size and asks the library:
32 x 32 and 64 x 64 tiles whose four waves share K (none, one or several slices each, evenly or not; 64 x 64 is the
choice from nine k-tiles on), the ring of two stages on 64 x 64 tiles, the ring of five on 128 x 128 (again from
nine), and the three-stage 256 x 192 and 256 x 256 tiles from one k-tile on. A block then runs every epilogue on
the small tiles, two streams in one launch, against the oracle."""
import numpy as np
import pytest
import torch

import seeded_inputs as si
from oracle import dit_oracle as O
from tests.conftest import weights_f64
from tests.gpu_util import block_cfg, dev, host64, rel_err, upload_block
from tests.plan_util import gemm_plan

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def d():
    from paper_2606_19004_amd import ditstep
    return ditstep


def patch(d, b, n, hidden, k, skew=0, bias_skew=None):
    g = torch.Generator(device="cuda").manual_seed(b * n + hidden + k)
    c = d.block_config(hidden, hidden // 64, 64, 4 * hidden, n, 0, 1, n)
    # at most 60 nonzero +-1 entries per row keep every partial sum an integer below 2^8
    nz = min(60, k)
    pos = torch.rand(b * n, k, generator=g, device="cuda").argsort(1)[:, :nz]
    lat = torch.zeros(b * n, k, device="cuda").scatter_(1, pos, torch.randint(0, 2, (b * n, nz), generator=g, device="cuda") * 2.0 - 1)
    w = torch.randint(-1, 2, (hidden * k + skew,), generator=g, device="cuda").to(torch.bfloat16)[skew:].view(hidden, k)
    bias_skew = skew if bias_skew is None else bias_skew
    bias = torch.randint(-2, 3, (hidden + bias_skew,), generator=g, device="cuda").to(torch.bfloat16)[bias_skew:]
    z = torch.zeros(2 * hidden * max(hidden, 256), dtype=torch.bfloat16, device="cuda")
    sw = {nm: z for nm in ("t1_w", "t1_b", "t2_w", "t2_b", "fmod_w", "fmod_b", "fout_w", "fout_b")}
    sw["in_w"], sw["in_b"] = w, bias
    x = torch.full((b, n, hidden), 0.5, dtype=torch.bfloat16, device="cuda")
    d.dit_patch_embed(c, d.step_weights(sw), lat.view(b, n, k), x, d.workspace(2 * b * n * k + 256))
    want = lat.double() @ w.double().t() + bias.double()
    assert want.abs().max() <= 256
    assert torch.equal(x.double().view(-1, hidden), want)


@pytest.mark.parametrize("k", [64, 128, 256, 320, 384, 576, 1280])
@pytest.mark.parametrize("rows,hidden", [(1, 64), (31, 64), (33, 128), (65, 320), (127, 448)])
def test_small_tiles_exact(d, rows, hidden, k):
    patch(d, 1, rows, hidden, k)


@pytest.mark.parametrize("k", [64, 192, 256, 320, 384, 1024])
@pytest.mark.parametrize("b,n,hidden", [(2, 161, 3072), (3, 427, 1536), (5, 205, 3008), (1, 1024, 3072), (4, 1000, 2048)])
def test_larger_tiles_exact(d, b, n, hidden, k):
    patch(d, b, n, hidden, k)


T32, T64, RING64, T128, T192, T256 = ((32, 32, 0, 1, 0), (64, 64, 0, 1, 0), (64, 64, 0, 1, 2), (128, 128, 0, 1, 5),
                                      (256, 192, 0, 1, 0), (256, 256, 0, 1, 0))


@pytest.mark.parametrize("tile,rows,hidden,ks", [(T32, 1, 64, (192, 256, 320, 576)), (T32, 33, 128, (192, 384, 1280)),
                                                 (T32, 127, 448, (256, 320, 576)), (RING64, 65, 320, (64, 128)),
                                                 (RING64, 161, 3072, (192, 512)), (T64, 200, 3072, (576, 640, 704, 1024)),
                                                 (T64, 2000, 320, (576, 640, 704, 1280)), (T64, 3000, 192, (576, 832)),
                                                 (T128, 700, 1536, (576, 640, 704, 1280)), (T128, 1025, 3008, (576, 1024)),
                                                 (T192, 16383, 448, (64, 128, 192, 256, 320, 576)), (T192, 4000, 2048, (64, 384)),
                                                 (T256, 24001, 448, (64, 128, 192, 256, 320, 576)), (T256, 16384, 3072, (64, 192))])
def test_tile_exact(d, tile, rows, hidden, ks):
    c = d.block_config(hidden, hidden // 64, 64, 4 * hidden, rows, 0, 1, rows)
    for k in ks:
        assert gemm_plan(c, 1, "patch", k) == tile
        patch(d, 1, rows, hidden, k)


# 64 x 64 tiles in a ring of two stages: one to many k-tiles, whole and ragged rows, one tile to six per compute unit
@pytest.mark.parametrize("rows,hidden,k", [(1, 64, 64), (65, 128, 128), (2177, 320, 64), (1000, 640, 192), (8193, 64, 256),
                                           (700, 3072, 320), (1999, 3072, 512), (24575, 256, 448)])
def test_short_k_ring_exact(d, rows, hidden, k):
    c = d.block_config(hidden, hidden // 64, 64, 4 * hidden, rows, 0, 1, rows)
    assert gemm_plan(c, 1, "patch", k) == (64, 64, 0, 1, 2)
    patch(d, 1, rows, hidden, k)


def test_weights_at_8_byte_alignment(d):
    for rows, hidden, k in ((33, 128, 256), (1281, 1536, 1024), (300, 3072, 512)):
        patch(d, 1, rows, hidden, k, skew=4)


def test_patch_bias_at_any_element_alignment(d):
    for rows, hidden, k in ((33, 128, 256), (200, 3072, 512), (1281, 1536, 1024), (16384, 3072, 64)):
        for skew in (1, 2, 3):
            patch(d, 1, rows, hidden, k, bias_skew=skew)


# every epilogue with both streams in one launch, on 32 x 32 to 256 x 192 tiles by size
@pytest.mark.parametrize("hidden,hd,gh,gw,n_txt,b", [(128, 64, 3, 11, 1, 2), (576, 64, 13, 9, 45, 2), (1024, 128, 19, 21, 90, 2),
                                                     (1024, 64, 9, 7, 130, 1)])
def test_block_small_tiles(d, hidden, hd, gh, gw, n_txt, b):
    cfg = si.Shape("tiles", hidden, hidden // hd, hd, gh, gw, n_txt, b)
    inp = si.block_inputs(cfg)
    w = upload_block(inp["weights"], "bf16")
    c = block_cfg(d, cfg)
    xi, xt = dev(inp["x_img"], "bf16"), dev(inp["x_txt"], "bf16")
    d.dit_block_forward(c, d.block_weights(w["img"], w["txt"]), dev(inp["temb"]), xi, xt,
                        d.workspace(d.dit_block_workspace_bytes(c, b)))
    ri, rt = O.block_forward(cfg, weights_f64(inp["weights"], "bf16"), inp["temb"].astype(np.float64),
                             si.as_f64(inp["x_img"], "bf16"), si.as_f64(inp["x_txt"], "bf16"))
    assert rel_err(host64(xi), ri) <= 2e-2
    assert rel_err(host64(xt), rt) <= 2e-2
