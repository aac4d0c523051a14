"""The MLP down-projection with K shared out between workgroups (few rows, long K), against float64, run
after run the same bits: which workgroup of a tile finishes last differs from run to run, the order of the
sum does not. Each size names the tile columns and the number of parts that it has to take: two and three parts
on 256 x 192 and 256 x 256 tiles, whole and ragged row tiles, columns that do not fill the last tile, both
streams, one of them of a single row, and k-tile counts that the parts do not share evenly. Parts = 1: near the
sizes above, but unshared, on 128 x 128 tiles or, with more rows, on the three-stage 256-row ones."""
import pytest
import torch

from tests.plan_util import gemm_plan

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def d():
    from paper_2606_19004_amd import ditstep
    return ditstep


def lin(x, w, b):
    return x @ w.double().t() + b.double()


@pytest.mark.parametrize("hidden,mlp,gh,gw,n_txt,b,cols,parts",
                         [(1024, 16384, 32, 32, 256, 1, 256, 3), (1024, 16384, 25, 40, 217, 1, 256, 3),
                          (1088, 16448, 37, 27, 1, 1, 128, 1), (3072, 12288, 32, 32, 256, 1, 192, 3),
                          (3072, 12288, 32, 32, 256, 2, 256, 2), (3072, 12288, 31, 33, 250, 2, 256, 2),
                          (2048, 8192, 22, 28, 15, 2, 128, 1),
                          # rows that do not fill their tiles do not need the tiles' scratch
                          (3072, 12288, 31, 33, 250, 1, 192, 3), (3072, 12288, 25, 40, 256, 1, 192, 3),
                          (1536, 6144, 28, 23, 1, 1, 192, 3), (1152, 6400, 41, 22, 1, 1, 192, 3),
                          (704, 2240, 42, 40, 250, 3, 192, 2), (1984, 7936, 43, 45, 1, 1, 192, 2),
                          (640, 2560, 1283, 1, 478, 4, 192, 2), (1088, 8704, 39, 41, 63, 6, 192, 1),
                          (1216, 4544, 40, 28, 7, 4, 256, 2),
                          (1024, 4096, 43, 30, 1, 4, 256, 2), (1792, 11648, 24, 23, 1, 1, 256, 3), (1088, 8704, 39, 41, 21, 8, 256, 1)])
def test_mlp_down_split(d, hidden, mlp, gh, gw, n_txt, b, cols, parts):
    bf, n = torch.bfloat16, gh * gw
    g = torch.Generator(device="cuda").manual_seed(hidden + mlp + b * n)

    def randn(*shape, std=1.0, dtype=bf):
        return torch.empty(shape, dtype=dtype, device="cuda").normal_(0.0, std, generator=g)

    c = d.block_config(hidden, hidden // 64, 64, mlp, n, n_txt, gh, gw)
    assert gemm_plan(c, b, "mlp_down")[1::2] == (cols, parts)
    w = [{k + s: randn(*(shp if s == "_w" else shp[:1]), std=0.02) for k, shp in
          {"mod": (6 * hidden, hidden), "qkv": (3 * hidden, hidden), "out": (hidden, hidden), "mlp1": (mlp, hidden),
           "mlp2": (hidden, mlp)}.items() for s in ("_w", "_b")} for _ in range(2)]
    bw = d.block_weights(*w)
    temb, x0 = randn(b, hidden, dtype=torch.float32), [randn(b, n, hidden), randn(b, n_txt, hidden)]
    ws = d.workspace(d.dit_block_workspace_bytes(c, b))
    first = None
    for _ in range(6):
        x = [t.clone() for t in x0]
        ws.random_(0, 256, generator=g)          # nothing in the workspace needs to start at zero
        d.dit_block_mlp(c, bw, temb, x[0], x[1], ws)
        if first is None:
            first = x
        assert all(torch.equal(p.view(torch.int16), q.view(torch.int16)) for p, q in zip(x, first))
    t64 = temb.double()
    for s in range(2):
        m = lin(t64 / (1 + torch.exp(-t64)), w[s]["mod_w"], w[s]["mod_b"])[:, None]
        xd = x0[s].double()
        xc = xd - xd.mean(-1, keepdim=True)
        h = xc / torch.sqrt((xc * xc).mean(-1, keepdim=True) + 1e-6) * (1 + m[..., 4 * hidden:5 * hidden]) + m[..., 3 * hidden:4 * hidden]
        u = lin(h, w[s]["mlp1_w"], w[s]["mlp1_b"])
        u = 0.5 * u * (1 + torch.tanh((2 / torch.pi) ** 0.5 * (u + 0.044715 * u ** 3)))
        want = xd + m[..., 5 * hidden:] * lin(u, w[s]["mlp2_w"], w[s]["mlp2_b"])
        assert (first[s].double() - want).abs().max() <= 2e-2 * want.abs().max()
