"""The bf16 GEMM's choice of tile on the host: each tile is the choice somewhere, and the sizes that the rule was
measured at keep theirs."""
import pytest

from paper_2606_19004_amd import ditstep as d
from tests.plan_util import gemm_plan


def cfg(hidden, n_img, n_txt, mlp=None):
    return d.block_config(hidden, hidden // 64, 64, mlp or 4 * hidden, n_img, n_txt, 1, n_img)


@pytest.mark.parametrize("op,want", [("out", (128, 128, 0, 1, 5)), ("qkv", (256, 192, 0, 1, 0)), ("mlp_up", (256, 256, 0, 1, 0)), ("mlp_down", (256, 192, 0, 3, 0))])
def test_one_seed_at_512(op, want):
    assert gemm_plan(cfg(3072, 1024, 256), 1, op) == want


@pytest.mark.parametrize("hidden,n,n_txt,b,op,want", [(320, 143, 37, 2, "out", (32, 32, 0, 1, 0)), (3072, 256, 64, 1, "out", (64, 64, 0, 1, 0)),
                                                      (3072, 1024, 256, 16, "qkv", (256, 256, 192, 1, 0)),
                                                      (3072, 1024, 256, 2, "mlp_down", (256, 256, 0, 2, 0)),
                                                      (3072, 1024, 256, 8, "mlp_down", (256, 256, 0, 1, 0))])
def test_tiles_by_size(hidden, n, n_txt, b, op, want):
    assert gemm_plan(cfg(hidden, n, n_txt), b, op) == want


# the patch embedding (K = latent width): 64 x 64 tiles in a ring of two stages from half a tile per compute unit to
# six, below that at one or two k-tiles only; others past that and for K above 512
@pytest.mark.parametrize("hidden,n,k,want", [(64, 8, 64, (64, 64, 0, 1, 2)), (64, 8, 128, (64, 64, 0, 1, 2)), (64, 8, 192, (32, 32, 0, 1, 0)),
                                             (64, 9000, 64, (64, 64, 0, 1, 2)), (640, 1000, 512, (64, 64, 0, 1, 2)),
                                             (640, 360, 512, (32, 32, 0, 1, 0)), (1280, 4096, 512, (64, 64, 0, 1, 2)),
                                             (640, 1000, 576, (64, 64, 0, 1, 0)), (3072, 16384, 64, (256, 256, 0, 1, 0))])
def test_short_k(hidden, n, k, want):
    assert gemm_plan(cfg(hidden, n, 0), 1, "patch", k) == want
