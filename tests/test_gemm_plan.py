"""The bf16 GEMM's choice of tile on the host: each tile is the choice somewhere, and the sizes that the rule was
measured at keep theirs."""
import pytest

from paper_2606_19004_amd import ditstep as d
from tests.plan_util import gemm_plan


def cfg(hidden, n_img, n_txt, mlp=None):
    return d.block_config(hidden, hidden // 64, 64, mlp or 4 * hidden, n_img, n_txt, 1, n_img)


@pytest.mark.parametrize("op,want", [("out", (128, 128, 0, 1)), ("qkv", (256, 192, 0, 1)), ("mlp_up", (256, 256, 0, 1)), ("mlp_down", (256, 192, 0, 3))])
def test_one_seed_at_512(op, want):
    assert gemm_plan(cfg(3072, 1024, 256), 1, op) == want


@pytest.mark.parametrize("hidden,n,n_txt,b,op,want", [(320, 143, 37, 2, "out", (32, 32, 0, 1)), (3072, 256, 64, 1, "out", (64, 64, 0, 1)),
                                                      (3072, 1024, 256, 16, "qkv", (256, 256, 192, 1)),
                                                      (3072, 1024, 256, 2, "mlp_down", (256, 256, 0, 2)),
                                                      (3072, 1024, 256, 8, "mlp_down", (256, 256, 0, 1))])
def test_tiles_by_size(hidden, n, n_txt, b, op, want):
    assert gemm_plan(cfg(hidden, n, n_txt), b, op) == want
