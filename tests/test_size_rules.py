"""The library's size rules on the host. The bf16 GEMM's choice of tile: each tile is the choice somewhere, and the sizes that the rule was
measured at keep theirs."""
import pytest

from paper_2606_19004_amd import ditstep as d
from tests.plan_util import gemm_plan, reward_check_in_launch


def cfg(hidden, n_img, n_txt, mlp=None):
    return d.block_config(hidden, hidden // 64, 64, mlp or 4 * hidden, n_img, n_txt, 1, n_img)


@pytest.mark.parametrize("op,want", [("out", (128, 128, 0, 1, 5)), ("qkv", (256, 192, 0, 1, 0)), ("mlp_up", (256, 256, 0, 1, 0)), ("mlp_down", (256, 192, 0, 3, 0))])
def test_one_seed_at_512(op, want):
    assert gemm_plan(cfg(3072, 1024, 256), 1, op) == want


@pytest.mark.parametrize("hidden,n,n_txt,b,op,want", [(320, 143, 37, 2, "out", (32, 32, 0, 1, 0)), (3072, 256, 64, 1, "out", (64, 64, 0, 1, 0)),
                                                      (3072, 1024, 256, 16, "qkv", (256, 256, 192, 1, 0)),
                                                      (3072, 1024, 256, 2, "mlp_down", (256, 256, 0, 2, 0)),
                                                      # as above with rows that do not fill their tiles
                                                      (3072, 1024, 250, 1, "mlp_down", (256, 192, 0, 3, 0)),
                                                      (3072, 1023, 256, 1, "mlp_down", (256, 192, 0, 3, 0)),
                                                      (3072, 640, 64, 1, "mlp_down", (256, 192, 0, 3, 0)),
                                                      (576, 1196, 501, 4, "mlp_down", (256, 192, 0, 2, 0)),
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


# the check of the rewards inside the statistics launch: up to 16384 rewards, and not where many groups each look at
# all of them
@pytest.mark.parametrize("groups,n,want", [(1, 1, True), (64, 16, True), (4, 4096, True), (5, 4096, False), (1024, 16, True),
                                           (512, 32, True), (4096, 1, True), (2048, 8, False), (4096, 4, False), (16384, 1, False)])
def test_reward_check(groups, n, want):
    assert reward_check_in_launch(groups, n) == want
