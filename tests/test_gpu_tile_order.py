"""Every tile and every K split of a product belongs to exactly one workgroup, whatever number of tile rows is left behind the last
eight: small whole numbers, whose sums are exact in any order, against their product in 64 bits."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dt", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("tiles_m,tiles_n", [(1, 1), (1, 19), (7, 3), (8, 1), (9, 5), (10, 8), (13, 11), (23, 7)])
def test_every_tile_once(tiles_m, tiles_n, dt):
    from paper_1908_00213_amd import binding as B
    gen = torch.Generator(device="cuda").manual_seed(tiles_m * 100 + tiles_n)
    ints = lambda *s: torch.randint(-8, 9, s, generator=gen, device="cuda").to(dt)
    K = 1536                                    # sums of at most 1536 * 64 < 2^24
    for tile in (0, 1):
        b = 64 << tile
        M, N = tiles_m * b - 4, tiles_n * b
        x, w = ints(M, K), ints(K, N)
        want = x.double() @ w.double()
        for splits in (1, 3):
            B.gemm_plan_override(tile, splits, -1)
            try:
                y = torch.full((M, N), float("nan"), device="cuda")
                need = B.gemm_workspace_bytes(x, w, y)
                assert (need > 0) == (splits > 1)
                B.gemm(x, w, y, ws=torch.empty(max(need, 1), dtype=torch.uint8, device="cuda"))
            finally:
                B.gemm_plan_override(-1, -1, -1)
            assert torch.equal(y.double(), want), (tile, splits)
        y = torch.full((M, N), float("nan"), device="cuda")      # and as it is planned
        B.gemm(x, w, y, ws=torch.empty(max(B.gemm_workspace_bytes(x, w, y), 1), dtype=torch.uint8, device="cuda"))
        assert torch.equal(y.double(), want), tile
