"""Which tile a forward or backward-data product is cut into (host rule, no GPU)."""
import os

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LDS_BYTES = 160 * 1024                                   # of a compute unit


@pytest.fixture(scope="module")
def P():
    if not os.path.exists(os.path.join(ROOT, "paper_1807_06629_amd", "libprsgd.so")):
        from paper_1807_06629_amd.build import build
        build()
    from paper_1807_06629_amd import prsgd
    return prsgd


# minibatch rows, layer columns, workers: from one tile to many rounds of them
SHAPES = [(b, n, w) for b in (1, 8, 31, 32, 33, 64, 65, 100, 128, 129, 300, 512)
          for n in (10, 100, 256, 300, 1000, 1024, 4096) for w in (1, 8, 12, 16, 64, 200)]


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_a_compute_unit_holds_two_workgroups_of_the_smaller_tiles(P, dtype):
    seen = set()
    for b, n, w in SHAPES:
        rows, cols, lds = P.prsgd_product_tile(b, n, w, dtype)
        seen.add((rows, cols))
        # an operand tile is 128 bytes deep; three in flight, or four in half of the LDS (small launches with requesting wavefronts, fp32)
        assert lds <= max(3 * (rows + cols) * 128, LDS_BYTES // 2), (b, n, w, rows, cols, lds)
        if (rows, cols) != (128, 128):
            assert 2 * lds <= LDS_BYTES, (b, n, w, rows, cols, lds)
    assert seen == ({(32, 64), (64, 64), (128, 64), (128, 128)} if dtype == "bf16" else {(32, 32), (64, 64)})


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_no_tile_is_taller_than_the_minibatch(P, dtype):
    for b, n, w in SHAPES:
        rows, cols, _ = P.prsgd_product_tile(b, n, w, dtype)
        assert rows <= (32 if b <= 32 else 64 if b <= 64 else 128), (b, n, w, rows, cols)


# (rows, columns of a layer, tile): four tiles in flight are the launches with requesting wavefronts, three the others
@pytest.mark.parametrize("batch,cols,tile", [(64, 1024, (64, 64)), (64, 1000, (64, 64)), (32, 1024, (32, 64)), (31, 1001, (32, 64))])
def test_two_small_tiles_per_compute_unit_have_no_requesting_wavefronts(P, batch, cols, tile):
    stage = sum(tile) * 128
    assert P.prsgd_product_tile(batch, cols, 31, "bf16") == (*tile, 4 * stage)      # 496 tiles
    assert P.prsgd_product_tile(batch, cols, 32, "bf16") == (*tile, 3 * stage)      # 512


def test_bad_arguments_are_rejected(P):
    for bad in ((0, 1, 1), (1, 0, 1), (1, 1, 0)):
        with pytest.raises(P.PrsgdError):
            P.prsgd_product_tile(*bad, "f32")
