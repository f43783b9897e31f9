"""The C-ABI library loads and exports every function include/gllm_stage.h declares (no GPU needed)."""
import os
import re
import time

import pytest

from paper_2504_14775_amd import binding as B
from paper_2504_14775_amd import synth

HEADER = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "include", "gllm_stage.h")


def declared_functions():
    text = open(HEADER).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(gllm_[a-z0-9_]+)\s*\(", text)))


def test_header_declares_the_expected_entry_points():
    names = declared_functions()
    for n in ("gllm_stage_create", "gllm_stage_forward", "gllm_stage_load_layer", "gllm_stage_bind_kv_pool",
              "gllm_stage_bind_workspace", "gllm_stage_destroy", "gllm_last_error"):
        assert n in names


def test_library_exports_every_declared_function():
    lib = B.load_library()
    for n in declared_functions():
        assert hasattr(lib, n), n
    assert set(B.EXPORTS) == set(declared_functions())


def test_status_names_and_profile_classes():
    lib = B.load_library()
    for code, name in B.STATUS.items():
        assert lib.gllm_status_name(code).decode() == name
    n = lib.gllm_profile_num_classes()
    names = [lib.gllm_profile_class_name(i).decode() for i in range(n)]
    assert "gemm_gate_up_swiglu" in names and "attn_decode" in names and len(set(names)) == n


def test_create_rejects_bad_configs_before_touching_a_device():
    shape = synth.SHAPES["tiny"]
    import dataclasses
    for bad, status in [
        (dict(page_size=8), -7),
        (dict(head_dim=96), -7),
        (dict(n_q_heads=5), -7),
        (dict(hidden=200), -7),
        (dict(hidden=192), -7),          # a multiple of 64 but not of 128: the header states 128
        (dict(num_layers=0), -1),
    ]:
        cfg = B.make_config(dataclasses.replace(shape, **bad), 64, 8, 8, 128)
        with pytest.raises(B.GllmError) as e:
            B.Stage(cfg)
        assert e.value.status == status, (bad, e.value)
    cfg = B.make_config(shape, 64, 8, 4, 128)          # 4 pages cannot hold 128 positions
    with pytest.raises(B.GllmError) as e:
        B.Stage(cfg)
    assert e.value.status == -1


def test_gemm_planner_choices_are_launchable():
    """Host logic of the tile / split-K planner: whatever it picks must satisfy the launch rules of that tile
    (column multiple, split divides the 64-wide k-steps, splits only in store mode), for the stage shapes and a
    sweep of ragged row counts."""
    col_multiple = {0: 128, 1: 128, 3: 256, 4: 256, 5: 192, 6: 128, 7: 128, 8: 256, 9: 192, 13: 128, 14: 256, 15: 128}
    seen = set()
    for shape in synth.SHAPES.values():
        H, I = shape.hidden, shape.intermediate
        pad = lambda v, q: (v + q - 1) // q * q
        n_qkv = pad((shape.n_q_heads + 2 * shape.n_kv_heads) * shape.head_dim, 256)
        problems = [(n_qkv, pad(H, 64), 0), (pad(H, 256), pad(shape.n_q_heads * shape.head_dim, 64), 0),
                    (2 * pad(I, 256), pad(H, 64), 2), (pad(H, 256), pad(I, 256), 0), (2 * pad(I, 256), pad(H, 64), 1), (24768, pad(H, 64), 0)]
        for m in (1, 17, 100, 128, 200, 256, 257, 288, 289, 322, 384, 448, 512, 600, 1000, 1100, 2048, 2560, 4160):
            for n, k, mode in problems:
                tile, splits = B.gllm_op_gemm_plan(m, n, k, mode, 8)
                seen.add((tile, splits))
                assert tile in col_multiple and n % col_multiple[tile] == 0, (shape.name, m, n, k, mode, tile)
                assert 1 <= splits <= 8 and (k // 64) % splits == 0
                if mode != 0:
                    assert splits == 1 and (mode == 1 or tile not in (5, 9))
                if tile == 7:
                    assert m <= 64
                if tile == 8:
                    assert m > 384 and 0 < m % 256 <= 128
                if tile == 9:
                    assert 256 < m <= 288 and n % 128 != 0
                if tile == 13:
                    assert 256 < m <= 384
                if tile == 4:
                    tiles = ((m + 255) // 256) * (n // 256)
                    assert splits == 1 and tiles >= 256 and 0 < tiles % 256 <= 128
                assert B.gllm_op_gemm_plan(m, n, k, mode, 8) == (tile, splits)          # deterministic
                assert B.gllm_op_gemm_plan(m, n, k, mode, 1)[1] == 1                    # the cap is respected
                few = B.gllm_op_gemm_plan(m, n, k, mode, 2 ** 31 - 1)[1]                # no cap: as many as there are k-steps, at most
                assert (k // 64) % few == 0
    # big problems get 256x256 tiles (with a short last band where rows are left over), few rows the deep 128x128 or the
    # 64x128 one, rows between them bands of equal height; factors are no powers of two only
    assert {3, 6, 7, 8, 9, 13, 14, 15}.issubset({t for t, _ in seen}), seen
    assert {3, 5, 6}.intersection({s for _, s in seen}), seen
    # the vocabulary projection of a micro-batch of 256 decode rows plus one chunk end: one band
    assert B.gllm_op_gemm_plan(257, 128256, 4096, 0, 1) == (13, 1) and B.gllm_op_gemm_plan(289, 128256, 4096, 0, 1) == (13, 1)
    assert B.gllm_op_gemm_plan(256, 128256, 4096, 0, 1)[0] == 3
    assert B.gllm_op_gemm_plan(2048, 4096, 14336, 0, 8) == (3, 2) and B.gllm_op_gemm_plan(2048, 4096, 4096, 0, 8) == (15, 1)
    # columns that 128 does not divide, 257..288 rows: two bands of 256x192 tiles in one round, one band of 288x192 where these take two
    assert B.gllm_op_gemm_plan(257, 20160, 4096, 0, 1) == (5, 1) and B.gllm_op_gemm_plan(257, 24768, 4096, 0, 1) == (9, 1)
    with pytest.raises(B.GllmError):
        B.gllm_op_gemm_plan(128, 100, 4096, 0, 8)


def test_gemm_planner_ends_on_the_largest_problems():
    """Tiles are counted, not walked through, whatever the sizes: a short last band (row-mixed launch) over millions of columns,
    any number of splits allowed."""
    t = time.perf_counter()
    for m, n, k in ((2 ** 20 + 1, 2 ** 30, 2 ** 20), (513, 2 ** 31 - 256, 2 ** 31 - 64), (2 ** 31 - 1, 256, 64)):
        tile, splits = B.gllm_op_gemm_plan(m, n, k, 0, 2 ** 31 - 1)
        assert tile >= 0 and (k // 64) % splits == 0, (m, n, k)
    assert time.perf_counter() - t < 5.0


# us per product on MI355X with cold weights (median of three runs, forms in random order), of the (tile, splits) that come
# near the best one and of those that a planner could confuse with them; products in several planes include reading these at
# 6 TB/s
MEASURED_PRODUCTS = [
    ((65, 128256, 4096, 0, 1), {(0, 1): 169, (14, 1): 169, (3, 1): 183, (6, 1): 203, (15, 1): 204}),
    ((128, 128256, 4096, 0, 1), {(14, 1): 173, (0, 1): 187, (3, 1): 190, (5, 1): 216, (6, 1): 217, (15, 1): 218}),
    ((160, 128256, 4096, 0, 1), {(14, 1): 178, (3, 1): 192, (15, 1): 223, (5, 1): 224}),
    ((256, 128256, 4096, 0, 1), {(14, 1): 216, (3, 1): 222, (1, 1): 249, (15, 1): 251, (5, 1): 253}),
    ((257, 128256, 4096, 0, 1), {(13, 1): 237, (14, 1): 327, (8, 1): 341, (15, 1): 360, (3, 1): 379}),
    ((320, 128256, 4096, 0, 1), {(13, 1): 289, (14, 1): 343, (15, 1): 384, (3, 1): 389}),
    ((128, 128256, 8192, 0, 1), {(14, 1): 323, (6, 1): 361, (0, 1): 364, (3, 1): 378}),
    ((128, 152064, 5120, 0, 1), {(4, 1): 261, (14, 1): 279, (6, 1): 290, (0, 1): 290, (3, 1): 321}),
    ((288, 152064, 8192, 0, 1), {(13, 1): 608, (14, 1): 744, (8, 1): 782, (15, 1): 838, (3, 1): 883}),
    ((800, 57344, 8192, 2, 1), {(4, 1): 608, (14, 1): 660, (8, 1): 682, (15, 1): 721, (3, 1): 735}),
    ((773, 55296, 5120, 2, 1), {(4, 1): 384, (8, 1): 389, (14, 1): 410, (15, 1): 452, (3, 1): 464}),
    ((160, 55296, 5120, 2, 1), {(14, 1): 97.5, (3, 1): 121, (15, 1): 130}),
    ((1030, 28672, 4096, 2, 1), {(8, 1): 196, (15, 1): 235, (0, 1): 239, (14, 1): 240, (3, 1): 273}),
    ((1100, 28672, 4096, 2, 1), {(8, 1): 210, (0, 1): 242, (15, 1): 242, (14, 1): 247, (3, 1): 273}),
    ((1152, 28672, 4096, 2, 1), {(8, 1): 214, (14, 1): 224, (0, 1): 246, (15, 1): 250, (3, 1): 271}),
    ((1100, 27648, 5120, 2, 1), {(8, 1): 256, (15, 1): 302, (14, 1): 302, (0, 1): 316, (3, 1): 332}),
    ((257, 28672, 4096, 2, 1), {(13, 1): 61.2, (14, 1): 68.7, (15, 1): 81}),
    ((773, 4096, 4096, 0, 8), {(6, 1): 34.3, (0, 2): 34.7, (14, 2): 40.3, (6, 2): 41.7, (3, 4): 42.1, (1, 1): 42.2}),
    ((800, 4096, 4096, 0, 8), {(0, 2): 35.1, (6, 1): 35.2, (14, 2): 41.1, (3, 4): 42.1, (1, 1): 42.3}),
    ((550, 6144, 4096, 0, 8), {(6, 1): 36.3, (0, 2): 39.7, (0, 1): 43.6, (14, 2): 44.3, (6, 2): 44.9, (15, 1): 47.9}),
    ((600, 5120, 5120, 0, 8), {(1, 2): 40.8, (3, 4): 46, (14, 2): 46.5, (6, 1): 46.7, (0, 2): 47.4, (8, 4): 49}),
    ((256, 5120, 13824, 0, 8), {(15, 6): 47.5, (3, 8): 50.6, (0, 3): 52.1, (6, 3): 52.4, (15, 4): 52.4, (0, 6): 57}),
    ((256, 10240, 8192, 0, 8), {(15, 2): 57.1, (3, 4): 58.4, (0, 2): 68.6, (15, 4): 71.4, (6, 2): 71.7}),
    ((320, 5120, 27648, 0, 8), {(13, 6): 87.3, (14, 6): 93.3, (15, 3): 105, (13, 4): 110}),
    ((200, 4096, 14336, 0, 8), {(15, 7): 36.3, (15, 8): 36.4, (6, 4): 37.4, (1, 8): 37.5, (0, 8): 40.5}),
    ((2048, 4096, 14336, 0, 8), {(3, 2): 183, (15, 1): 192, (3, 4): 204, (15, 2): 206, (0, 1): 216}),
]


@pytest.mark.parametrize("problem,us", MEASURED_PRODUCTS)
def test_gemm_planner_stays_near_the_fastest_measured_form(problem, us):
    """The planner of the stage and the head: a column-mixed launch costs its whole rounds and its half-width ones, a row-mixed
    one starts its low tiles as compute units become free, a nearly empty last round behind whole ones costs more than its
    share, and of tiles that all wait for their loads the lighter one is better: the pick is within 6 % of the fastest form
    measured (runs differ by up to 3 %)."""
    tile, splits = B.gllm_op_gemm_plan(*problem)
    assert us.get((tile, splits), float("inf")) <= 1.06 * min(us.values()), (problem, tile, splits)


# us of norm, projection and greedy sampling on MI355X by the width of the tiles of one band (0: whole rounds of 192 columns, a last one of 128)
MEASURED_WIDTHS = [
    ((257, 32896, 4096), {128: 123}),
    ((257, 49152, 4096), {128: 137, 192: 112}),
    ((257, 65664, 4096), {128: 203, 192: 176, 0: 160}),
    ((288, 79104, 8192), {128: 381, 192: 352, 0: 330}),
    ((272, 89856, 5120), {128: 262, 192: 239, 0: 277}),
    ((257, 100352, 4096), {128: 259, 0: 246}),
    ((257, 128256, 4096), {128: 310, 192: 293, 0: 281}),
    ((272, 131328, 8192), {128: 612, 192: 537, 0: 579}),
    ((288, 152064, 4096), {128: 356, 192: 369, 0: 352}),
    ((288, 196608, 8192), {128: 857, 192: 800, 0: 841}),
]


@pytest.mark.parametrize("problem,us", MEASURED_WIDTHS)
def test_one_band_of_288_rows_goes_by_the_fastest_width(problem, us):
    m, n, k = problem
    assert us[B.gllm_op_gemm_tile_columns(m, n, k, 0, 13)] == min(us.values())
    if n % 192 == 0:
        assert B.gllm_op_gemm_tile_columns(m, n, k, 0, 9) == B.gllm_op_gemm_tile_columns(m, n, k, 0, 13)


def test_tile_columns_of_other_tiles():
    for tile, want in ((0, 128), (1, 128), (2, 256), (3, 256), (5, 192), (6, 128), (14, 256), (15, 128)):
        assert B.gllm_op_gemm_tile_columns(200, 768, 4096, 0, tile) == want, tile
    assert B.gllm_op_gemm_tile_columns(257, 576, 4096, 0, 9) == 192 and B.gllm_op_gemm_tile_columns(257, 768, 4096, 1, 9) == 192
    assert B.gllm_op_gemm_tile_columns(300, 49152, 4096, 0, 13) == 128 and B.gllm_op_gemm_tile_columns(257, 49152, 4096, 0, 13, 2) == 128
    assert B.gllm_op_gemm_tile_columns(257, 49152, 4096, 2, 13) == 128
    assert B.gllm_op_gemm_tile_columns(64, 4096, 4096, 0, 7, 4) == 64 and B.gllm_op_gemm_tile_columns(64, 152064, 5120, 0, 7) == 128
    assert B.gllm_op_gemm_tile_columns(80, 4096, 4096, 0, 6, 4) == 64
    for bad in ((257, 576, 4096, 2, 9, 1), (256, 768, 4096, 0, 13, 1), (200, 768, 4096, 0, 99, 1), (200, 100, 4096, 0, 0, 1), (200, 768, 4096, 0, 0, 3)):
        with pytest.raises(B.GllmError):
            B.gllm_op_gemm_tile_columns(*bad)
