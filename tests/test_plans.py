"""Launch plans, which the host computes from sizes alone (no GPU needed)."""
import ctypes as C
import os

import pytest

from util import binding, internal


@pytest.fixture(scope="module", autouse=True)
def built():
    if not os.path.exists(binding.LIB_PATH):
        from paper_2603_17942_amd import build
        build.build(verbose=False)


@pytest.mark.parametrize("m,ff,full,batch", [
    (128, 14336, 0b001, 0b001), (320, 14336, 0b001, 0b001), (352, 14336, 0b010, 0b011), (400, 14336, 0b010, 0b011),
    (512, 14336, 0b010, 0b010), (640, 14336, 0b001, 0b011), (1344, 14336, 0b001, 0b011), (2112, 14336, 0b010, 0b011),
    (400, 12288, 0b010, 0b011), (560, 12288, 0b100, 0b110), (640, 12288, 0b001, 0b111), (2048, 12288, 0b010, 0b011)])
def test_gate_up_tiles(m, ff, full, batch):
    """Tiles launched for the gate/up projection (bit 0 gemm_plan's, 1: 256 x 256, 2: 192 x 320) of m rows, and of a batch of m
    block rows, of which only the device knows how many are there: one that suits two thirds of them, and one that suits all
    (640 rows: up to 512 there one round of 256 x 256, more two of the ring)."""
    tiles = internal("gate_up_tiles", C.c_int, C.c_int, C.c_int, C.c_void_p, C.c_bool, restype=C.c_uint)
    assert tiles(m, ff, 4096, None, False) == full
    assert tiles(m, ff, 4096, None, True) == batch
    assert tiles(m, ff, 4096, 8, True) == 0b001             # results off the 16-byte alignment of the wide tiles' stores


class TileCost(C.Structure):
    _fields_ = [(n, C.c_int) for n in ("rt", "ct", "start", "chunk", "busy")]


class GateUpRule(C.Structure):
    _fields_ = [(n, C.c_int) for n in ("mt", "chunks", "blocks", "launched")] + [("tile", C.c_int * 3), ("cost", TileCost * 3)]


@pytest.mark.parametrize("m,ff,rows_cols", [
    (320, 12288, (5, 6)), (321, 12288, (6, 6)), (352, 12288, (6, 6)), (384, 12288, (6, 6)), (352, 11008, (6, 6)), (385, 12288, (8, 6)), (176, 18944, (6, 6)),
    (352, 14336, (6, 8)), (512, 14336, (8, 8)), (576, 12288, (6, 10)), (1024, 14336, (8, 8))])
def test_gate_up_tile_of_one_sequence(m, ff, rows_cols):
    """The one tile (in 32 rows, 32 columns) of the gate/up projection of m rows: 192 x 192 for 321 to 384 rows x 24576, which the rule
    of rounds alone gave 192 x 256 (70 to 73 us against 65 to 66)."""
    r = internal("gate_up_rule", C.c_int, C.c_int, C.c_int, C.c_void_p, C.c_bool, restype=GateUpRule)(m, ff, 4096, None, False)
    launched = [t for t in range(3) if r.launched >> t & 1]
    assert len(launched) == 1 and (r.cost[launched[0]].rt, r.cost[launched[0]].ct) == rows_cols


class GemmPlan(C.Structure):
    _fields_ = [(n, C.c_int) for n in ("splits", "mt", "nb", "m_tiles", "n_tiles", "ct")]


@pytest.mark.parametrize("n,k", [(6144, 4096), (4096, 4096), (4096, 14336), (4096, 12288), (28672, 4096), (1024, 8192), (544, 2048), (96, 640), (32, 64)])
def test_gemm_parts(n, k):
    """A product's split-K parts are no fewer than one round of the 256 CUs holds of tiles of 128 columns (up to 128 rows) or of 160
    x 256 (above), each of 512 of K or more: a running fp32 sum's error grows with the root of its terms, so the parts bound it.
    Up to 128 rows the parts do not depend on the rows."""
    one, batch = (internal(f, *[C.c_int] * a, restype=GemmPlan) for f, a in (("gemm_plan", 4), ("batch_gemm_plan", 3)))
    of_128 = one(binding.ESP_BF16, 128, n, k).splits
    for m in (1, 17, 32, 33, 68, 101, 128, 129, 160, 161, 200, 320, 321, 400, 512, 576, 700, 1024, 1344, 2112):
        tiles = -(-n // 128) if m <= 128 else -(-n // 256) * -(-(-(-m // 32)) // 5)
        least = max(1, min(256 // tiles, k // 512, 8))
        p = one(binding.ESP_BF16, m, n, k)
        assert least <= p.splits <= 8 and (m > 128 or p.splits == of_128), (m, p.splits, least)
        if m > 128:
            assert batch(m, n, k).splits >= least, (m, least)


@pytest.mark.parametrize("m,n,k,splits", [(192, 28672, 4096, 1), (180, 24576, 4096, 1), (1, 24576, 4096, 1), (128, 18944, 2048, 1), (1344, 4096, 4096, 1), (1344, 4096, 14336, 2), (320, 4096, 4096, 8),
                                          (68, 6144, 4096, 5), (2112, 4096, 4096, 1), (512, 28672, 4096, 1), (64, 96, 64, 1)])
def test_product_plan(m, n, k, splits):
    """A product on its own needs a launch more for its parts: whole where it used to be, unless the parts save more than that."""
    p = internal("product_plan", *[C.c_int] * 3, restype=GemmPlan)(m, n, k)
    assert p.splits == splits
    assert binding.load_library().esp_gemm_scratch_bytes(m, n, k) >= splits * m * n * 4


@pytest.mark.parametrize("n,k", [(6144, 4096), (4096, 4096), (4096, 14336), (28672, 4096), (2048, 2048), (544, 2048), (160, 1664), (32, 64)])
def test_row_major_gemm_plan(n, k):
    """Row-major weights have a kernel with tiles of its own, 128 columns wide up to 128 rows and 160 x 256 above: as many parts as
    one round of the 256 CUs has room for, and a tile the kernel is built for."""
    plan, scratch = internal("row_major_plan", *[C.c_int] * 3, restype=GemmPlan), binding.load_library().esp_gemm_scratch_bytes
    for m in (1, 32, 33, 68, 128, 129, 160, 161, 192, 320, 321, 512, 1024, 1344, 2112):
        p = plan(m, n, k)
        cols = 128 if m <= 128 else 256
        tiles = -(-n // cols) * (1 if m <= 128 else -(-m // 160))
        assert p.splits == max(1, min(256 // tiles, k // 512, 8)), (m, p.splits)
        assert p.splits == 1 or p.m_tiles * p.n_tiles * p.splits <= 256
        assert (p.nb, p.mt) in [(1, 1), (1, 2), (1, 3), (1, 4), (2, 3), (2, 4), (2, 5)] and (p.nb == 1) == (m <= 128)
        assert p.m_tiles * p.mt * 32 >= m and p.n_tiles * cols >= n and p.ct * 32 == cols
        assert scratch(m, n, k) >= p.splits * m * n * 4


class AttnPlan(C.Structure):
    _fields_ = [("nsplit", C.c_int), ("tiles_per_split", C.c_int), ("q_tiles", C.c_int), ("ct_wg", C.c_int)]


def attn_plan(dtype, hd, batch, rows, hq, hkv, keys):
    p = internal("attn_plan", *[C.c_int] * 7, restype=AttnPlan)(dtype, hd, batch, rows, hq, hkv, keys)
    return p.q_tiles, p.ct_wg, p.nsplit, p.tiles_per_split


@pytest.mark.parametrize("dtype,hd", [(binding.ESP_F32, 64), (binding.ESP_F32, 128), (binding.ESP_BF16, 64)])
def test_generic_attention_splits_grow_with_the_root_of_the_tiles(dtype, hd):
    """The generic kernel's merge walks the splits one after the other: with few rows a long cache is not cut into a key tile
    each (63 splits at 4000 keys took twice as long as 16), a short one is; many rows fill the chip without splits."""
    for keys, splits in [(0, 1), (60, 1), (64, 2), (188, 3), (319, 5), (1000, 8), (4000, 16), (16000, 32), (63999, 63)]:
        _, _, ns, tps = attn_plan(dtype, hd, 1, 1, 4, 2, keys)
        nt = (keys + 1 + 63) // 64
        assert ns == splits and (ns - 1) * tps < nt <= ns * tps, (keys, ns, tps)
    assert attn_plan(dtype, hd, 4, 300, 4, 2, 4000)[2] == 1


@pytest.mark.parametrize("batch,rows,keys,plan", [
    # not one split with four or more column tiles
    (2, 512, 64, (8, 8, 2, 5)), (5, 200, 600, (3, 9, 2, 7)), (3, 320, 256, (5, 8, 2, 5)), (8, 101, 256, (2, 7, 2, 3)), (8, 200, 8192, (3, 9, 4, 33)),
    # not two column tiles with every CU on a long split
    (3, 132, 1024, (3, 6, 3, 7)), (2, 101, 2048, (2, 7, 7, 5)), (1, 101, 4096, (2, 7, 14, 5)),
    (1, 68, 2048, (5, 2, 6, 6)), (1, 1, 2048, (1, 1, 17, 2)), (6, 200, 1024, (5, 5, 1, 20)), (5, 68, 64, (5, 2, 1, 3))])
def test_ring_attention_plan(batch, rows, keys, plan):
    """(workgroups per kv head and split, column tiles in each, splits, key tiles in each) of 32 query heads on 8 kv heads, at
    shapes where others that the plan has taken were measured to be 3 to 25 % slower."""
    assert attn_plan(binding.ESP_BF16, 128, batch, rows, 32, 8, keys) == plan


def test_ring_attention_plans_fit_their_workspace():
    """Whatever the plan, its partials fit what a context reserves for its largest batch and block."""
    c = C
    need = internal("attn_partial_floats", *[c.c_int] * 6, c.POINTER(AttnPlan), restype=c.c_size_t)
    bound = internal("attn_partial_floats_bound", *[c.c_int] * 6, restype=c.c_size_t)
    fn = internal("attn_plan", *[c.c_int] * 7, restype=AttnPlan)
    for dtype, hd, hq, hkv in [(binding.ESP_BF16, 128, 32, 8), (binding.ESP_BF16, 128, 16, 2), (binding.ESP_F32, 64, 4, 2)]:
        for batch in (1, 2, 5, 16):
            for rows in (1, 7, 50, 101, 320, 576):
                most = bound(dtype, batch, 576, hq, hkv, hd)
                for keys in (0, 300, 2048, 9000, 32768):
                    p = fn(dtype, hd, batch, rows, hq, hkv, keys)
                    assert 1 <= p.nsplit <= 64 and p.nsplit * p.tiles_per_split * 64 >= keys + rows
                    assert need(dtype, batch, rows, hq, hkv, hd, p) <= most, (dtype, batch, rows, keys)


@pytest.mark.parametrize("hkv,batch,rows,keys,shares", [
    # workgroups for three quarters of the CUs, and no more than two sequences to a share
    (8, 16, 132, 8192, 16), (8, 16, 1, 16384, 32), (8, 64, 1, 4096, 32), (4, 64, 1, 8192, 63), (2, 16, 200, 32768, 42),
    (1, 256, 1, 4000, 0), (1, 1024, 1, 4000, 0), (2, 64, 1, 8000, 0), (2, 64, 68, 8192, 0), (8, 128, 1, 4096, 0), (4, 128, 1, 8192, 0)])
def test_attention_shares(hkv, batch, rows, keys, shares):
    """Shares of a batch's attention, four query heads to a kv head, at shapes whose longest split takes 45 us and more."""
    plan = internal("attn_plan", *[C.c_int] * 7, restype=AttnPlan)(binding.ESP_BF16, 128, batch, rows, 4 * hkv, hkv, keys)
    n = internal("attn_shares", *[C.c_int] * 6, C.POINTER(AttnPlan))(binding.ESP_BF16, 128, batch, rows, 4 * hkv, hkv, plan)
    assert n == shares


@pytest.mark.parametrize("hd,batch,rows,heads,keys,splits,merges", [
    (64, 1, 60, 4, 128, 3, True), (64, 4, 20, 4, 128, 3, True), (64, 1, 20, 4, 1000, 8, True), (64, 1, 124, 4, 128, 4, True), (64, 4, 60, 4, 512, 3, True),
    (64, 1, 200, 4, 1000, 5, False), (64, 1, 400, 4, 128, 2, False), (64, 4, 20, 4, 512, 5, False), (64, 4, 124, 4, 16000, 2, False), (64, 1, 20, 4, 16000, 32, False),
    (64, 4, 400, 4, 4000, 1, True), (128, 1, 60, 4, 128, 3, True), (128, 4, 60, 4, 512, 3, False), (128, 1, 200, 4, 128, 3, False)])
def test_generic_attention_merges_where_all_workgroups_fit(hd, batch, rows, heads, keys, splits, merges):
    """Splits that are waves of one workgroup only where every (row, head) has its place on a CU at once, or there is one."""
    plan = internal("attn_plan", *[C.c_int] * 7, restype=AttnPlan)(binding.ESP_F32, hd, batch, rows, heads, 2, keys)
    assert plan.nsplit == splits
    assert internal("attn_generic_merges", C.c_int, C.POINTER(AttnPlan), C.c_int64, restype=C.c_bool)(hd, plan, batch * rows * heads) is merges
