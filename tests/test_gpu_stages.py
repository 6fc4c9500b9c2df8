"""Stage parity on the GPU: each C-ABI entry point against the oracle on the same seeded
inputs.  Integer / index work must be bit-exact; floating point within the stated tolerance
(row-wise max |diff| / max |oracle|: 2e-2 for bf16 inputs, 1e-4 for fp32)."""
import ctypes

import numpy as np
import pytest
import torch

from util import O, internal, oracle_model, small_shape, synth, to_np

pytestmark = pytest.mark.gpu

TOL = {"bf16": 2e-2, "f32": 1e-4}


@pytest.fixture(scope="module")
def B():
    from paper_2603_17942_amd import binding
    binding.load_library()
    assert torch.cuda.is_available(), "GPU tests need a GPU; there is no fallback path"
    return binding


def rel_err_rows(got, want):
    got, want = np.asarray(got, np.float64), np.asarray(want, np.float64)
    den = np.max(np.abs(want), axis=-1, keepdims=True)
    den[den == 0] = 1.0
    return float(np.max(np.abs(got - want) / den))


# ---------------------------------------------------------------------------------------- GEMM
@pytest.mark.parametrize("M,N,K", [(1, 32, 64), (5, 96, 64), (68, 384, 512), (33, 128, 4096), (97, 2048, 1024),
                                   (200, 640, 1024), (320, 512, 4096), (130, 6144, 512), (64, 1056, 256),
                                   (200, 256, 64), (160, 96, 128), (129, 32, 192), (1344, 512, 256)])
def test_gemm_bf16(B, M, N, K):
    print(f"gemm bf16 M={M} N={N} K={K}", flush=True)
    a = synth.normal_like((M, K), 1.0, 11, 0, "cuda", torch.bfloat16)
    w = synth.normal_like((N, K), 0.05, 11, 1, "cuda", torch.bfloat16)
    got = B.gemm(a, w).cpu().numpy()
    got_packed = B.gemm(a, B.pack_weight(w), packed=True).cpu().numpy()
    assert np.array_equal(got, got_packed)   # the streaming layout only moves bytes
    want = to_np(a) @ to_np(w).T            # fp64 on the same bf16 values
    # products of bf16 values are exact in fp32; only the accumulation order differs
    assert rel_err_rows(got, want) < 1e-5
    # split-K must not make a row depend on the other rows of the block (the split count is a
    # function of (N, K) within the <= 128-row tile class)
    if 1 < M <= 128:
        got1 = B.gemm(a[:1].contiguous(), w).cpu().numpy()
        assert np.array_equal(got1[0], got[0])


@pytest.mark.parametrize("chunks", [1, 5, 6, 7, 8, 9, 12, 13, 17, 26])
@pytest.mark.parametrize("M", [1, 64, 65, 128])
def test_gemm_bf16_ring_depth(B, M, chunks):
    """Reduction lengths below, at and above the depth of the operand ring of the small-row kernel: one
    group of 64-wide chunks, an exact number of groups, and a last group that is partly padding; N = 160 leaves the
    second column tile one live wave."""
    N, K = 160, 64 * chunks
    print(f"gemm bf16 ring M={M} N={N} K={K}", flush=True)
    a = synth.normal_like((M, K), 1.0, 12, 0, "cuda", torch.bfloat16)
    w = synth.normal_like((N, K), 0.05, 12, 1, "cuda", torch.bfloat16)
    got = B.gemm(a, B.pack_weight(w), packed=True).cpu().numpy()
    assert np.array_equal(got, B.gemm(a, w).cpu().numpy())      # same chunks in the same order
    assert rel_err_rows(got, to_np(a) @ to_np(w).T) < 1e-5      # fp32 sums of at most 1664 exact products


@pytest.mark.parametrize("M", [64, 65, 96, 128, 640, 641])
def test_gemm_bf16_cache_policy_edges(B, M):
    """Packed weights are loaded nontemporally, row-major ones the ordinary way, and both add in the same order (the row count up to
    which that is so: test_gemm_tiles_cache_policy_edge)."""
    N, K = 544, 512
    print(f"gemm bf16 cache policy M={M} N={N} K={K}", flush=True)
    a = synth.normal_like((M, K), 1.0, 14, 0, "cuda", torch.bfloat16)
    w = synth.normal_like((N, K), 0.05, 14, 1, "cuda", torch.bfloat16)
    wp = B.pack_weight(w)
    got = B.gemm(a, wp, packed=True).cpu().numpy()
    assert np.array_equal(got, B.gemm(a, w).cpu().numpy())
    assert rel_err_rows(got, to_np(a) @ to_np(w).T) < 1e-5      # fp32 sums of 512 exact products


def test_gemm_bf16_rows_beyond_4_gib(B):
    """Activations of more bytes than a 32-bit offset reaches (524288 rows of 4096): rows on both sides of that line, and the last."""
    M, N, K = 524288 + 333, 64, 4096
    print(f"gemm bf16 M={M} N={N} K={K}", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    a = torch.empty(M, K, dtype=torch.bfloat16, device="cuda").normal_(generator=g)
    w = torch.empty(N, K, dtype=torch.bfloat16, device="cuda").normal_(0, 0.05, generator=g)
    wp = B.pack_weight(w)
    got, first = B.gemm(a, wp, packed=True), B.gemm_argmax(a, wp)
    for rows in (slice(0, 300), slice(524288 - 300, 524288 + 300), slice(M - 300, M)):
        want = a[rows].double() @ w.double().T
        assert rel_err_rows(got[rows].cpu().numpy(), want.cpu().numpy()) < 1e-5      # fp32 sums of 4096 exact products
        assert torch.equal(first[rows].long(), got[rows].argmax(1))


def test_lists_of_rows_beyond_4_gib_are_refused(B):
    """The LM head reads its rows by a list, whose offsets have 32 bits: hidden states of more bytes are refused before anything is
    launched (a forward pass without the arg-max has no list)."""
    shape = small_shape(d_model=65536, n_q_heads=1, n_kv_heads=1, head_dim=64, d_ff=64, vocab=64, n_layers=1, dtype="bf16")
    batch, rows = 33, 1000                                   # 33000 rows of 128 KB
    mat = lambda r, c: torch.zeros(r, c, dtype=torch.bfloat16, device="cuda")   # noqa: E731
    d = shape.d_model
    w = {"embed": mat(64, d), "lm_head": mat(64, d), "final_norm": mat(1, d)[0], "layers": [dict(
        wq=mat(64, d), wk=mat(64, d), wv=mat(64, d), wo=mat(d, 64), w_gate=mat(64, d), w_up=mat(64, d), w_down=mat(d, 64),
        norm_attn=mat(1, d)[0], norm_mlp=mat(1, d)[0], q_norm=mat(1, 64)[0], k_norm=mat(1, 64)[0])]}
    eng = B.Engine(shape, w, batch, rows, 1088)
    blk = B.BlockBuffers(batch, rows, 1, 1)
    blk.upload_trees([[0]] * batch, [[-1]] * batch)
    eng.block_from_tree(blk)
    kv = B.KvCache(shape, [1088] * batch)
    hidden = torch.full((batch * rows, d), 3.0, dtype=torch.bfloat16, device="cuda")
    i32 = dict(dtype=torch.int32, device="cuda")
    zeros = torch.zeros(batch * rows, **i32)
    with pytest.raises(B.EspError) as e:
        eng.tree_forward(blk, mat(1, d), kv, hidden, zeros)
    assert e.value.code == 3
    with pytest.raises(B.EspError) as e:
        eng.mask_topk(blk, zeros, zeros, hidden, 4, torch.zeros(batch, 4, **i32), torch.zeros(batch, 4, device="cuda"), zeros)
    assert e.value.code == 3
    assert bool((hidden[-1] == 3).all()) and not bool(kv.k.any())
    eng.close()


class GemmPlan(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int) for n in ("splits", "mt", "nb", "m_tiles", "n_tiles", "wm")]


@pytest.mark.parametrize("M,N,K,live", [(161, 320, 1024, 1), (161, 320, 1024, 96), (192, 544, 512, 97), (192, 320, 2048, 192), (192, 320, 512, 0),
                                        (129, 256, 2048, 100), (320, 512, 4096, 160), (320, 512, 4096, 161), (640, 256, 4096, 481), (1344, 256, 2048, 700)])
def test_gemm_bf16_live_rows(B, M, N, K, live):
    """Packed rows of a batch on every tile above 128 rows, in several split-K parts: the rows that are there get what they get
    alone (each part's sums run over K in the same order), parts keep the stride of all M rows, no other row is written."""
    c = ctypes
    plan = internal("gemm_plan", *[c.c_int] * 4, restype=GemmPlan)(B.ESP_BF16, M, N, K)
    fn = internal("launch_gemm", c.c_void_p, c.c_int, c.c_void_p, c.c_void_p, c.c_void_p, c.c_void_p, *[c.c_int] * 3, c.POINTER(GemmPlan),
                  c.c_bool, c.c_int, c.c_void_p)
    print(f"gemm live rows M={M} N={N} K={K} live={live} mt={plan.mt} splits={plan.splits}", flush=True)
    assert plan.nb == 2 and (plan.splits > 1 or K < 1024)
    a = synth.normal_like((M, K), 1.0, 15, 0, "cuda", torch.bfloat16)
    wp = B.pack_weight(synth.normal_like((N, K), 0.05, 15, 1, "cuda", torch.bfloat16))
    n = torch.tensor([live], dtype=torch.int32, device="cuda")
    got, want = (torch.full((plan.splits, M, N), -7.0, device="cuda") for _ in range(2))
    for out, m_live in ((want, None), (got, n.data_ptr())):
        assert fn(torch.cuda.current_stream().cuda_stream, B.ESP_BF16, a.data_ptr(), None, wp.data_ptr(), out.data_ptr(), M, N, K, plan, True, 0,
                  m_live) == 0
    assert torch.equal(got[:, :live], want[:, :live]) and bool((got[:, live:] == -7).all())
    assert rel_err_rows(want.sum(0).cpu().numpy(), B.gemm(a, wp, packed=True).cpu().numpy()) < 1e-6


@pytest.mark.parametrize("M,N,K", [(1, 512, 128), (68, 4096, 256), (128, 1056, 192), (129, 768, 256), (320, 4096, 512),
                                   (200, 2048, 128), (1344, 1280, 256), (700, 33 * 32, 192), (180, 512, 64)])
def test_gemm_argmax_epilogue(B, M, N, K):
    """Sec. 2 Eq. 3: the greedy choice per row, taken in the LM-head GEMM's epilogue (small-tile kernel up
    to 128 rows, large-tile kernel above).  Against the same GEMM's written logits the arg-max must be
    exact, lowest index on ties; planted exact ties (duplicated weight rows) make the tie rule visible,
    also across column tiles and across the waves of a workgroup."""
    print(f"gemm arg-max M={M} N={N} K={K}", flush=True)
    a = synth.normal_like((M, K), 1.0, 13, 0, "cuda", torch.bfloat16)
    w = synth.normal_like((N, K), 0.05, 13, 1, "cuda", torch.bfloat16)
    # duplicate the winning weight row of a few rows at a higher and a lower index
    logits0 = B.gemm(a, w)
    win = logits0.argmax(dim=1)
    for r in range(0, M, max(1, M // 7)):
        n = int(win[r])
        for other in ((n + 40) % N, (n + N - 300) % N, (n + 129) % N):
            w[other] = w[n]
    wp = B.pack_weight(w)
    logits = B.gemm(a, wp, packed=True).cpu().numpy()
    want = np.array([O.argmax_lowest(row) for row in logits], dtype=np.int32)
    got = B.gemm_argmax(a, wp).cpu().numpy()
    assert np.array_equal(got, want), np.nonzero(got != want)[0][:8]
    ties = int(sum((logits[i] == logits[i].max()).sum() > 1 for i in range(M)))
    assert ties >= 1


@pytest.mark.parametrize("M,ff,K,live,tile", [
    (353, 14336, 64, None, 1), (512, 14336, 128, None, 1), (511, 14336, 704, None, 1), (1024, 14336, 192, None, 1), (993, 14368, 64, None, 1),
    (576, 12288, 64, None, 2), (545, 12288, 128, None, 2), (571, 12288, 1088, None, 2), (570, 12320, 192, None, 2),
    (700, 14336, 192, 520, 0), (700, 14336, 64, 1, 0),                                               # live rows of a batch, one tile
    (512, 14336, 192, 385, 1), (512, 14336, 64, 1, 1), (512, 14336, 64, 256, 1), (512, 14336, 64, 257, 1), (512, 14336, 64, 512, 1),
    (640, 14336, 192, 0, 1), (640, 14336, 192, 300, 1), (640, 14336, 192, 512, 1), (640, 14336, 192, 640, 1),   # two tiles launched
    (640, 14336, 192, 513, 0), (640, 14336, 64, 1, 0), (640, 14336, 64, 640, 0),
    (560, 12288, 128, 1, 2), (560, 12288, 128, 193, 2), (560, 12288, 128, 560, 2), (560, 12288, 128, 512, 1),
    (640, 12288, 128, 500, 1), (640, 12288, 128, 570, 2), (640, 12288, 128, 640, 0), (760, 12288, 128, 760, 0),
    (320, 14336, 128, None, 0), (640, 1056, 64, None, 0), (1, 96, 64, None, 0)])
def test_gemm_swiglu(B, M, ff, K, live, tile):
    """The gate/up projection with the SwiGLU in its epilogue, on gemm_plan's tiles (tile 0) and on the wide ones of 256 x 256
    (1) and 192 x 320 (2): remainders of rows and of columns, one to many chunks of K, an odd number of them, and of a batch
    any number of live rows.  The tile is the one that the sizes ask for, or, in a batch that several are launched for, the
    one that is handed the rows, so a case that would run on another fails.  The products are exact in fp32; the sums'
    order and the hardware's exp and reciprocal (1 ulp each) leave 2e-6 of the row's largest value before the bf16 rounding
    of half an ulp of eight bits (2^-8).  Rows that are not live stay as they were."""
    c = ctypes
    fn = internal("launch_gemm_swiglu", *[c.c_void_p] * 4, *[c.c_int] * 3, c.c_void_p)
    tiles = internal("gate_up_tiles", c.c_int, c.c_int, c.c_int, c.c_void_p, c.c_bool, restype=c.c_uint)
    print(f"swiglu M={M} ff={ff} K={K} live={live} tile={tile}", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(M + ff + K)
    a = torch.randn(M, K, device="cuda", generator=g).bfloat16()
    wg, wu = (torch.randn(ff, K, device="cuda", generator=g).mul_(K ** -0.5).bfloat16() for _ in range(2))
    w = torch.stack([wg.view(ff // 32, 32, K), wu.view(ff // 32, 32, K)], 1).reshape(2 * ff, K).contiguous()   # blocks of 32 alternate
    packed = B.pack_weight(w)
    act = torch.full((M + 1, ff), -7.0, dtype=torch.bfloat16, device="cuda")
    launched = tiles(M, ff, K, act.data_ptr(), live is not None)
    assert launched == 1 << tile or (live is not None and launched & (1 << tile)), bin(launched)
    # rows and tree rows of the batch, then what each tile computes
    counts = None if live is None else torch.tensor([live, 0] + [live if t == tile else 0 for t in range(3)], dtype=torch.int32, device="cuda")
    assert fn(torch.cuda.current_stream().cuda_stream, a.data_ptr(), packed.data_ptr(), act.data_ptr(), M, ff, K,
              None if counts is None else counts.data_ptr()) == 0
    rows = M if live is None else live
    if rows:
        gate, up = a[:rows].double() @ wg.double().T, a[:rows].double() @ wu.double().T
        want = gate / (1 + torch.exp(-gate)) * up
        err = (act[:rows].double() - want).abs()
        assert bool((err <= want.abs() * 2.0 ** -8 + 2e-6 * want.abs().amax(1, keepdim=True)).all()), float((err / want.abs().clamp_min(1e-9)).max())
    assert bool((act[rows:] == -7).all())


ROW_TILES = 12                                            # the first are for up to 128 rows; 32-row and 32-column tiles
GEMM_TILES = [(rt, ct) for rt in (1, 2, 3, 4) for ct in (2, 4, 6)] + [
    (3, 8), (4, 4), (4, 6), (4, 8), (5, 6), (5, 8), (6, 6), (6, 8), (6, 10), (8, 6), (8, 8)]


class TilePlan(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int) for n in ("splits", "mt", "nb", "m_tiles", "n_tiles", "ct")]


class TileGemm(ctypes.Structure):
    _fields_ = ([(n, ctypes.c_void_p) for n in ("A", "a_rows", "W", "out")] + [(n, ctypes.c_int) for n in ("M", "N", "K", "splits", "tile")] +
                [("draw_pos", ctypes.c_void_p), ("seed", ctypes.c_uint32), ("m_live", ctypes.c_void_p), ("pairs", ctypes.c_void_p)])


@pytest.mark.parametrize("tile", range(len(GEMM_TILES)))
@pytest.mark.parametrize("M,N,K,splits,live", [
    (129, 544, 64, 1, None), (257, 352, 128, 1, None), (160, 1056, 192, 1, None), (300, 96, 256, 1, None), (192, 256, 320, 1, None),
    (513, 416, 704, 3, None), (256, 640, 512, 8, None), (320, 320, 1088, 2, None), (385, 192, 1536, 1, None),
    (200, 320, 1088, 2, 77), (700, 288, 448, 1, 513), (300, 256, 384, 1, 1), (300, 256, 384, 1, 0), (1, 96, 64, 1, None), (33, 320, 1600, 1, None),
    (128, 544, 448, 7, None)])
def test_gemm_tiles(B, tile, M, N, K, splits, live):
    """Every tile at remainders of rows and columns, from one chunk of K (fewer than the loads reach ahead) to many, in
    parts, and with rows of a batch that are not there: bit for bit what the kernel for row-major weights gives, which adds in
    the same order; with one part also its arg-max and SwiGLU epilogues against the same logits (ties: the lowest column).
    The tiles for up to 128 rows also as several row tiles."""
    c = ctypes
    rt, ct = GEMM_TILES[tile]
    print(f"tile {rt}x{ct} M={M} N={N} K={K} splits={splits} live={live}", flush=True)
    gemm = internal("launch_gemm", c.c_void_p, c.c_int, c.c_void_p, c.c_void_p, c.c_void_p, c.c_void_p, *[c.c_int] * 3, c.POINTER(TilePlan),
                    c.c_bool, c.c_int, c.c_void_p)
    a = synth.normal_like((M, K), 1.0, 16, 0, "cuda", torch.bfloat16)
    w = synth.normal_like((N, K), K ** -0.5, 16, 1, "cuda", torch.bfloat16)
    w[N // 2:] = w[:N - N // 2]                              # every column twice: ties of the arg-max
    wp = B.pack_weight(w)
    n = None if live is None else torch.tensor([live], dtype=torch.int32, device="cuda")
    st = torch.cuda.current_stream().cuda_stream
    plan = TilePlan(splits, rt, 1 if tile < ROW_TILES else 2, (M + 32 * rt - 1) // (32 * rt), (N // 32 + ct - 1) // ct, ct)
    got, want = (torch.full((splits, M, N), -7.0, device="cuda") for _ in range(2))
    assert gemm(st, B.ESP_BF16, a.data_ptr(), None, wp.data_ptr(), got.data_ptr(), M, N, K, plan, True, 0, None if n is None else n.data_ptr()) == 0
    ref_plan = TilePlan(splits, 1, 1, (M + 31) // 32, (N + 127) // 128, 4)   # row-major weights: one row tile a workgroup
    assert gemm(st, B.ESP_BF16, a.data_ptr(), None, w.data_ptr(), want.data_ptr(), M, N, K, ref_plan, False, 0, None) == 0
    rows = M if live is None else live
    assert torch.equal(got[:, :rows], want[:, :rows]) and bool((got[:, rows:] == -7).all())
    ref = a.double() @ w.double().T
    assert float((want.double().sum(0) - ref).abs().max()) <= 2e-5 * float(ref.abs().max())   # fp32 sums of up to 1536 exact products
    if splits > 1 or not rows:
        return
    n_live = None if n is None else n.data_ptr()
    for both in (False, True) if tile < ROW_TILES else (False,):
        pairs, logits = torch.full((plan.n_tiles, M, 2), -7.0, device="cuda"), torch.full((M, N), -7.0, device="cuda")
        g = TileGemm(a.data_ptr(), None, wp.data_ptr(), logits.data_ptr(), M, N, K, 1, tile, None, 0, n_live, pairs.data_ptr())
        assert internal("launch_gemm_tile_both" if both else "launch_gemm_tile_argmax", c.c_void_p, c.POINTER(TileGemm))(st, g) == 0
        for t in range(plan.n_tiles):
            cols = want[0, :rows, t * 32 * ct:(t + 1) * 32 * ct]
            best = cols.amax(1)
            assert torch.equal(pairs[t, :rows, 0], best)
            first = (cols == best[:, None]).int().argmax(1) + t * 32 * ct
            assert torch.equal(pairs[t, :rows, 1].contiguous().view(torch.int32).long(), first)
        assert bool((pairs[:, rows:] == -7).all())
        assert torch.equal(logits[:rows], want[0, :rows]) if both else bool((logits == -7).all())
    if N % 64 == 0:
        act = torch.full((M + 1, N // 2), -7.0, dtype=torch.bfloat16, device="cuda")
        for offset in (0, 1):                                # results on and off the 16-byte alignment of the wide stores
            flat = act.view(-1)[offset:offset + M * (N // 2)]
            g.out = flat.data_ptr()
            assert internal("launch_gemm_tile_swiglu", c.c_void_p, c.POINTER(TileGemm))(st, g) == 0
            blocks = want[0, :rows].double().view(rows, N // 64, 2, 32)
            gate, up = blocks[:, :, 0].reshape(rows, -1), blocks[:, :, 1].reshape(rows, -1)
            r = gate / (1 + torch.exp(-gate)) * up
            # exp and reciprocal to 1 ulp each, then the rounding to bf16
            res = flat.view(M, N // 2)[:rows].double()
            assert bool(((res - r).abs() <= r.abs() * (2.0 ** -8 + 1e-6) + 1e-30).all())
            assert bool((flat.view(M, N // 2)[rows:] == -7).all()) if offset == 0 else True


@pytest.mark.parametrize("tile", range(ROW_TILES, len(GEMM_TILES)))
@pytest.mark.parametrize("M", [2400, 2401])
def test_gemm_tiles_cache_policy_edge(B, tile, M):
    """Both sides of the row count up to which weights are loaded nontemporally, every tile above 128 rows: one product on all tiles, bit for bit
    what the kernel for row-major weights gives, and its arg-max and SwiGLU epilogues."""
    c, (rt, ct), N, K = ctypes, GEMM_TILES[tile], 256, 192
    print(f"tile {rt}x{ct} M={M}", flush=True)
    a = synth.normal_like((M, K), 1.0, 18, 0, "cuda", torch.bfloat16)
    w = synth.normal_like((N, K), K ** -0.5, 18, 1, "cuda", torch.bfloat16)
    wp, want, st = B.pack_weight(w), B.gemm(a, w), torch.cuda.current_stream().cuda_stream
    got, pairs, n_tiles = torch.full((M, N), -7.0, device="cuda"), torch.full((8, M, 2), -7.0, device="cuda"), (N // 32 + ct - 1) // ct
    act = torch.full((M, N // 2), -7.0, dtype=torch.bfloat16, device="cuda")
    for name, out in (("out", got), ("argmax", got), ("swiglu", act)):
        g = TileGemm(a.data_ptr(), None, wp.data_ptr(), out.data_ptr(), M, N, K, 1, tile, None, 0, None, pairs.data_ptr())
        assert internal(f"launch_gemm_tile_{name}", c.c_void_p, c.POINTER(TileGemm))(st, g) == 0
    assert torch.equal(got, want)
    best = torch.stack([want[:, 32 * ct * t:32 * ct * (t + 1)].amax(1) for t in range(n_tiles)])
    assert torch.equal(pairs[:n_tiles, :, 0], best)
    blocks = want.double().view(M, N // 64, 2, 32)
    gate, up = blocks[:, :, 0].reshape(M, -1), blocks[:, :, 1].reshape(M, -1)
    r = gate / (1 + torch.exp(-gate)) * up
    assert bool(((act.double() - r).abs() <= r.abs() * (2.0 ** -8 + 1e-6) + 1e-30).all())   # exp and reciprocal to 1 ulp, then bf16


def test_arg_max_epilogue_is_no_slower_than_writing_the_logits(B):
    """2048 workgroups of 256 x 256 with two chunks of K: the arg-max leaves 8 bytes a row and workgroup where the logits are 537 MB (the
    epilogue took longer with the noise of a draw as a branch inside its loop)."""
    c, M, N, K, tile = ctypes, 2048, 65536, 128, len(GEMM_TILES) - 1
    a = synth.normal_like((M, K), 1.0, 19, 0, "cuda", torch.bfloat16)
    wp = B.pack_weight(synth.normal_like((N, K), K ** -0.5, 19, 1, "cuda", torch.bfloat16))
    out, pairs = torch.empty(M, N, device="cuda"), torch.empty(N // 256, M, 2, device="cuda")
    best = {}
    for name in ("out", "argmax"):
        g = TileGemm(a.data_ptr(), None, wp.data_ptr(), out.data_ptr(), M, N, K, 1, tile, None, 0, None, pairs.data_ptr())
        fn = internal(f"launch_gemm_tile_{name}", c.c_void_p, c.POINTER(TileGemm))
        times = []
        for _ in range(12):
            e = [torch.cuda.Event(enable_timing=True) for _ in (0, 1)]
            e[0].record()
            assert fn(torch.cuda.current_stream().cuda_stream, g) == 0
            e[1].record()
            e[1].synchronize()
            times.append(e[0].elapsed_time(e[1]))
        best[name] = min(times)
    print(f"out {best['out']:.3f} ms, arg-max {best['argmax']:.3f} ms", flush=True)
    assert best["argmax"] < 0.8 * best["out"], best


@pytest.mark.parametrize("M,N,K", [(1, 1, 1), (13, 4096, 256), (52, 688, 256), (52, 256, 688), (70, 130, 77)])
def test_gemm_f32(B, M, N, K):
    print(f"gemm f32 M={M} N={N} K={K}", flush=True)
    a = synth.normal_like((M, K), 1.0, 12, 0, "cuda", torch.float32)
    w = synth.normal_like((N, K), 0.05, 12, 1, "cuda", torch.float32)
    got = B.gemm(a, w).cpu().numpy()
    want = to_np(a) @ to_np(w).T
    assert rel_err_rows(got, want) < 1e-5


# ---------------------------------------------------------------------------------------- Top-K
@pytest.mark.parametrize("offset", (0, 1))
@pytest.mark.parametrize("M,ff,K", [(1, 1, 1), (31, 15, 7), (32, 16, 64), (33, 17, 77), (60, 688, 256), (13, 130, 1028)])
def test_gemm_swiglu_f32(B, M, ff, K, offset):
    """Gate and up features side by side in a tile: the logits are those of the plain product bit for bit, so only the
    activation's own roundings are left (exp 2, sum 1/2, quotient 2.5, product 1/2 units of 2^-23).  Operands on and off a 16-byte
    boundary, remainders of rows, features and K, nothing written behind the last feature."""
    print(f"gemm swiglu f32 M={M} ff={ff} K={K} offset={offset}", flush=True)
    a, w = (torch.zeros(n * K + offset, device="cuda")[offset:].view(n, K) for n in (M, 2 * ff))
    a.copy_(synth.normal_like((M, K), 1.0, 13, 0, "cuda", torch.float32))
    w.copy_(synth.normal_like((2 * ff, K), K ** -0.5, 13, 1, "cuda", torch.float32))
    act = torch.full((M * ff + 1,), -7.0, device="cuda")
    c = ctypes
    run = internal("launch_gemm_swiglu_f32", c.c_void_p, c.c_void_p, c.c_void_p, c.c_void_p, c.c_int, c.c_int, c.c_int)
    assert run(torch.cuda.current_stream().cuda_stream, a.data_ptr(), w.data_ptr(), act.data_ptr(), M, ff, K) == 0
    gate, up = B.gemm(a, w).double().split(ff, dim=1)
    want = gate / (1 + torch.exp(-gate)) * up
    got = act[:-1].view(M, ff).double()
    assert bool(((got - want).abs() <= 5.5 * 2.0 ** -23 * want.abs() + 1e-37).all()) and float(act[-1]) == -7


def check_topk(ids, ps, logits, kp, tol):
    """Oracle comparison with the near-tie rule: position j must match where the oracle's gap
    between ranks j and j+1 exceeds the band; probabilities within tolerance everywhere."""
    for r in range(logits.shape[0]):
        want_ids, want_ps = O.softmax_topk(logits[r], kp + 1)
        np.testing.assert_allclose(ps[r], want_ps[:kp], rtol=1e-4, atol=1e-9)
        for j in range(kp):
            gap_ok = (want_ps[j] - want_ps[j + 1]) > tol * want_ps[j] if j + 1 < len(want_ps) else True
            prev_ok = j == 0 or (want_ps[j - 1] - want_ps[j]) > tol * want_ps[j - 1]
            if gap_ok and prev_ok:
                assert ids[r, j] == want_ids[j], (r, j)
        assert len(set(ids[r].tolist())) == kp


@pytest.mark.parametrize("rows,vocab,kp", [(1, 211, 5), (4, 4096, 6), (3, 128256, 10), (5, 2048, 32),
                                           (2, 151936, 12), (7, 2049, 4), (65, 128256, 10), (66, 128256, 31)])
def test_softmax_topk(B, rows, vocab, kp):
    print(f"topk rows={rows} vocab={vocab} kp={kp}", flush=True)
    logits = synth.normal_like((rows, vocab), 2.0, 21, rows, "cuda", torch.float32)
    ids, ps = B.softmax_topk(logits, kp)
    check_topk(ids.cpu().numpy(), ps.cpu().numpy(), to_np(logits), kp, 1e-6)


def test_softmax_topk_exact_ties_take_lowest_id(B):
    logits = torch.zeros((2, 5000), dtype=torch.float32)
    logits[0, [4000, 7, 2100]] = 3.0
    logits[0, [9, 4999]] = 1.5
    logits[1, :] = -2.0                      # all equal: ids 0..kp-1
    ids, ps = B.softmax_topk(logits.cuda(), 6)
    assert ids[0].tolist() == [7, 2100, 4000, 9, 4999, 0]
    assert ids[1].tolist() == [0, 1, 2, 3, 4, 5]
    want = O.softmax_topk(logits[0].numpy(), 6)
    assert ids[0].tolist() == want[0].tolist()
    np.testing.assert_allclose(ps[0].cpu().numpy(), want[1], rtol=1e-5)


def test_softmax_topk_adversarial_orders_and_masked_logits(B):
    """Rows that defeat the streaming kernel's shortcuts: strictly ascending values (every block
    raises the bound), descending values, -inf entries, fewer finite logits than Kp, Kp == vocab,
    and many rows (one wave per row, several segments per row for few rows)."""
    vocab, kp = 20000, 9
    asc = torch.arange(vocab, dtype=torch.float32) * 1e-3
    desc = asc.flip(0)
    holes = synth.normal_like((vocab,), 1.0, 31, 0, "cpu", torch.float32).clone()
    holes[::3] = float("-inf")
    few = torch.full((vocab,), float("-inf"))
    few[[5, 17000, 9999]] = torch.tensor([0.5, 2.0, -1.0])
    logits = torch.stack([asc, desc, holes, few]).cuda()
    ids, ps = B.softmax_topk(logits, kp)
    ids, ps = ids.cpu().numpy(), ps.cpu().numpy()
    for r in range(3):
        want_ids, want_ps = O.softmax_topk(logits[r].cpu().numpy(), kp)
        assert ids[r].tolist() == want_ids.tolist()
        np.testing.assert_allclose(ps[r], want_ps, rtol=1e-4)
    assert ids[3, :3].tolist() == [17000, 5, 9999] and np.all(ids[3, 3:] == -1) and np.all(ps[3, 3:] == 0)
    np.testing.assert_allclose(ps[3, :3].sum(), 1.0, rtol=1e-5)
    small = synth.normal_like((2, 8), 1.0, 32, 0, "cuda", torch.float32)
    ids, ps = B.softmax_topk(small, 8)
    for r in range(2):
        want_ids, want_ps = O.softmax_topk(to_np(small)[r], 8)
        assert ids[r].tolist() == want_ids.tolist()
        np.testing.assert_allclose(ps[r].cpu().numpy(), want_ps, rtol=1e-5)
    many = synth.normal_like((700, 4100), 2.0, 33, 0, "cuda", torch.float32)
    ids, ps = B.softmax_topk(many, 10)
    check_topk(ids.cpu().numpy(), ps.cpu().numpy(), to_np(many), 10, 1e-6)


@pytest.mark.parametrize("rows,vocab,kp", [(1, 2048, 10), (3, 32000, 10), (70, 4100, 31), (2, 151936, 5)])
def test_softmax_topk_finite_masks(B, rows, vocab, kp):
    """Large finite masks that fill every logit of one lane (four columns of each 256), whole ranges of the row,
    or all but a few columns; rows without a positive value, with both zeros, and with values to 1e31 (ids only)."""
    print(f"topk masks rows={rows} vocab={vocab} kp={kp}", flush=True)
    col = np.arange(vocab)
    lane = (col // 4) % 64 == 5
    base = to_np(synth.normal_like((rows, vocab), 2.0, 23, rows, "cpu", torch.float32)).astype(np.float32)
    lowest = np.finfo(np.float32).min
    kinds = {"lane": lambda v: np.where(lane, -1e9, v), "lane, lowest": lambda v: np.where(lane, lowest, v),
             "row, lowest": lambda v: np.where(col > 0, lowest, v), "half, 1e30": lambda v: np.where(col < vocab // 2, -1e30, v),
             "tail": lambda v: np.where(col >= vocab - 300, -1e9, v), "few left": lambda v: np.where(col >= kp + 3, -1e9, v),
             "negative": lambda v: -np.abs(v) - 1, "relu": lambda v: np.maximum(v, -0.0),
             "spread": lambda v: np.where(col % 97 == 0, v * 1e30, v)}
    for name, f in kinds.items():
        logits = f(base).astype(np.float32)
        ids, ps = B.softmax_topk(torch.as_tensor(logits).cuda(), kp)
        ids, ps = ids.cpu().numpy(), ps.cpu().numpy()
        for r in range(0, rows, 23):
            want_ids = np.lexsort((col, -logits[r].astype(np.float64)))[:kp]    # the oracle ties what underflows to 0
            _, want_ps = O.softmax_topk(logits[r], kp)
            assert ids[r].tolist() == want_ids.tolist(), (name, r)
            if name != "spread":
                np.testing.assert_allclose(ps[r], want_ps, rtol=1e-5, atol=1e-30, err_msg=name)


def test_softmax_topk_ties_across_blocks(B):
    """Equal values in later blocks of a segment do not displace listed ones, a larger one does, and equal ones of the
    same block go by id; negative values, zeros of both signs, infinity among them."""
    rows, vocab, kp = 300, 20000, 6                        # several blocks a wave
    for value in (-3.5, 0.0, -0.0, 2.0, -1e9):
        logits = torch.full((rows, vocab), value)
        logits[1::3, 9000] = value + abs(value) * 0.25 + 1
        logits[2::3, [17000, 16900]] = value + abs(value) * 0.25 + 1
        logits[2::3, 5] = -0.0 if value == 0 else value
        ids, ps = B.softmax_topk(logits.cuda(), kp)
        assert ids[0].tolist() == [0, 1, 2, 3, 4, 5]
        assert ids[1].tolist() == [9000, 0, 1, 2, 3, 4]
        assert ids[2].tolist() == [16900, 17000, 0, 1, 2, 3]
        assert bool((ids[3:] == ids[:3].repeat(rows // 3 - 1, 1)).all())
    few = torch.full((rows, vocab), float("-inf"))
    few[:, [19000, 18999, 3000]] = torch.finfo(torch.float32).min
    ids, _ = B.softmax_topk(few.cuda(), kp)
    assert bool((ids == torch.tensor([3000, 18999, 19000, -1, -1, -1], device="cuda", dtype=torch.int32)).all())


def test_softmax_topk_nan_row_says_so(B):
    """A NaN among the logits makes the row's probabilities NaN wherever it lies, also far from the row's maximum;
    other rows are untouched."""
    logits = synth.normal_like((6, 32000), 2.0, 24, 0, "cpu", torch.float32).clone()
    want = O.softmax_topk(logits[5].numpy(), 8)
    logits[:4, 11] = 400.0
    logits[0, 0], logits[1, 31999], logits[2, 5000], logits[3, 17] = (float("nan"),) * 4
    ids, ps = B.softmax_topk(logits.cuda(), 8)
    assert bool(torch.isnan(ps[:4]).all()) and not bool(torch.isnan(ps[4:]).any())
    assert ids[5].tolist() == want[0].tolist()


def test_softmax_topk_never_hands_out_more_than_one(B):
    """Rows with all but a vanishing share of the probability on one token (maxima 15 to 40 over a floor of -30):
    the first probability is 1 to rounding and never above it, and the tree built from such lists is one."""
    rows, vocab, kp = 256, 4096, 10
    top = torch.linspace(15.0, 40.0, rows)
    logits = torch.full((rows, vocab), -30.0) + synth.normal_like((rows, vocab), 1.0, 22, 0, "cpu", torch.float32)
    logits[torch.arange(rows), (torch.arange(rows) * 37) % vocab] = top
    ids, ps = B.softmax_topk(logits.cuda(), kp)
    ids, ps = ids.cpu().numpy(), ps.cpu().numpy()
    assert ids[:, 0].tolist() == ((np.arange(rows) * 37) % vocab).tolist()
    # round(m log2 e) is off by at most half a unit in the last place of values below 64, 2^-19, i.e. 1.33e-6 of the
    # term; the exponentials and the division add 3 * 2^-24 each at most
    assert ps.max() <= 1.0 and ps[:, 0].min() > 1 - 2e-6
    check_topk(ids[::16], ps[::16], logits[::16].numpy(), kp, 1e-6)
    for r in range(0, rows, 4):
        O.build_prune_tree(O.TreeParams(B=64, k=4, K=8, expand_width=0), ids[r:r + 4], ps[r:r + 4], 1, n_depths=4)


# ---------------------------------------------------------------------------------------- engine fixture
@pytest.fixture(scope="module")
def tiny_engine(B):
    shape = small_shape(d_model=128, n_q_heads=4, n_kv_heads=2, head_dim=64, d_ff=176, vocab=517, n_layers=2)
    w = synth.make_weights(shape, seed=3, unit_gains=False)
    eng = B.Engine(shape, w, max_batch=3, max_rows_per_seq=640, max_kv_len=2048)
    yield shape, w, eng
    eng.close()


# ---------------------------------------------------------------------------------------- block descriptor
def bits_to_matrix(anc_row_words, n):
    out = np.zeros(n, dtype=bool)
    for c in range(n):
        out[c] = (int(anc_row_words[c // 64]) >> (c % 64)) & 1
    return out


def check_block(blk, b, tok, par, k, layout):
    ob = O.make_block(tok, par, k, layout)
    r0 = b * blk.rows_per_seq
    R = ob.n_rows
    assert int(blk.n_rows[b]) == R and int(blk.n_nodes[b]) == len(tok)
    sl = slice(r0, r0 + R)
    assert blk.depth[sl].tolist() == ob.depth.tolist()
    assert blk.mask_j[sl].tolist() == ob.mask_j.tolist()
    assert blk.attach[sl].tolist() == ob.attach.tolist()
    assert blk.tok[r0:r0 + len(tok)].tolist() == [int(t) for t in tok]
    assert all(t == -1 for t in blk.tok[r0 + len(tok):r0 + R].tolist())
    anc = blk.anc[sl].cpu().numpy().astype(np.uint64)
    for r in range(R):
        assert np.array_equal(bits_to_matrix(anc[r], R), ob.visible[r]), r
    return ob


@pytest.mark.parametrize("k,layout,n_nodes", [(0, 0, 7), (3, 0, 13), (4, 0, 64), (4, 1, 64), (5, 0, 96), (2, 1, 1),
                                              (1, 0, 1), (4, 0, 128)])
def test_block_from_tree(B, tiny_engine, k, layout, n_nodes):
    shape, w, eng = tiny_engine
    print(f"block_from_tree k={k} layout={layout} n={n_nodes}", flush=True)
    rows = n_nodes * (k + 1) if layout == 0 else n_nodes + k
    blk = B.BlockBuffers(2, min(rows + 3, 640), k, layout)
    t0, p0 = synth.make_random_tree(n_nodes, max(k, 1) if k else 6, shape.vocab, seed=30 + n_nodes)
    t1, p1 = synth.make_random_tree(max(1, n_nodes // 2), max(k, 1) if k else 6, shape.vocab, seed=31)
    blk.upload_trees([t0.tolist(), t1.tolist()], [p0.tolist(), p1.tolist()])
    eng.block_from_tree(blk)
    assert eng.device_status() == 0
    check_block(blk, 0, t0.numpy(), p0.numpy(), k, layout)
    check_block(blk, 1, t1.numpy(), p1.numpy(), k, layout)


def test_block_from_tree_rejects_malformed_tree(B, tiny_engine):
    shape, w, eng = tiny_engine
    blk = B.BlockBuffers(2, 24, 1, 0)
    blk.upload_trees([[1, 2, 3], [4, 5, 6, 7]], [[-1, 0, 2], [-1, 0, 1, 1]])   # seq 0: parent not before child
    eng.block_from_tree(blk)
    assert eng.device_status() & B.DEV_BAD_TREE
    assert int(blk.n_rows[0]) == 0 and int(blk.n_rows[1]) == 8
    assert eng.device_status() == 0   # sticky word was cleared by the read


@pytest.mark.parametrize("n", [64, 65, 513, 1024])
def test_block_from_tree_long_chains(B, tiny_engine, n):
    """Prompt chains and deep random trees across the 64-node groups, up to the largest block."""
    shape, w, _ = tiny_engine
    eng = B.Engine(shape, w, 2, n, 2 * n)
    rng = np.random.default_rng(n)
    chain = [-1] + list(range(n - 1))
    deep = [-1] + [int(rng.integers(max(0, i - 3), i)) for i in range(1, n)]
    blk = B.BlockBuffers(2, n, 0, 0)
    blk.upload_trees([[1] * n, [2] * n], [chain, deep])
    eng.block_from_tree(blk)
    assert eng.device_status() == 0
    for b, par in enumerate((chain, deep)):
        check_block(blk, b, np.full(n, b + 1), np.asarray(par), 0, 0)


@pytest.mark.parametrize("Bn,k,K,kp", [(256, 2, 32, 32), (256, 3, 12, 12), (200, 3, 10, 12), (256, 8, 2, 32), (65, 5, 8, 10),
                                         (1, 2, 4, 6)])
def test_build_prune_tree_large_and_smallest(B, tiny_engine, Bn, k, K, kp):
    """More candidates than threads of the builder (its threshold search), more than that holds in registers
    ((256, 3, 12, 12): 1871), lists longer than what a node takes of them, the largest tree and the root alone."""
    shape, w, eng = tiny_engine
    rng = np.random.default_rng(Bn)
    ids, ps = random_lists(rng, k, kp, 500)
    rows = Bn + k
    nxt = B.BlockBuffers(1, rows, k, 1)
    emit = np.zeros((1, B.MAX_MASKS + 1), dtype=np.int32)
    emit[0, 0] = 501
    dev = lambda a: torch.as_tensor(a).cuda()
    one = np.array([1], dtype=np.int32)
    eng.build_prune_tree(B.tree_params(Bn, k, K, 0, True, False, 1), dev(ids[None]), dev(ps[None]), kp, dev(one * k), dev(one),
                         dev(emit), nxt)
    assert eng.device_status() == 0
    tok, par, _ = O.build_prune_tree(O.TreeParams(B=Bn, k=k, K=K, expand_width=0, prune_parent=True), ids, ps, 501, n_depths=k)
    n = int(nxt.n_nodes[0])
    assert n == len(tok)
    assert nxt.tok[:n].tolist() == tok.tolist() and nxt.parent[:n].tolist() == par.tolist()
    check_block(nxt, 0, tok, par, k, 1)


# ---------------------------------------------------------------------------------------- tree builder
def random_lists(rng, k, kp, vocab):
    ids = np.zeros((k, kp), dtype=np.int32)
    ps = np.zeros((k, kp), dtype=np.float32)
    for i in range(k):
        ids[i] = rng.choice(vocab, size=kp, replace=False)
        ps[i] = np.sort(rng.dirichlet(np.ones(kp + 3))[:kp])[::-1].astype(np.float32)
    return ids, ps


@pytest.mark.parametrize("Bn,k,K,kp,width,layout,prune,static", [
    (15, 3, 4, 6, 1, 0, True, None),
    (64, 4, 8, 10, 0, 0, True, None),
    (64, 4, 8, 10, 0, 1, False, None),
    (96, 5, 10, 12, 0, 0, True, None),
    (10, 2, 100, 12, 1, 0, True, None),
    (30, 1, 100, 32, 1, 0, True, None),
    (2, 2, 3, 5, 1, 0, True, None),
    (20, 2, 15, 17, 1, 0, True, [15, 4]),
    (6, 2, 3, 5, 1, 1, True, [3, 2]),
    (32, 4, 8, 10, 3, 0, True, None),
])
def test_build_prune_tree_bit_exact(B, tiny_engine, Bn, k, K, kp, width, layout, prune, static):
    shape, w, eng = tiny_engine
    print(f"build_tree B={Bn} k={k} K={K} kp={kp} width={width} layout={layout} static={static}", flush=True)
    rng = np.random.default_rng(Bn * 100 + k)
    batch = 3
    vocab_small = 40          # small vocabulary: repeats with the parent's token do occur
    nodes = Bn if static is None else 1 + sum(static)
    rows = nodes * (k + 1) if layout == 0 else nodes + k
    nxt = B.BlockBuffers(batch, rows, k, layout)
    ids = np.zeros((batch, k, kp), dtype=np.int32)
    ps = np.zeros((batch, k, kp), dtype=np.float32)
    for b in range(batch):
        ids[b], ps[b] = random_lists(rng, k, kp, vocab_small)
    # exact probability ties across parents and a zero-probability tail in sequence 2
    ps[2, :, kp // 2:] = ps[2, :, kp // 2:kp // 2 + 1]
    n_lists = np.array([k, max(k - 1, 0), k], dtype=np.int32)
    n_emit = np.array([1, 2, 1], dtype=np.int32)
    emit = np.zeros((batch, B.MAX_MASKS + 1), dtype=np.int32)
    emit[0, 0] = ids[0, 0, 0]          # root token equals the best depth-1 candidate
    emit[1, 1] = 7
    emit[2, 0] = 3
    params = B.tree_params(Bn, k, K, width, prune, False, layout, static)
    dev = lambda a: torch.as_tensor(a).cuda()
    eng.build_prune_tree(params, dev(ids), dev(ps), kp, dev(n_lists), dev(n_emit), dev(emit), nxt)
    assert eng.device_status() == 0
    op = O.TreeParams(B=Bn, k=k, K=K, expand_width=width, prune_parent=prune, static_widths=static)
    for b in range(batch):
        root = int(emit[b, n_emit[b] - 1])
        tok, par, _ = O.build_prune_tree(op, ids[b], ps[b], root, n_depths=int(n_lists[b]))
        r0 = b * rows
        n = int(nxt.n_nodes[b])
        assert n == len(tok)
        assert nxt.tok[r0:r0 + n].tolist() == tok.tolist()
        assert nxt.parent[r0:r0 + n].tolist() == par.tolist()
        check_block(nxt, b, tok, par, k, layout)
    if static is None:
        return
    # Fixed tree, same block again (Sec. 4.3: its rows are built once; later calls only write tokens):
    # new lists and roots, every sequence with all k lists -- then a call in which a list of sequence
    # 1 runs out of entries, so that its tree is smaller and must be rebuilt in full -- then full lists
    # again.  Every call is checked against the oracle like the first one.
    for rnd in range(3):
        for b in range(batch):
            ids[b], ps[b] = random_lists(rng, k, kp, vocab_small)
        n_lists[:] = k
        if rnd == 1:
            ids[1, 0, 1:] = -1                       # depth 1 of sequence 1 has a single entry
            ps[1, 0, 1:] = 0.0
        emit[:, 0] = rng.integers(0, vocab_small, size=batch)
        n_emit[:] = 1
        eng.build_prune_tree(params, dev(ids), dev(ps), kp, dev(n_lists), dev(n_emit), dev(emit), nxt)
        assert eng.device_status() == 0
        for b in range(batch):
            # (a negative id ends a list on the device; the oracle is handed the list cut there)
            li = [ids[b, i][:1] if (rnd == 1 and b == 1 and i == 0) else ids[b, i] for i in range(k)]
            lp = [ps[b, i][:1] if (rnd == 1 and b == 1 and i == 0) else ps[b, i] for i in range(k)]
            tok, par, _ = O.build_prune_tree(op, li, lp, int(emit[b, 0]), n_depths=k)
            r0 = b * rows
            n = int(nxt.n_nodes[b])
            assert n == len(tok), (rnd, b, n, len(tok))
            assert nxt.tok[r0:r0 + n].tolist() == tok.tolist(), (rnd, b)
            assert nxt.parent[r0:r0 + n].tolist() == par.tolist(), (rnd, b)
            check_block(nxt, b, tok, par, k, layout)


def test_build_prune_tree_with_every_probability_tied(B, tiny_engine):
    """All list entries carry the same probability (a power of two, so the products are exact and
    equal per depth): every selection is decided by creation order alone.  (Children that do not beat the
    last of a full set are not created, so that at most 110 candidates meet here; the next test goes past 256.)
    Bit-exact against the oracle."""
    shape, w, eng = tiny_engine
    Bn, k, K, kp, layout = 96, 5, 10, 12, 0
    batch = 2
    rows = Bn * (k + 1)
    nxt = B.BlockBuffers(batch, rows, k, layout)
    rng = np.random.default_rng(77)
    ids = np.stack([np.stack([rng.permutation(500)[:kp] for _ in range(k)]) for _ in range(batch)]).astype(np.int32)
    ps = np.full((batch, k, kp), 0.0625, dtype=np.float32)
    ps[1, :, 0] = 0.125                                   # sequence 1: one better entry per list, ties below it
    n_lists = np.array([k, k], dtype=np.int32)
    n_emit = np.array([1, 1], dtype=np.int32)
    emit = np.zeros((batch, B.MAX_MASKS + 1), dtype=np.int32)
    emit[:, 0] = [501, 502]
    params = B.tree_params(Bn, k, K, 0, True, False, layout, None)
    dev = lambda a: torch.as_tensor(a).cuda()
    eng.build_prune_tree(params, dev(ids), dev(ps), kp, dev(n_lists), dev(n_emit), dev(emit), nxt)
    assert eng.device_status() == 0
    op = O.TreeParams(B=Bn, k=k, K=K, expand_width=0, prune_parent=True)
    for b in range(batch):
        tok, par, _ = O.build_prune_tree(op, ids[b], ps[b], int(emit[b, 0]), n_depths=k)
        r0 = b * rows
        n = int(nxt.n_nodes[b])
        assert n == len(tok)
        assert nxt.tok[r0:r0 + n].tolist() == tok.tolist()
        assert nxt.parent[r0:r0 + n].tolist() == par.tolist()


@pytest.mark.parametrize("Bn,k,K,kp,better", [(200, 2, 32, 32, 0), (200, 2, 32, 32, 5), (129, 2, 20, 20, 3), (256, 2, 32, 32, 31),
                                              (40, 2, 17, 17, 0), (256, 3, 12, 12, 2)])
def test_build_prune_tree_cut_inside_a_tied_run(B, tiny_engine, Bn, k, K, kp, better):
    """More candidates than the builder has threads (its threshold search), with the cut at B - 1 inside a run of
    equal probabilities: the first created of them stay.  `better` entries of the second list lie above the
    run; rows 1 and 2 of the batch have a zero tail and distinct values instead."""
    shape, w, eng = tiny_engine
    batch, rows = 3, Bn + k
    rng = np.random.default_rng(Bn + better)
    ids = np.stack([np.stack([rng.permutation(500)[:kp] for _ in range(k)]) for _ in range(batch)]).astype(np.int32)
    ps = np.full((batch, k, kp), 2.0 ** -5, dtype=np.float32)
    ps[0, 1, :better] = 2.0 ** -4
    ps[1, :, kp // 2:] = 0.0
    for i in range(k):
        ps[2, i] = np.sort(rng.uniform(0.01, 0.03, kp))[::-1]
    # until the last depth the set is not full, so that all children are created (less the parent's own token)
    assert sum(kp * (kp - 1) ** i for i in range(k - 1)) < Bn - 1 and sum(kp * (kp - 1) ** i for i in range(k)) > 256
    emit = np.full((batch, B.MAX_MASKS + 1), 501, dtype=np.int32)
    one = np.ones(batch, dtype=np.int32)
    dev = lambda a: torch.as_tensor(a).cuda()
    nxt = B.BlockBuffers(batch, rows, k, 1)
    print(f"tied run B={Bn} K={K} better={better}", flush=True)
    eng.build_prune_tree(B.tree_params(Bn, k, K, 0, True, False, 1), dev(ids), dev(ps), kp, dev(one * k), dev(one), dev(emit), nxt)
    assert eng.device_status() == 0
    for b in range(batch):
        tok, par, _ = O.build_prune_tree(O.TreeParams(B=Bn, k=k, K=K, expand_width=0, prune_parent=True), ids[b], ps[b], 501,
                                         n_depths=k)
        n = int(nxt.n_nodes[b])
        assert n == len(tok)
        assert nxt.tok[b * rows:b * rows + n].tolist() == tok.tolist()
        assert nxt.parent[b * rows:b * rows + n].tolist() == par.tolist()


@pytest.mark.parametrize("Bn,k,K,kp,layout", [(64, 4, 8, 10, 1), (96, 5, 10, 12, 0), (5, 3, 4, 4, 1)])
def test_build_prune_tree_refuses_a_node_without_its_parent(B, tiny_engine, Bn, k, K, kp, layout):
    """List entries above 1 (here the first of each list, by a few units in the last place, over a tail of tiny
    ones) let a child outrank its parent, and the cut at B - 1 can fall between them: what Alg. 1 selects is then
    no tree (the oracle cannot name a parent row).  The sequence is refused with the status bit, nothing is
    written for it, and its neighbours in the batch are built as usual."""
    shape, w, eng = tiny_engine
    batch = 3
    rng = np.random.default_rng(5 * Bn)
    op = O.TreeParams(B=Bn, k=k, K=K, expand_width=0, prune_parent=True)
    ids = np.zeros((batch, k, kp), dtype=np.int32)
    ps = np.zeros((batch, k, kp), dtype=np.float32)
    for b in (0, 2):
        ids[b], ps[b] = random_lists(rng, k, kp, 500)
    for _ in range(200):                            # the first draw whose selection is not ancestor-closed
        ids[1], _p = random_lists(rng, k, kp, 500)
        ps[1] = np.sort(rng.uniform(1e-11, 2.5e-8, (k, kp)))[:, ::-1].astype(np.float32)
        ps[1, :, 0] = 1.0000005
        try:
            O.build_prune_tree(op, ids[1], ps[1], 501, n_depths=k)
        except KeyError:
            break
    else:
        raise AssertionError("no draw without an orphan")
    rows = Bn * (k + 1) if layout == 0 else Bn + k
    nxt = B.BlockBuffers(batch, rows, k, layout)
    nxt.n_rows.fill_(-7), nxt.n_nodes.fill_(-7), nxt.tok.fill_(-7), nxt.parent.fill_(-7)
    emit = np.full((batch, B.MAX_MASKS + 1), 501, dtype=np.int32)
    dev = lambda a: torch.as_tensor(a).cuda()
    one = np.ones(batch, dtype=np.int32)
    print(f"refused tree B={Bn} k={k} K={K}", flush=True)
    eng.build_prune_tree(B.tree_params(Bn, k, K, 0, True, False, layout), dev(ids), dev(ps), kp, dev(one * k), dev(one), dev(emit),
                         nxt)
    assert eng.device_status() == B.DEV_BAD_TREE
    assert int(nxt.n_rows[1]) == 0 and int(nxt.n_nodes[1]) == 0
    assert bool((nxt.tok[rows:2 * rows] == -7).all()) and bool((nxt.parent[rows:2 * rows] == -7).all())
    for b in (0, 2):
        tok, par, _ = O.build_prune_tree(op, ids[b], ps[b], 501, n_depths=k)
        assert nxt.parent[b * rows:b * rows + len(tok)].tolist() == par.tolist()
        check_block(nxt, b, tok, par, k, layout)


@pytest.mark.parametrize("Bn,k,K,kp,width", [(12, 4, 5, 8, 0), (24, 3, 6, 6, 2), (15, 4, 4, 6, 1), (90, 3, 10, 12, 0),
                                             (200, 2, 32, 32, 0)])
def test_build_prune_tree_lists_above_one(B, tiny_engine, Bn, k, K, kp, width):
    """Lists that are no probabilities (scores above 1, NaN, negative entries): Alg. 1 as it is written, bit-exact
    against the oracle, and refused exactly where the nodes it selects are no tree.  Includes pools of more than
    256 candidates."""
    shape, w, eng = tiny_engine
    rng = np.random.default_rng(Bn)
    op = O.TreeParams(B=Bn, k=k, K=K, expand_width=width, prune_parent=True)
    params = B.tree_params(Bn, k, K, width, True, False, 1)
    dev = lambda a: torch.as_tensor(a).cuda()
    batch, rows = 3, Bn + k
    one = np.ones(batch, dtype=np.int32)
    emit = np.full((batch, B.MAX_MASKS + 1), 501, dtype=np.int32)
    built = refused = 0
    for rnd in range(8):
        ids = np.zeros((batch, k, kp), dtype=np.int32)
        ps = np.zeros((batch, k, kp), dtype=np.float32)
        for b in range(batch):
            ids[b], ps[b] = random_lists(rng, k, kp, 60)
            ps[b] *= np.float32(1.0000005 / ps[b].max()) if rnd % 4 == 0 else rng.choice([1, 2, 4, 20], (k, 1)).astype(np.float32)
        same = ps.copy()                              # what the oracle is handed
        if rnd == 3:
            ps[0], same[0] = np.nan, 1.0              # all equal: creation order decides
            ps[1, :, -1], same[1, :, -1] = -0.5, 0.0
        nxt = B.BlockBuffers(batch, rows, k, 1)
        print(f"lists above one B={Bn} k={k} K={K} width={width} draw {rnd}", flush=True)
        eng.build_prune_tree(params, dev(ids), dev(ps), kp, dev(one * k), dev(one), dev(emit), nxt)
        bad = False
        for b in range(batch):
            try:
                tok, par, _ = O.build_prune_tree(op, ids[b], same[b], 501, n_depths=k)
            except KeyError:
                bad, refused = True, refused + 1
                assert int(nxt.n_nodes[b]) == 0 and int(nxt.n_rows[b]) == 0
                continue
            built += 1
            n = int(nxt.n_nodes[b])
            assert n == len(tok), (rnd, b)
            assert nxt.tok[b * rows:b * rows + n].tolist() == tok.tolist(), (rnd, b)
            check_block(nxt, b, tok, par, k, 1)
            assert nxt.parent[b * rows:b * rows + n].tolist() == par.tolist(), (rnd, b)
        assert eng.device_status() == (B.DEV_BAD_TREE if bad else 0)
    print(f"built {built}, refused {refused}", flush=True)
    assert built >= 3


def test_build_static_tree_ignores_list_values(B, tiny_engine):
    """A fixed tree takes its entries by place: its shape does not depend on the values beside them."""
    shape, w, eng = tiny_engine
    rng = np.random.default_rng(8)
    k, kp, widths = 3, 6, [4, 3, 2]
    ids, ps = random_lists(rng, k, kp, 500)
    dev = lambda a: torch.as_tensor(a).cuda()
    one = np.ones(1, dtype=np.int32)
    emit = np.full((1, B.MAX_MASKS + 1), 501, dtype=np.int32)
    tok, par, _ = O.build_prune_tree(O.TreeParams(B=10, k=k, K=4, expand_width=1, static_widths=widths), ids, ps, 501, n_depths=k)
    for value in (ps, np.full_like(ps, np.nan), ps * 30, -ps):
        nxt = B.BlockBuffers(1, 10 + k, k, 1)
        eng.build_prune_tree(B.tree_params(10, k, 4, 1, True, False, 1, widths), dev(ids[None]), dev(value[None].astype(np.float32)), kp,
                             dev(one * k), dev(one), dev(emit), nxt)
        assert eng.device_status() == 0
        n = int(nxt.n_nodes[0])
        assert nxt.tok[:n].tolist() == tok.tolist() and nxt.parent[:n].tolist() == par.tolist()


# ---------------------------------------------------------------------------------------- verify + KV commit
def test_verify_accept_and_kv_commit(B, tiny_engine):
    shape, w, eng = tiny_engine
    rng = np.random.default_rng(5)
    k, layout, batch = 3, 0, 3
    trees = []
    for b in range(batch):
        t, p = synth.make_random_tree(20 + 5 * b, 3, 6, seed=40 + b, max_children=4)   # tokens in 0..5
        trees.append((t.numpy().copy(), p.numpy().copy()))
    rows = 35 * (k + 1)
    blk = B.BlockBuffers(batch, rows, k, layout)
    blk.upload_trees([t.tolist() for t, _ in trees], [p.tolist() for _, p in trees])
    eng.block_from_tree(blk)
    kv = B.KvCache(shape, [512, 300, 700])
    L0 = [100, 37, 250]
    kv.set_len(L0)
    # fill the block's scratch slots with recognisable rows
    krows, vrows = [], []
    for b in range(batch):
        n = int(blk.n_rows[b])
        kr = synth.normal_like((shape.n_layers, n, shape.n_kv_heads, shape.head_dim), 1.0, 50 + b, 0, "cuda")
        vr = synth.normal_like((shape.n_layers, n, shape.n_kv_heads, shape.head_dim), 1.0, 50 + b, 1, "cuda")
        for l in range(shape.n_layers):
            eng.kv_store(kv, l, b, L0[b], kr[l].contiguous(), vr[l].contiguous())
        krows.append(kr.cpu().numpy()); vrows.append(vr.cpu().numpy())
    g = rng.integers(0, 6, size=batch * rows).astype(np.int32)
    # make sequence 0 accept a full root-to-depth-3 path
    t0, p0 = trees[0]
    d3 = [i for i in range(len(t0)) if O.make_block(t0, p0, 0, 0).depth[i] == 3]
    if d3:
        c = d3[0]
        while p0[c] >= 0:
            g[p0[c]] = t0[c]
            c = p0[c]
    i32 = dict(dtype=torch.int32, device="cuda")
    n_emit = torch.zeros(batch, **i32)
    emit = torch.zeros((batch, B.MAX_MASKS + 1), **i32)
    acc = torch.zeros((batch, B.MAX_MASKS + 1), **i32)
    star = torch.zeros(batch, **i32)
    eng.verify_accept(blk, torch.as_tensor(g).cuda(), kv, n_emit, emit, acc, star)
    assert eng.device_status() == 0
    total_acc = 0
    for b in range(batch):
        tok, par = trees[b]
        n_star, accepted, emitted = O.verify_accept(tok, par, g[b * rows:b * rows + len(tok)])
        ne = int(n_emit[b])
        assert ne == len(emitted)
        assert emit[b, :ne].tolist() == emitted
        assert acc[b, :ne].tolist() == [0] + accepted
        assert int(star[b]) == n_star
        assert int(kv.len[b]) == L0[b] + ne
        total_acc += len(accepted)
        for l in range(shape.n_layers):
            kk, vv = eng.kv_load(kv, l, b, L0[b], ne)
            want_rows = [0] + accepted
            assert np.array_equal(kk.cpu().numpy(), krows[b][l][want_rows])
            assert np.array_equal(vv.cpu().numpy(), vrows[b][l][want_rows])
    assert total_acc >= 3


# ---------------------------------------------------------------------------------------- QKV epilogue
@pytest.mark.parametrize("head_dim", [64, 128])
def test_qk_norm_sum_order(B, head_dim):
    """The per-head RMSNorm adds its squares as a balanced tree over the rotary pairs, farthest pairs first:
    bit for bit.  K and V share one weight matrix and every row sits at position 0 (no rotation), so the V
    rows in the cache are the norm's inputs and the K rows its outputs."""
    shape = small_shape(d_model=128, n_q_heads=3, n_kv_heads=3, head_dim=head_dim, d_ff=176, vocab=517, n_layers=1,
                        qk_norm=True)
    w = synth.make_weights(shape, seed=6, unit_gains=False)
    w["layers"][0]["wv"] = w["layers"][0]["wk"]
    batch = 16
    eng = B.Engine(shape, w, batch, 1, 64)
    kv = B.KvCache(shape, [64] * batch)
    kv.set_len([0] * batch)
    blk = B.BlockBuffers(batch, 1, 0, 0)
    blk.upload_trees([[31 * b + 1] for b in range(batch)], [[-1]] * batch)
    eng.block_from_tree(blk)
    hidden = torch.zeros((batch, shape.d_model), dtype=torch.float32, device="cuda")
    eng.tree_forward(blk, None, kv, hidden, None)
    assert eng.device_status() == 0
    k, v = (np.stack(t) for t in zip(*[[x.cpu().numpy()[0] for x in eng.kv_load(kv, 0, b, 0, 1)] for b in range(batch)]))
    eng.close()
    half = head_dim // 2
    x0, x1 = v[..., :half], v[..., half:]                      # [batch, heads, pairs]
    s = (x1.astype(np.longdouble) ** 2 + x0 * x0).astype(np.float32)     # fma(x1, x1, x0 * x0)
    while s.shape[-1] > 1:
        n = s.shape[-1] // 2
        s = s[..., :n] + s[..., n:]
    inv = np.float32(1) / np.sqrt(s / np.float32(head_dim) + np.float32(shape.rms_eps))
    gain = w["layers"][0]["k_norm"].cpu().numpy().astype(np.float32)
    assert np.array_equal(k, v * (inv * gain))


@pytest.mark.parametrize("dtype,head_dim,d_model,hq,hkv,qk_norm", [
    ("bf16", 64, 512, 3, 1, False), ("bf16", 64, 1024, 6, 2, True), ("bf16", 64, 1536, 3, 3, True), ("bf16", 64, 2048, 2, 1, False),
    ("bf16", 64, 2560, 5, 1, True), ("bf16", 64, 3072, 3, 1, True), ("bf16", 64, 3584, 3, 3, False), ("bf16", 64, 4096, 3, 1, True),
    ("bf16", 128, 512, 3, 1, True), ("bf16", 128, 3584, 3, 3, True), ("f32", 64, 128, 3, 1, True), ("f32", 128, 128, 3, 3, False),
    ("f32", 128, 192, 5, 1, True)])
def test_qkv_epilogue_forms(B, dtype, head_dim, d_model, hq, hkv, qk_norm):
    """One layer against the oracle for every form of the QKV epilogue: head widths, types, QK-norm, and the 1 to 8
    split-K parts that d_model / 512 gives the bf16 projection.  Odd numbers of heads leave the last workgroup partial;
    two sequences of different length leave padding rows."""
    shape = small_shape(d_model=d_model, n_q_heads=hq, n_kv_heads=hkv, head_dim=head_dim, d_ff=128, vocab=256, n_layers=1,
                        qk_norm=qk_norm, dtype=dtype)
    w = synth.make_weights(shape, seed=7, unit_gains=False)
    m = oracle_model(shape, w)
    k, layout, lens = 2, 0, [70, 5]
    trees = [synth.make_random_tree(n, 4, shape.vocab, seed=60 + n) for n in (9, 6)]
    rows = 9 * (k + 1) + 2
    print(f"qkv epilogue {dtype} hd={head_dim} d={d_model} heads {hq}/{hkv} qk_norm={qk_norm}", flush=True)
    eng = B.Engine(shape, w, 2, rows, 256)
    blk = B.BlockBuffers(2, rows, k, layout)
    blk.upload_trees([t.tolist() for t, _ in trees], [p.tolist() for _, p in trees])
    eng.block_from_tree(blk)
    kv = B.KvCache(shape, [128, 64])
    old = []
    for b, n in enumerate(lens):
        old.append([synth.normal_like((n, hkv, head_dim), 1.0, 80 + b, i, "cuda", eng.dt) for i in (0, 1)])
        eng.kv_store(kv, 0, b, 0, *old[b])
    kv.set_len(lens)
    masks = synth.normal_like((k, d_model), 0.02, 81, 0, "cuda", eng.dt)
    hidden = torch.zeros((2 * rows, d_model), dtype=eng.dt, device="cuda")
    eng.tree_forward(blk, masks, kv, hidden, None)
    assert eng.device_status() == 0
    for b, n in enumerate(lens):
        ob = O.make_block(trees[b][0].numpy(), trees[b][1].numpy(), k, layout)
        R = ob.n_rows
        kc, vc = ([to_np(t)] for t in old[b])
        _, want_h, want_k, want_v = O.tree_forward(m, ob, to_np(masks), kc, vc, n, want_logits_rows=[0])
        got_k, got_v = eng.kv_load(kv, 0, b, n, R)
        for what, got, want in (("hidden", hidden[b * rows:b * rows + R], want_h), ("k", got_k, want_k[0]), ("v", got_v, want_v[0])):
            err = rel_err_rows(to_np(got).reshape(R, -1), np.asarray(want).reshape(R, -1))
            assert err < TOL[dtype], (what, b, err)
        # old rows and the slots behind the block are untouched
        before = eng.kv_load(kv, 0, b, 0, n)
        assert all(torch.equal(x, y) for x, y in zip(before, old[b]))
        after = eng.kv_load(kv, 0, b, n + R, kv.caps[b] - n - R)
        assert all(bool((x == 0).all()) for x in after)
    eng.close()


class BlockDev(ctypes.Structure):
    _fields_ = ([(n, ctypes.c_int) for n in ("batch", "rows_per_seq", "k_masks", "layout", "anc_words")] +
                [(n, ctypes.c_void_p) for n in ("n_rows", "n_nodes", "tok", "parent", "depth", "mask_j", "attach", "anc", "packed")])


class KvDev(ctypes.Structure):
    _fields_ = ([(n, ctypes.c_void_p) for n in ("k", "v", "len", "base", "seq_cap")] + [("capacity", ctypes.c_int64), ("len_bound", ctypes.c_int)])


class PackedEnd(ctypes.Structure):
    _fields_ = [("rows", ctypes.c_void_p * 3), ("width", ctypes.c_int * 3)]


class NodeLists(ctypes.Structure):
    _fields_ = [("max_nodes", ctypes.c_int)] + [(n, ctypes.c_void_p) for n in ("a_rows", "out_rows", "positions", "row_positions")]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d,hd,rows,nodes", [(64, 128, 75, 70), (320, 64, 9, 3), (4096, 128, 5, 1), (8192 + 12, 128, 4, 4)])
def test_embed_norm_and_lists(B, dtype, d, hd, rows, nodes):
    """A row's embedding, rotary table and norm, and the LM head's lists behind them: fewer columns than the table has entries, more
    than a thread has, lists of several workgroups, rows and a whole sequence that are not there."""
    print(f"embed {dtype} d={d} hd={hd} rows={rows} nodes={nodes}", flush=True)
    c, dt, vocab, k, theta, eps = ctypes, torch.float32 if dtype == "f32" else torch.bfloat16, 50, 4, 5e5, 1e-5
    g = torch.Generator().manual_seed(17)
    ints = lambda *shape, hi: torch.randint(0, hi, shape, generator=g, dtype=torch.int32).cuda()
    emb, masks = (synth.normal_like((n, d), 1.0, 19, i, "cuda", dt) for i, n in enumerate((vocab, k)))
    gain = synth.normal_like((d,), 1.0, 19, 2, "cuda", dt)
    dev = lambda v: torch.tensor(v, dtype=torch.int32, device="cuda")
    n_rows, n_nodes = dev([rows, rows - 1, 1, rows]), dev([nodes, max(nodes - 2, 1), 1, nodes])
    lens, base, cap = dev([1000, 3, 70000, -1]), dev([0, 2048, 4096, 128000]), dev([2000, 1024, 100000, 1000])   # the last one is invalid
    tok, depth = ints(4, rows, hi=vocab), ints(4, rows, hi=7)
    mask_j = torch.where(torch.arange(rows, device="cuda")[None] < n_nodes[:, None], 0, 1 + ints(4, rows, hi=k))
    M = 4 * rows
    h, rope, xn = torch.full((M, d), -7.0, device="cuda"), torch.zeros(M, hd // 2, 2, device="cuda"), torch.full((M, d), -7.0, dtype=dt, device="cuda")
    lists = torch.full((3, 4 * nodes), -7, dtype=torch.int32, device="cuda")
    where, status = torch.zeros(M, dtype=torch.int32, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda")
    p = lambda t: t.data_ptr()
    blk = BlockDev(4, rows, k, 0, 2, p(n_rows), p(n_nodes), p(tok), None, p(depth), p(mask_j), None, None, None)
    kv = KvDev(None, None, p(lens), p(base), p(cap), 1 << 20, 80000)
    run = internal("launch_embed", c.c_void_p, c.c_int, c.POINTER(BlockDev), c.POINTER(KvDev), c.c_void_p, c.c_void_p, c.c_void_p, c.c_int, c.c_int,
                   c.c_void_p, c.c_int, c.c_float, c.c_void_p, c.c_size_t, c.POINTER(PackedEnd), c.POINTER(NodeLists), c.c_void_p, c.c_float, c.c_void_p)
    assert run(torch.cuda.current_stream().cuda_stream, B.ESP_F32 if dtype == "f32" else B.ESP_BF16, blk, kv, p(emb), p(masks), p(h), d, vocab, p(rope), hd,
               theta, p(status), 0, PackedEnd(), NodeLists(nodes, p(lists[0]), p(lists[1]), p(lists[2]), p(where)), p(gain), eps, p(xn)) == 0
    live = (torch.arange(rows, device="cuda")[None] < n_rows[:, None]) & (torch.arange(4, device="cuda")[:, None] < 3)
    want = torch.where((mask_j > 0)[..., None], masks[(mask_j - 1).clamp(min=0).long()], emb[tok.long()]).float() * live[..., None]
    assert torch.equal(h, want.view(M, d)) and int(status) != 0
    norm = want.double() / (want.double().square().mean(-1, keepdim=True) + eps).sqrt() * gain.double()
    # fp32 sums of d squares in a tree of at most 3 + 6 + 16 levels, root and quotient, two products; then the rounding to bf16
    tol = 2.0 ** -8 if dtype == "bf16" else 20 * 2.0 ** -23
    assert bool(((xn.double() - norm.view(M, d)).abs() <= tol * norm.view(M, d).abs() + 1e-30).all())
    pos = torch.where(live, lens[:, None] + depth, 0).double().view(M, 1)
    angle = pos * theta ** (-2.0 * torch.arange(hd // 2, dtype=torch.float64, device="cuda") / hd)
    assert float((rope.double() - torch.stack((angle.cos(), angle.sin()), -1)).abs().max()) <= 2.0 ** -24 + 1e-10   # rounding; 77000 radians to 2^-52
    assert torch.equal(where.view(4, rows), lens[:, None] + depth + 1)
    for m in range(4 * nodes):
        s, i = divmod(m, nodes)
        there = i < int(n_nodes[s])
        row = s * rows + (i if there else 0)
        assert lists[:, m].tolist() == [row, row if there else -1, int(lens[s]) + int(depth.view(-1)[row]) + 1]


# ---------------------------------------------------------------------------- packed rows of a batch
@pytest.mark.parametrize("head_dim,counts,sample,invalid", [
    (128, [14, 1, 5], False, []), (128, [1, 14, 3, 14, 9, 2], True, []), (64, [2, 14, 8, 1], True, []), (128, [1, 1, 1, 1], False, []),
    (128, [14, 2, 9, 14, 1, 7, 3, 14, 14, 5, 1, 12], True, []), (128, [3, 14, 6, 2], False, [0, 2]), (64, [4, 1, 14], False, [0, 1, 2])])
def test_packed_rows_of_a_ragged_batch(B, head_dim, counts, sample, invalid):
    """Above 128 block rows a batch's live rows go through the layers packed together.  A row's sums do not depend on
    the rows beside it (one split-K part and one key split at these sizes), so every sequence comes out bit for bit as
    it does alone, with its rows where they were; rows that are not there are zero, also in the K/V cache, and so is the row
    behind the live ones in what goes into the projections, which stands for all of them there.  A sequence longer
    than the bound has no rows and sets the status, also where no sequence is left; twelve sequences' tree rows take the
    large-tile arg-max."""
    shape = small_shape(d_model=256, n_q_heads=4, n_kv_heads=2, head_dim=head_dim, d_ff=384, vocab=1024, n_layers=2, qk_norm=True,
                        dtype="bf16")
    w = synth.make_weights(shape, seed=9, unit_gains=False)
    k, layout, batch = 3, 0, len(counts)
    rows = 14 * (k + 1)
    lens = [(37 * b + 5) % 61 for b in range(batch)]
    print(f"packed rows hd={head_dim} counts={counts} sample={sample}", flush=True)
    masks = synth.normal_like((batch, k, 256), 0.02, 91, 0, "cuda", torch.bfloat16)

    def forward(which):
        n = len(which)
        eng = B.Engine(shape, w, n, rows, 256)
        eng.set_sampling(sample, 5)
        blk = B.BlockBuffers(n, rows, k, layout)
        trees = [synth.make_random_tree(counts[b], 4, shape.vocab, seed=70 + b) for b in which]
        blk.upload_trees([t.tolist() for t, _ in trees], [p.tolist() for _, p in trees])
        eng.block_from_tree(blk)
        kv = B.KvCache(shape, [128] * n)
        for i, b in enumerate(which):
            if lens[b]:
                for layer in range(2):
                    kf, vf = (synth.normal_like((lens[b], 2, head_dim), 1.0, 92 + b, 2 * layer + j, "cuda", torch.bfloat16) for j in (0, 1))
                    eng.kv_store(kv, layer, i, 0, kf, vf)
        kv.set_len([lens[b] for b in which])
        for i, b in enumerate(which):
            if b in invalid:
                kv.len[i] = kv.len_bound + 1
        hidden = torch.full((n * rows, 256), 7.0, dtype=torch.bfloat16, device="cuda")
        nxt = torch.full((n * rows,), -7, dtype=torch.int32, device="cuda")
        eng.tree_forward(blk, masks[which].contiguous() if n > 1 else masks[which[0]], kv, hidden, nxt)
        assert (eng.device_status() != 0) == any(b in invalid for b in which)
        planes = [torch.stack([torch.stack(eng.kv_load(kv, layer, i, 0, 128)) for layer in range(2)]) for i in range(n)]
        if n > 1:   # the workspace begins with the fp32 residual rows, then the rows that go into the projections
            live = sum(counts[b] * (k + 1) for b in which if b not in invalid)
            xn = eng.workspace[eng._ws_off + n * rows * 256 * 4:][:n * rows * 256 * 2].view(torch.bfloat16).reshape(n * rows, 256)
            assert bool((xn[live:live + 1] == 0).all()) and bool((xn[:live] != 0).any(1).all())
        eng.close()
        return hidden.reshape(n, rows, 256), nxt.reshape(n, rows), planes

    hidden, nxt, planes = forward(list(range(batch)))
    for b in range(batch):
        h1, n1, p1 = forward([b])
        live = 0 if b in invalid else counts[b] * (k + 1)
        assert torch.equal(hidden[b, :live], h1[0, :live]) and bool((hidden[b, live:] == 0).all()), b
        assert torch.equal(nxt[b], n1[0]), b
        assert torch.equal(planes[b], p1[0]) and bool((planes[b][:, :, lens[b] + live:] == 0).all()), b


@pytest.mark.parametrize("counts", [[80, 80], [80, 40], [80, 1], [60, 68]])
def test_packed_rows_with_two_gate_up_tiles(B, counts):
    """Two sequences of up to 320 rows, for which two gate/up tiles are launched and the number of live rows decides between
    them.  Each sequence alone takes other split-K parts: equal to the tolerance of bf16 models.  A profiling span covers both
    launches."""
    shape = small_shape(d_model=256, n_q_heads=4, n_kv_heads=2, head_dim=64, d_ff=14336, vocab=512, n_layers=2, dtype="bf16")
    tiles = internal("gate_up_tiles", ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.c_void_p, ctypes.c_bool, restype=ctypes.c_uint)
    assert tiles(640, 14336, 256, None, True) == 0b011
    w = synth.make_weights(shape, seed=9, unit_gains=False)
    k, rows = 3, 320
    print(f"packed rows, two gate/up tiles, counts={counts}", flush=True)
    masks = synth.normal_like((k, 256), 0.02, 91, 0, "cuda", torch.bfloat16)

    def forward(which):
        n = len(which)
        eng = B.Engine(shape, w, n, rows, 512)
        blk = B.BlockBuffers(n, rows, k, 0)
        trees = [synth.make_random_tree(counts[b], 4, shape.vocab, seed=70 + b) for b in which]
        blk.upload_trees([t.tolist() for t, _ in trees], [p.tolist() for _, p in trees])
        eng.block_from_tree(blk)
        kv = B.KvCache(shape, [rows] * n)
        kv.set_len([0] * n)
        hidden = torch.full((n * rows, 256), 7.0, dtype=torch.bfloat16, device="cuda")
        eng.profile_enable(["gemm_layer"])
        eng.tree_forward(blk, masks, kv, hidden, torch.zeros(n * rows, dtype=torch.int32, device="cuda"))
        spans, ms = eng.profile_read("gemm_layer")
        assert eng.device_status() == 0 and spans == 4 * shape.n_layers and 0 < ms < 1000
        eng.close()
        return to_np(hidden).reshape(n, rows, 256)

    both = forward([0, 1])
    for b in (0, 1):
        live = counts[b] * (k + 1)
        assert rel_err_rows(both[b, :live], forward([b])[0, :live]) < TOL["bf16"]
        assert np.all(both[b, live:] == 0)


class AttnPlan(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int) for n in ("nsplit", "tiles_per_split", "q_tiles", "ct_wg")]


@pytest.mark.parametrize("rows,lens,invalid", [
    ([36] * 16, [8192] * 16, []),                                          # equal: cuts at the same places in every sequence
    ([36, 1, 20, 9, 36, 30, 2, 36] * 2, [8192, 63, 1, 4000, 64, 0, 129, 8000] + [0, 0, 2000, 300, 8191, 65, 0, 12], []),
    ([132, 7, 100, 60, 33, 132, 80, 12], [5000, 8100, 0, 64, 700, 8192, 3, 2500], [1, 6]),   # two column groups; sequences that are not valid
    ([40] * 16, [8192] + [0] * 15, []),                                    # nearly all shares in one sequence
    ([40] * 16, [8192] * 16, list(range(16)))])                            # nobody there
def test_attention_shares_of_a_batch(B, rows, lens, invalid):
    """A batch's sequences as one line of work cut into equal shares: every sequence gets what it gets alone (there in equal
    splits), to the bf16 rounding of the result and of the probabilities, which depends on where the keys are split; rows that are not there
    are zero."""
    c = ctypes
    batch, most = len(rows), max(rows)
    shape = small_shape(d_model=256, n_q_heads=32, n_kv_heads=8, head_dim=128, d_ff=64, vocab=64, n_layers=1, dtype="bf16")
    plan = internal("attn_plan", *[c.c_int] * 7, restype=AttnPlan)(B.ESP_BF16, 128, batch, most, 32, 8, max(lens))
    shares = internal("attn_shares", *[c.c_int] * 6, c.POINTER(AttnPlan))(B.ESP_BF16, 128, batch, most, 32, 8, plan)
    print(f"attention shares rows={rows} lens={lens} plan={[getattr(plan, n) for n, _ in plan._fields_]} shares={shares}", flush=True)
    assert shares > 1
    w = synth.make_weights(shape, seed=3)
    g = torch.Generator(device="cuda")
    g.manual_seed(7)
    kvs = [[torch.randn(n + r, 8, 128, device="cuda", generator=g).bfloat16() for _ in (0, 1)] for n, r in zip(lens, rows)]
    qs = [torch.randn(r, 32, 128, device="cuda", generator=g).bfloat16() for r in rows]

    def run(which, pad):
        eng = B.Engine(shape, w, len(which), pad, max(lens) + pad)
        blk = B.BlockBuffers(len(which), pad, 0, 0)
        trees = [synth.make_random_tree(rows[b], 6, shape.vocab, seed=b) for b in which]
        blk.upload_trees([t.tolist() for t, _ in trees], [p.tolist() for _, p in trees])
        eng.block_from_tree(blk)
        kv = B.KvCache(shape, [lens[b] + pad for b in which])
        for i, b in enumerate(which):
            eng.kv_store(kv, 0, i, 0, *kvs[b])
        kv.set_len([lens[b] for b in which])
        for i, b in enumerate(which):
            if b in invalid:
                kv.len[i] = kv.len_bound + 1
        q = torch.zeros(len(which) * pad, 32, 128, dtype=torch.bfloat16, device="cuda")
        for i, b in enumerate(which):
            q[i * pad:i * pad + rows[b]] = qs[b]
        out = torch.full_like(q, 7.0)
        eng.attn_tree(blk, kv, 0, q, out)
        first = out.clone()
        eng.attn_tree(blk, kv, 0, q, out)
        assert torch.equal(first, out)                       # a second pass over the same buffers
        eng.close()
        return out.view(len(which), pad, 32, 128).float()

    got = run(list(range(batch)), most)
    for b in range(batch):
        live = 0 if b in invalid else rows[b]
        assert bool((got[b, live:] == 0).all()), b
        if live:
            want = run([b], rows[b])[0]
            err = (got[b, :live] - want).norm() / want.norm()
            assert float(err) < 5e-3, (b, float(err))        # two roundings to bf16 (2^-9 of a value at most) and those of the probabilities


class BlockDev(ctypes.Structure):
    _fields_ = ([(n, ctypes.c_int) for n in ("batch", "rows_per_seq", "k_masks", "layout", "anc_words")] +
                [(n, ctypes.c_void_p) for n in ("n_rows", "n_nodes", "tok", "parent", "depth", "mask_j", "attach", "anc", "packed")])


class KvDev(ctypes.Structure):
    _fields_ = ([(n, ctypes.c_void_p) for n in ("k", "v", "len", "base", "seq_cap")] + [("capacity", ctypes.c_int64), ("len_bound", ctypes.c_int)])


def attention_cuts(B, lens, rows, q_tiles, shares, seq_cap=8320, rows_per_seq=132):
    """(call that fills the table of the cuts for 4 query heads to a kv head, table)"""
    c, batch = ctypes, len(lens)
    dev = [torch.tensor(v, dtype=torch.int32, device="cuda") for v in (rows, lens, [i * seq_cap for i in range(batch)], [seq_cap] * batch)]
    table = torch.full((2 + 2 * (shares + 1) + 2 * batch,), -7, dtype=torch.int32, device="cuda")
    blk = BlockDev(batch, rows_per_seq, 0, 0, 3, dev[0].data_ptr())
    kv = KvDev(None, None, dev[1].data_ptr(), dev[2].data_ptr(), dev[3].data_ptr(), batch * seq_cap, 8192)
    fn = internal("launch_attn_cuts", c.c_void_p, c.POINTER(BlockDev), c.POINTER(KvDev), c.c_int, c.c_int, c.POINTER(AttnPlan), c.c_int, c.c_void_p)
    plan = AttnPlan(1, 130, q_tiles, 12)

    def run(keep=dev):
        assert fn(torch.cuda.current_stream().cuda_stream, blk, kv, 32, 8, plan, shares, table.data_ptr()) == 0
    return run, table


@pytest.mark.parametrize("batch,q_tiles,shares", [(2, 1, 32), (16, 2, 16), (63, 1, 32), (64, 1, 63), (65, 1, 63), (126, 2, 63), (126, 1, 63)])
def test_attention_cuts(B, batch, q_tiles, shares):
    """The table of a batch's cuts against whole numbers: share x begins where x / shares of the weight of all key tiles lies before
    it, inside one sequence; sequences without rows, without keys and not valid among them."""
    most = 96 if q_tiles == 1 else 132                       # twelve column tiles of 8 rows for a workgroup
    rows = [(17 * i) % (most + 1) if i % 5 else most for i in range(batch)]
    lens = [(i * 977) % 8000 if i % 7 else 0 for i in range(batch)]
    lens[-1] = 9000                                          # over the host's bound
    print(f"attention cuts batch={batch} q_tiles={q_tiles} shares={shares}", flush=True)
    time_of = [84, 70, 104, 110, 120, 126, 138, 150, 165, 175, 208, 218]
    unit = [time_of[-(-(-(-r * 4 // 32)) // q_tiles) - 1] for r in rows]
    tiles = [(n + r + 63) // 64 if r and n <= 8192 else 0 for r, n in zip(rows, lens)]
    weight = [180 + t * u if t else 0 for t, u in zip(tiles, unit)]
    total = sum(weight)
    n = max(1, min(shares, total // 400))
    start = [sum(weight[:i]) for i in range(batch)]
    begin = [x * total // n for x in range(n)]
    want = [n, -7]
    for at in begin:
        s = max(i for i in range(batch) if weight[i] and start[i] <= at)
        want += [s, min(tiles[s], max(0, -(-(at - start[s] - 180) // unit[s])))]
    want += [batch, 0] + [-7] * (2 * (shares - n))
    for i in range(batch):
        of = [x for x in range(n) if begin[x] < start[i] + weight[i] and (begin[x + 1] if x + 1 < n else total) > start[i]]
        want += [of[0], of[-1]] if weight[i] else [0, -1]
    run, table = attention_cuts(B, lens, rows, q_tiles, shares)
    run()
    assert table.tolist() == want


def test_attention_cuts_do_not_wait_for_one_sequence_after_the_other(B):
    """The cuts of 126 sequences take as long as those of 2 (a chain of loads a sequence made it 4.3 times)."""
    best = []
    for batch in (2, 126):
        run, _ = attention_cuts(B, [64 * i for i in range(batch)], [8] * batch, 1, 63)
        for _ in range(20):
            run()
        times = []
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(100):
                run()
            b.record()
            b.synchronize()
            times.append(a.elapsed_time(b))
        best.append(min(times))
    assert best[1] < 2 * best[0], best


# ---------------------------------------------------------------------------------------- attention
def run_attention_case(B, shape, eng, n_nodes, k, layout, cache_lens, seed):
    batch = len(cache_lens)
    if k == 0:   # prefill-like chain block: row i sees rows 0..i
        sizes = [max(n_nodes - 3 * b, 1) for b in range(batch)]
        trees = [(torch.arange(n, dtype=torch.int32) % shape.vocab, torch.arange(-1, n - 1, dtype=torch.int32)) for n in sizes]
    else:
        trees = [synth.make_random_tree(n_nodes - 3 * b, max(k, 2), shape.vocab, seed=seed + b)
                 for b in range(batch)]
    rows = n_nodes * (k + 1) if layout == 0 else n_nodes + k
    blk = B.BlockBuffers(batch, rows, k, layout)
    blk.upload_trees([t.tolist() for t, _ in trees], [p.tolist() for _, p in trees])
    eng.block_from_tree(blk)
    kv = B.KvCache(shape, [L + rows + 5 for L in cache_lens])
    kv.set_len(cache_lens)
    dt = eng.dt
    hq, hkv, hd = shape.n_q_heads, shape.n_kv_heads, shape.head_dim
    layer = shape.n_layers - 1
    q = synth.normal_like((batch * rows, hq, hd), 1.0, seed, 7, "cuda", dt)
    oracle_in = []
    for b in range(batch):
        R = int(blk.n_rows[b])
        L = cache_lens[b]
        kf = synth.normal_like((L + R, hkv, hd), 1.0, seed + b, 8, "cuda", dt)
        vf = synth.normal_like((L + R, hkv, hd), 1.0, seed + b, 9, "cuda", dt)
        eng.kv_store(kv, layer, b, 0, kf, vf)
        oracle_in.append((to_np(kf), to_np(vf), R, L))
    out = torch.zeros_like(q)
    eng.attn_tree(blk, kv, layer, q, out)
    assert eng.device_status() == 0
    got = to_np(out).reshape(batch, rows, hq, hd)
    qn = to_np(q).reshape(batch, rows, hq, hd)
    worst = 0.0
    for b in range(batch):
        kf, vf, R, L = oracle_in[b]
        ob = O.make_block(trees[b][0].numpy(), trees[b][1].numpy(), k, layout)
        want = O.tree_attention(qn[b, :R], kf[:L], vf[:L], kf[L:], vf[L:], ob.visible)
        worst = max(worst, rel_err_rows(got[b, :R].reshape(R * hq, hd), want.reshape(R * hq, hd)))
        assert np.all(got[b, R:] == 0)
    return worst


@pytest.mark.parametrize("n_nodes,k,layout,cache_lens", [
    (13, 3, 0, [128]), (5, 2, 1, [0, 3]), (20, 2, 0, [700, 64, 1]), (64, 0, 0, [190])])
def test_attn_tree_f32(B, tiny_engine, n_nodes, k, layout, cache_lens):
    shape, w, eng = tiny_engine
    print(f"attn f32 n={n_nodes} k={k} layout={layout} L={cache_lens}", flush=True)
    err = run_attention_case(B, shape, eng, n_nodes, k, layout, cache_lens, seed=60)
    assert err < 1e-4


@pytest.mark.parametrize("dtype,head_dim,offset", [("f32", 64, 1), ("f32", 128, 0), ("f32", 128, 1), ("bf16", 64, 0), ("bf16", 64, 1)])
def test_attn_tree_generic_forms(B, monkeypatch, dtype, head_dim, offset):
    """The generic attention kernel at both types and head widths, with caches that start off a 16-byte boundary, splits of
    one and of several key tiles, and a last tile with one key."""
    class Shifted(B.KvCache):
        def __init__(self, *a):
            super().__init__(*a)
            n = self.k.numel()
            self.k, self.v = (torch.full((n + offset,), float("nan"), dtype=t.dtype, device="cuda")[offset:].view(t.shape)
                              for t in (self.k, self.v))
    monkeypatch.setattr(B, "KvCache", Shifted)
    shape = small_shape(d_model=256, n_q_heads=4, n_kv_heads=2, head_dim=head_dim, d_ff=128, vocab=512, n_layers=2, dtype=dtype)
    w = synth.make_weights(shape, seed=5)
    for n_nodes, k, layout, lens in [(11, 3, 0, [148, 64]), (1, 0, 0, [1000]), (90, 4, 0, [700]), (3, 2, 1, [64 - 5, 0])]:
        rows = n_nodes * (k + 1) if layout == 0 else n_nodes + k
        eng = B.Engine(shape, w, max_batch=len(lens), max_rows_per_seq=rows, max_kv_len=max(lens) + rows + 64)
        print(f"attn generic {dtype} hd={head_dim} offset={offset} n={n_nodes} L={lens}", flush=True)
        err = run_attention_case(B, shape, eng, n_nodes, k, layout, lens, seed=61)
        eng.close()
        assert err < TOL[dtype]


@pytest.mark.parametrize("dtype,head_dim", [("f32", 64), ("f32", 128), ("bf16", 64)])
def test_attn_tree_generic_splits(B, dtype, head_dim):
    """One split to more than a workgroup merges by itself (8 at a head of 64, 4 at 128), sequences that leave splits without a
    key tile, and rows that are not there."""
    shape = small_shape(d_model=256, n_q_heads=4, n_kv_heads=2, head_dim=head_dim, d_ff=128, vocab=512, n_layers=1, dtype=dtype)
    w = synth.make_weights(shape, seed=5)
    for n_nodes, lens in [(5, [0]), (5, [64, 1]), (5, [130]), (7, [250, 3]), (5, [300]), (6, [1000, 64, 600]), (1, [1400]), (6, [2600, 40])]:
        rows = n_nodes * 3
        eng = B.Engine(shape, w, max_batch=len(lens), max_rows_per_seq=rows, max_kv_len=max(lens) + rows + 64)
        print(f"attn generic {dtype} hd={head_dim} n={n_nodes} L={lens}", flush=True)
        err = run_attention_case(B, shape, eng, n_nodes, 2, 0, lens, seed=62)
        eng.close()
        assert err < TOL[dtype]


@pytest.fixture(scope="module")
def bf16_engine(B):
    shape = small_shape(d_model=256, n_q_heads=8, n_kv_heads=2, head_dim=128, d_ff=384, vocab=1024, n_layers=2,
                        dtype="bf16", qk_norm=True, rope_theta=1.0e6, rms_eps=1e-6)
    w = synth.make_weights(shape, seed=4, unit_gains=False)
    eng = B.Engine(shape, w, max_batch=3, max_rows_per_seq=640, max_kv_len=5000)
    yield shape, w, eng
    eng.close()


@pytest.mark.parametrize("n_nodes,k,layout,cache_lens", [
    (13, 3, 0, [128]), (5, 2, 1, [0, 3]), (64, 4, 0, [2048]), (64, 4, 1, [2048, 777, 63]),
    (17, 4, 0, [4100, 64, 1]), (128, 4, 0, [300]), (200, 0, 0, [129])])
def test_attn_tree_bf16_mfma(B, bf16_engine, n_nodes, k, layout, cache_lens):
    shape, w, eng = bf16_engine
    print(f"attn bf16 n={n_nodes} k={k} layout={layout} L={cache_lens}", flush=True)
    err = run_attention_case(B, shape, eng, n_nodes, k, layout, cache_lens, seed=70)
    assert err < 2e-2


@pytest.mark.parametrize("n_nodes,cache_lens", [(1, [900]), (7, [193]), (9, [1500, 3]), (16, [700]), (23, [64]), (31, [2100])])
def test_attn_tree_bf16_few_columns(B, bf16_engine, n_nodes, cache_lens):
    """One to four column tiles a kv head, in splits of two key tiles: one or two column tiles without waves that share one."""
    shape, w, eng = bf16_engine
    print(f"attn bf16 few columns n={n_nodes} L={cache_lens}", flush=True)
    assert run_attention_case(B, shape, eng, n_nodes, 0, 0, cache_lens, seed=75) < 2e-2


class AttnPlan(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int) for n in ("nsplit", "tiles_per_split", "q_tiles", "ct_wg")]


@pytest.mark.parametrize("n_nodes,ct_wg,cache_lens", [
    (1, 1, [4096, 30, 700, 1, 2111]), (1, 1, [63, 64, 65, 1500, 1, 127, 128, 3000, 700, 5, 640, 2000, 33, 900, 1200, 4096]),
    (7, 1, [1500, 3, 64, 800, 129, 1400, 1000, 190]), (12, 2, [2000, 1, 700, 1300, 61]), (9, 2, [4096, 129, 64]), (68, 2, [2048])])
def test_attn_tree_bf16_paired_columns(B, n_nodes, ct_wg, cache_lens):
    """One or two column tiles a workgroup in splits of three and more key tiles: two waves share a column tile, the other
    waves of four (with one column tile, two) only load.  Lengths leave splits empty, with one key and partly masked."""
    shape = small_shape(d_model=512, n_q_heads=32, n_kv_heads=8, head_dim=128, d_ff=128, vocab=512, n_layers=1, dtype="bf16")
    bound = max(cache_lens)
    p = internal("attn_plan", *[ctypes.c_int] * 7, restype=AttnPlan)(B.ESP_BF16, 128, len(cache_lens), n_nodes, 32, 8, bound)
    print(f"attn bf16 paired n={n_nodes} L={cache_lens} splits={p.nsplit}x{p.tiles_per_split}", flush=True)
    assert p.ct_wg == ct_wg and p.tiles_per_split >= 3
    eng = B.Engine(shape, synth.make_weights(shape, seed=5), max_batch=len(cache_lens), max_rows_per_seq=n_nodes, max_kv_len=bound + n_nodes + 64)
    err = run_attention_case(B, shape, eng, n_nodes, 0, 0, cache_lens, seed=77)
    eng.close()
    assert err < 2e-2


# ------------------------------------------------------------------------- mask initialisations
@pytest.mark.parametrize("hq,hkv,n_nodes,k,layout,cache_lens", [
    (2, 2, 40, 3, 0, [515]),            # no grouping: one query head per kv head
    (8, 1, 30, 4, 0, [260, 31]),        # eight query heads share one kv head: 1200 query columns per kv head
    (16, 2, 9, 2, 1, [70]),             # G = 8, few rows
    (4, 4, 120, 4, 1, [1000, 64, 129, 5]),
])
def test_attn_tree_bf16_other_head_groupings(B, hq, hkv, n_nodes, k, layout, cache_lens):
    """The MFMA attention kernel at other ratios of query to kv heads than the 4 of the two 8B shapes
    (query columns of a kv head = block rows x group size: from 124 to 1200 here, i.e. one to four
    workgroups per kv head and split, with and without paired waves)."""
    shape = small_shape(d_model=max(hq * 16, 128), n_q_heads=hq, n_kv_heads=hkv, head_dim=128, d_ff=256, vocab=512, n_layers=1,
                        dtype="bf16", qk_norm=False, rope_theta=1.0e4)
    w = synth.make_weights(shape, seed=5)
    rows = n_nodes * (k + 1) if layout == 0 else n_nodes + k
    eng = B.Engine(shape, w, max_batch=len(cache_lens), max_rows_per_seq=rows, max_kv_len=max(cache_lens) + rows + 64)
    print(f"attn bf16 hq={hq} hkv={hkv} n={n_nodes} k={k} layout={layout} L={cache_lens}", flush=True)
    err = run_attention_case(B, shape, eng, n_nodes, k, layout, cache_lens, seed=90)
    eng.close()
    assert err < 2e-2


@pytest.mark.parametrize("which,offset", [("tiny", 0), ("tiny", 1), ("bf16", 0), ("bf16", 1)])
def test_mask_mean(B, which, offset):
    """Eq. 4 at prompt lengths around the 64 token groups of eight rows, with d not a multiple of a workgroup's 64
    features, ids outside the vocabulary (they add nothing), and a table that starts off a vector's alignment.  fp32 sums
    of values below 5 sigma: n 2^-24 relative to the largest partial sum at most, far below the tolerances."""
    dt = torch.float32 if which == "tiny" else torch.bfloat16
    shape = small_shape(d_model=192 + 4 if which == "tiny" else 320, head_dim=64, d_ff=128,
                        dtype="f32" if which == "tiny" else "bf16", vocab=512)
    w = synth.make_weights(shape, seed=6, device="cuda")
    store = torch.zeros(shape.vocab * shape.d_model + offset, dtype=dt, device="cuda")
    w["embed"] = store[offset:].view(shape.vocab, shape.d_model).copy_(w["embed"].to("cuda"))
    eng = B.Engine(shape, w, 1, 8, 64)
    table = to_np(w["embed"])
    for n in (1, 2, 63, 64, 65, 511, 512, 513, 1500):
        tok = synth.uniform_ints(n, 2 * shape.vocab, 8, n).to("cuda", torch.int32) - shape.vocab // 2
        out = torch.full((3, shape.d_model), 9.0, dtype=dt, device="cuda")
        eng.mask_mean(tok, 3, out)
        ids = tok.cpu().numpy()
        want = table[ids[(ids >= 0) & (ids < shape.vocab)]].sum(0) / n
        got = to_np(out)
        assert np.array_equal(got[0], got[1]) and np.array_equal(got[0], got[2])
        assert np.max(np.abs(got[0] - want)) <= (1e-6 if which == "tiny" else 2.0 ** -8) * max(np.max(np.abs(want)), 1e-30), n
    eng.close()


@pytest.mark.parametrize("which", ["tiny", "bf16"])
def test_mask_last_k_and_gaussian_inits(B, tiny_engine, bf16_engine, which):
    """Sec. 4 mask-design variants a (last k prompt tokens) and b (Gaussian fit of the embedding
    table), and the mu + 5 sigma / mu + 10 sigma rows of the appendix, against the oracle."""
    shape, w, eng = tiny_engine if which == "tiny" else bf16_engine
    print(f"mask inits {which}", flush=True)
    m = oracle_model(shape, w)
    k = 3
    dt = torch.float32 if shape.dtype == "f32" else torch.bfloat16
    tol = 1e-4 if shape.dtype == "f32" else 2e-2
    out = torch.zeros((k, shape.d_model), dtype=dt, device="cuda")
    prompt = [5, 9, 2, 7, 11]
    eng.mask_last_k(torch.tensor(prompt, dtype=torch.int32, device="cuda"), k, out)
    assert np.array_equal(to_np(out), O.mask_last_k_init(m, prompt, k))     # a copy of table rows: exact
    z = synth.normal_like((k, shape.d_model), 1.0, 41, 0, "cuda", torch.float32)
    for zz, shift in [(z, 0.0), (None, 5.0), (None, 10.0), (z, -1.5)]:
        eng.mask_gaussian(zz, shift, k, out)
        want = O.mask_gaussian_init(m, k, None if zz is None else zz.cpu().numpy(), shift)
        assert rel_err_rows(to_np(out), want) <= tol
    with pytest.raises(RuntimeError):
        eng.mask_last_k(torch.tensor([1, 2], dtype=torch.int32, device="cuda"), 3, out)
