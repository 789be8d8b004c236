"""GPU parity of the individual kernels (through the C ABI) against the CPU oracle's functions."""
import zlib

import numpy as np
import pytest

import workload as wl
from oracle import attention_row, log_softmax, top_k

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    import paper_2408_15766_amd as P
    assert torch.cuda.is_available()
    return torch, P


def case_seed(*case):
    """A fixed seed per test case (the built-in hash of a tuple with a string in it changes from process to process)."""
    return zlib.crc32(repr(case).encode())


def rand_storage(rng, shape, dtype, scale=1.0):
    """float32 values that are exact in the storage type."""
    x = (rng.standard_normal(shape) * scale).astype(np.float32)
    return wl.round_to_bf16(x) if dtype == "bf16" else x


def to_dev(torch, x, dtype):
    t = torch.from_numpy(np.ascontiguousarray(x)).cuda()
    return t.to(torch.bfloat16) if dtype == "bf16" else t


GEMM_CASES = [
    # dtype, m, in, rows per segment, n_split
    ("fp32", 16, 256, (256, 256, 256), 1),      # tiny QKV
    ("fp32", 16, 256, (688, 688), 1),           # tiny gate/up: ragged 32-row blocks
    ("fp32", 16, 688, (256,), 1),               # tiny down: ragged K (688 = 10.75 iterations)
    ("fp32", 1, 688, (256,), 2),
    ("fp32", 33, 512, (96,), 2),
    ("bf16", 60, 4096, (1024, 256, 256), 4),    # GQA-style QKV, two token blocks
    ("bf16", 1, 4096, (512,), 4),               # plain decoding row
    ("bf16", 10, 11008, (128,), 8),             # draft frontier, long K, uneven slabs per split
    ("bf16", 64, 1280, (100,), 1),              # ragged rows, odd slab count
    ("bf16", 60, 256, (1000,), 1),              # one slab only
    ("bf16", 100, 2048, (160,), 2),             # four token blocks (tree-shape sweep sizes)
    ("bf16", 200, 1024, (96, 40), 2),           # two 128-row tiles (prefill), ragged second tile, two segments
    ("bf16", 512, 768, (300,), 1),              # four full tiles, ragged rows
    ("fp32", 129, 256, (64,), 1),               # second tile of a single row
]


@pytest.mark.parametrize("dtype,m,k,rows,n_split", GEMM_CASES)
def test_gemm_matches_matmul(env, dtype, m, k, rows, n_split):
    torch, P = env
    rng = np.random.default_rng(case_seed(dtype, m, k, rows))
    x = rand_storage(rng, (m, k), dtype)
    ws = [rand_storage(rng, (r, k), dtype, 0.05) for r in rows]
    part = P.spec_k_gemm(to_dev(torch, x, dtype), [to_dev(torch, w, dtype) for w in ws], n_split)
    torch.cuda.synchronize()
    got = part.cpu().numpy().astype(np.float64).sum(axis=0)
    want = x.astype(np.float64) @ np.concatenate(ws).astype(np.float64).T
    assert not np.isnan(got).any()
    tol = 2e-5 * np.sqrt(k) * 0.05 * (1 if dtype == "fp32" else 4)
    assert np.abs(got - want).max() < tol


@pytest.mark.parametrize("m,k,rows,n_split", [(1, 4, [1], 1), (16, 256, [257, 33, 31], 1), (17, 688, [48], 1), (33, 324, [4100], 1),
                                              (49, 1100, [96], 2), (81, 4096, [320], 4), (129, 512, [9000], 1), (700, 100, [64], 1)])
def test_gemm_fp32_matches_fp64(env, m, k, rows, n_split):
    """fp32 storage: one to many 16-token blocks, half and whole weight blocks, fewer than four 64-k tiles (wavefronts without
    work), ragged K and rows, K splits; a row alone gives the bits it has among the others."""
    torch, P = env
    g = torch.Generator(device="cuda"); g.manual_seed(case_seed("f32", m, k) & 0xFFFF)
    x = torch.randn(m, k, device="cuda", generator=g)
    ws = [torch.randn(r, k, device="cuda", generator=g) * 0.05 for r in rows]
    got = P.spec_k_gemm(x, ws, n_split)
    want = x.double() @ torch.cat(ws).double().t()
    assert (got.double().sum(0) - want).abs().max() <= 1e-6 * np.sqrt(k) * max(1.0, float(want.abs().max()))
    for i in sorted({0, m // 2, m - 1}):
        assert torch.equal(P.spec_k_gemm(x[i:i + 1].contiguous(), ws, n_split)[:, 0], got[:, i])


@pytest.mark.parametrize("m,k,rows,n_split", [(17, 100, [33000], 1), (31, 64, [20000, 33, 31], 1), (130, 260, [3000, 1111, 65], 1), (33, 516, [16400], 2),
                                              (258, 1100, [1001, 1030], 3), (300, 2752, [1000], 4), (520, 1024, [1100], 1)])
def test_gemm_fp32_tiled_matches_fp64_and_small_launches_bits(env, m, k, rows, n_split):
    """fp32 launches that fill the chip (more than 16 rows, 1024 workgroups of the small kernel): 32 x 64 tiles, one row or one block past a tile, segments that
    meet inside one, one to many 64-k tiles, groups of K without a tile, ragged K, K splits.  Rows alone take the other kernel and have
    the same bits, and so has the whole through an X that is not 16-byte aligned; SwiGLU in the epilogue likewise."""
    torch, P = env
    g = torch.Generator(device="cuda"); g.manual_seed(case_seed("f32t", m, k) & 0xFFFF)
    flat = torch.randn(m * k + 4, device="cuda", generator=g)
    ws = [torch.randn(r, k, device="cuda", generator=g) * 0.05 for r in rows]
    assert (m + 15) // 16 * sum((r + 31) // 32 for r in rows) * n_split >= 1024
    x, off = flat[:m * k].view(m, k), torch.empty(m * k + 1, device="cuda")[1:].view(m, k)
    off.copy_(x)
    got = P.spec_k_gemm(x, ws, n_split)
    want = x.double() @ torch.cat(ws).double().t()
    assert (got.double().sum(0) - want).abs().max() <= 1e-6 * np.sqrt(k) * max(1.0, float(want.abs().max()))
    assert torch.equal(P.spec_k_gemm(off, ws, n_split), got)
    for i in sorted({0, 15, 16, m // 2, m - 1}):
        assert torch.equal(P.spec_k_gemm(x[i:i + 1].contiguous(), ws, n_split)[:, 0], got[:, i])
    gate, up = torch.cat(ws), torch.cat(ws).flip(0)
    act = P.spec_k_gemm_swiglu(x, gate, up)
    gd = want
    ud = want.flip(1)
    ref = gd * torch.sigmoid(gd) * ud
    assert ((act.double() - ref).abs() <= 1e-5 * np.sqrt(k) * (1 + ref.abs())).all()
    assert torch.equal(P.spec_k_gemm_swiglu(off, gate, up), act)
    assert torch.equal(P.spec_k_gemm_swiglu(x[m - 1:].contiguous(), gate, up)[0], act[m - 1])


@pytest.mark.parametrize("m,k", [(17, 128), (48, 192), (49, 192), (33, 256), (40, 320), (80, 448), (81, 640)])
def test_gemm_fp32_tiled_ring_and_ragged_tiles(env, m, k):
    """The ring of half k tiles: every count from two tiles to one past its second turn; last token tiles of up to 16 rows, whose
    wavefronts share a weight block instead of the tokens, and of one row more."""
    torch, P = env
    g = torch.Generator(device="cuda"); g.manual_seed(case_seed("f32r", m, k) & 0xFFFF)
    x = torch.randn(m, k, device="cuda", generator=g)
    ws = [torch.randn(r, k, device="cuda", generator=g) * 0.05 for r in (32900, 47)]
    got = P.spec_k_gemm(x, ws, 1)
    want = x.double() @ torch.cat(ws).double().t()
    assert (got.double().sum(0) - want).abs().max() <= 1e-6 * np.sqrt(k) * max(1.0, float(want.abs().max()))
    for i in sorted({0, max(m // 32 * 32 - 1, 0), m // 32 * 32, m - 1}):
        assert torch.equal(P.spec_k_gemm(x[i:i + 1].contiguous(), ws, 1)[:, 0], got[:, i])


@pytest.mark.parametrize("dtype,m,k,rows", [("fp32", 16, 256, 688), ("bf16", 60, 4096, 1100), ("bf16", 1, 1280, 64), ("bf16", 200, 768, 300),
                                            ("bf16", 40, 256, 77), ("fp32", 33, 128, 77), ("bf16", 60, 512, 15), ("bf16", 130, 256, 45)])
def test_gemm_swiglu_epilogue_matches_oracle(env, dtype, m, k, rows):
    """Gate and up projections with SwiGLU applied inside the launch: silu(x.wg) * (x.wu) against fp64, ragged 16-column
    blocks, one row, two 128-row tiles (the prefill form), an odd number of columns (no paired stores) and fewer columns
    than one block.  bf16 storage rounds the result once (relative 2^-9)."""
    torch, P = env
    rng = np.random.default_rng(case_seed("swiglu", dtype, m, k, rows))
    x = rand_storage(rng, (m, k), dtype)
    wg, wu = rand_storage(rng, (rows, k), dtype, 0.05), rand_storage(rng, (rows, k), dtype, 0.05)
    act = P.spec_k_gemm_swiglu(to_dev(torch, x, dtype), to_dev(torch, wg, dtype), to_dev(torch, wu, dtype))
    torch.cuda.synchronize()
    got = act.float().cpu().numpy().astype(np.float64)
    g = x.astype(np.float64) @ wg.astype(np.float64).T
    u = x.astype(np.float64) @ wu.astype(np.float64).T
    want = g / (1.0 + np.exp(-g)) * u
    assert not np.isnan(got).any()
    tol = 1e-5 * np.sqrt(k) + (2.0 ** -8 * np.abs(want) if dtype == "bf16" else 0.0)
    assert (np.abs(got - want) <= tol).all()


def expected_packed(rows_of_block, n_blocks, k_elems, esz, src_bytes_of_row):
    """The packed layout written out from its definition: tiles of 32 rows x 256 bytes of k, tiles of a block consecutive
    along k, piece (j, lane) of a tile at byte j*1024 + lane*16 = row lane%32, k-bytes (lane/32)*128 + j*16 .. +16 of the
    tile; zero beyond the matrix.  rows_of_block(b, c) -> source row or None; src_bytes_of_row(r) -> the row as bytes."""
    row_bytes = k_elems * esz
    n_it = (row_bytes + 255) // 256
    out = np.zeros((n_blocks, n_it, 8, 64, 16), dtype=np.uint8)
    for b in range(n_blocks):
        for c in range(32):
            r = rows_of_block(b, c)
            if r is None:
                continue
            src = np.zeros(n_it * 256, dtype=np.uint8)
            src[:row_bytes] = src_bytes_of_row(r)
            t = src.reshape(n_it, 2, 8, 16)                      # [tile][half g][piece j][16 bytes]
            for g in range(2):
                out[b, :, :, g * 32 + c, :] = t[:, g]
    return out.reshape(-1)


@pytest.mark.parametrize("dtype,rows,k", [("bf16", 77, 200), ("fp32", 45, 100), ("bf16", 64, 256)])
def test_packed_layouts_match_their_definition(env, dtype, rows, k):
    """spec_pack_weight and spec_pack_gate_up against the layout the header defines, byte for byte: ragged rows, ragged
    k, zero padding; gate/up: block b = gate rows 16b..16b+15 then up rows 16b..16b+15."""
    torch, P = env
    rng = np.random.default_rng(case_seed("pack", dtype, rows, k))
    esz = 2 if dtype == "bf16" else 4
    w, u = rand_storage(rng, (rows, k), dtype), rand_storage(rng, (rows, k), dtype)
    dw, du = to_dev(torch, w, dtype), to_dev(torch, u, dtype)
    raw = lambda t: t.contiguous().view(torch.uint8).cpu().numpy().reshape(rows, k * esz)
    bw, bu = raw(dw), raw(du)
    got = P.spec_pack_weight(dw)
    nb = (rows + 31) // 32
    want = expected_packed(lambda b, c: b * 32 + c if b * 32 + c < rows else None, nb, k, esz, lambda r: bw[r])
    assert got.numel() == want.size == P.spec_packed_bytes(1 if dtype == "bf16" else 0, rows, k)
    assert np.array_equal(got.cpu().numpy(), want)
    got = P.spec_pack_gate_up(dw, du)
    nb = (rows + 15) // 16

    def src_row(b, c):
        r = b * 16 + (c & 15)
        return (r if c < 16 else rows + r) if r < rows else None
    both = np.concatenate([bw, bu])
    want = expected_packed(src_row, nb, k, esz, lambda r: both[r])
    assert got.numel() == want.size
    assert np.array_equal(got.cpu().numpy(), want)
    assert P.spec_packed_bytes(1, 32, 12) == 0 and P.binding.lib.spec_packed_gate_up_bytes(0, 32, 6) == 0      # k not a whole 16-byte piece


def test_gemm_row_is_independent_of_batch(env):
    """A row computed alone (plain decoding) is bit-identical to the same row inside a 60-row tree."""
    torch, P = env
    rng = np.random.default_rng(3)
    x = to_dev(torch, rand_storage(rng, (60, 2048), "bf16"), "bf16")
    w = to_dev(torch, rand_storage(rng, (320, 2048), "bf16", 0.05), "bf16")
    full = P.spec_k_gemm(x, [w], 2)
    for i in (0, 17, 31, 32, 59):
        one = P.spec_k_gemm(x[i:i + 1].contiguous(), [w], 2)
        assert torch.equal(one[:, 0], full[:, i])
    ten = P.spec_k_gemm(x[5:15].contiguous(), [w], 2)
    assert torch.equal(ten, full[:, 5:15])


# the tile a case takes in each of its two calls (partial sums; SwiGLU over the first matrix)
MANY_ROWS = [(129, 8, [31], 1, 256, 256), (129, 136, [32], 1, 128, 128), (255, 256, [225, 64, 40], 1, 128, 128), (257, 904, [520], 2, 128, 128),
             (512, 2056, [4096, 32, 64], 4, 192, 128), (640, 1096, [12290], 2, 128, 128), (1025, 384, [8192], 1, 192, 192),
             (510, 2056, [15990], 2, 256, 256), (509, 1160, [9010, 22000, 990], 1, 256, 192), (2045, 264, [7990], 1, 256, 256),
             (2045, 520, [3970, 20, 40], 2, 256, 256)]


@pytest.mark.parametrize("m,k,rows,n_split,tile,tile_swiglu", MANY_ROWS)
def test_gemm_many_rows_matches_fp64(env, m, k, rows, n_split, tile, tile_swiglu):
    """More than 128 bf16 rows: every tile shape of that launch (128 x 256, 256 x 192, 256 x 256), one row or one weight block
    past a tile, segments that meet inside a tile, K of less than one stage, of 2 / 4 / 6n stages and ragged, K splits; the
    same call on an X that is not 16-byte aligned takes the other path.  fp32 sums of k terms of size 0.05: relative error of
    the whole far below 1e-6 * sqrt(k)."""
    torch, P = env
    sizes = {256: (256, 256), 192: (256, 192), 128: (128, 256)}
    assert P.spec_k_gemm_tile(m, sum((r + 31) // 32 for r in rows), k, n_split) == sizes[tile]
    assert P.spec_k_gemm_tile(m, (rows[0] + 15) // 16, k) == sizes[tile_swiglu]
    g = torch.Generator(device="cuda"); g.manual_seed(case_seed(m, k) & 0xFFFF)
    flat = torch.randn(m * k + 8, device="cuda", generator=g).to(torch.bfloat16)
    ws = [(torch.randn(r, k, device="cuda", generator=g) * 0.05).to(torch.bfloat16) for r in rows]
    for off in (0, 4):
        x = flat[off:off + m * k].view(m, k)
        got = P.spec_k_gemm(x, ws, n_split)
        want = x.double() @ torch.cat(ws).double().t()
        err = got.double().sum(0) - want
        assert err.abs().max() <= 1e-6 * np.sqrt(k) * max(1.0, float(want.abs().max()))
        act = P.spec_k_gemm_swiglu(x, ws[0], ws[0].flip(0)).double()
        gate, up = want[:, :rows[0]], want[:, :rows[0]].flip(1)
        ref = gate * torch.sigmoid(gate) * up
        assert ((act - ref).abs() <= 2.0 ** -8 * ref.abs() + 1e-5 * np.sqrt(k)).all()


# m, k, weight rows, whole 256 x 256 tiles of the fullest XCD as the launch plans them, of all: none, one round, two; with and without a ragged end of up
# to 128 rows, lists of XCDs that differ by one weight tile, a last full tile of 129 .. 255 rows
SPLIT_TILES = [(600, 264, 20500, 0, 22), (700, 520, 20510, 32, 33), (1333, 264, 20600, 32, 55), (2049, 264, 16500, 64, 72), (2300, 136, 7000, 32, 36),
               (2047, 264, 18499, 64, 80)]


@pytest.mark.parametrize("m,k,rows,whole,tiles", SPLIT_TILES)
def test_gemm_whole_and_half_tiles_match_fp64_and_single_rows(env, m, k, rows, whole, tiles):
    """Launches whose last round runs in tiles of half the tokens: against fp64 (fp32 sums of k terms of size 0.05), and rows at the edges of
    tiles and halves have the bits they have alone; SwiGLU over a matrix of the same block count likewise."""
    torch, P = env
    assert P.spec_k_gemm_tile(m, (rows + 31) // 32, k) == (256, 256)
    assert P.spec_k_gemm_plan(m, (rows + 31) // 32, k) == P.spec_k_gemm_plan(m, (rows // 2 + 15) // 16, k) == (0, whole, tiles)
    g = torch.Generator(device="cuda"); g.manual_seed(case_seed("split", m, rows) & 0xFFFF)
    x = torch.randn(m, k, device="cuda", generator=g).to(torch.bfloat16)
    w = (torch.randn(rows, k, device="cuda", generator=g) * 0.05).to(torch.bfloat16)
    got = P.spec_k_gemm(x, [w], 1)[0]
    want = x.double() @ w.double().t()
    assert (got.double() - want).abs().max() <= 1e-6 * np.sqrt(k) * max(1.0, float(want.abs().max()))
    gate, up = w[:rows // 2], w[rows // 2:rows // 2 * 2]
    act = P.spec_k_gemm_swiglu(x, gate, up)
    gd, ud = want[:, :rows // 2], want[:, rows // 2:rows // 2 * 2]
    ref = gd * torch.sigmoid(gd) * ud
    assert ((act.double() - ref).abs() <= 2.0 ** -8 * ref.abs() + 1e-5 * np.sqrt(k)).all()
    for i in sorted({0, 127, 128, 255, 256, m // 2, m // 256 * 256 - 1, m // 256 * 256, m - 1} & set(range(m))):
        assert torch.equal(P.spec_k_gemm(x[i:i + 1].contiguous(), [w], 1)[0, 0], got[i])
        assert torch.equal(P.spec_k_gemm_swiglu(x[i:i + 1].contiguous(), gate, up)[0], act[i])


# m, k, weight rows, splits, wavefronts of a workgroup in the two calls (partial sums; SwiGLU, never split): eight with five to eight blocks spread over the
# compute units (the last wave of some without a block), with four blocks and few rows, and with eight adjacent ones; each beside the nearest size that
# keeps workgroups of four
WIDE_WGS = [(1, 264, 32790, 1, 8, 8), (33, 520, 41270, 1, 8, 8), (60, 264, 65500, 1, 8, 8), (100, 264, 57330, 1, 8, 8), (128, 136, 65540, 1, 4, 4),
            (65, 264, 128256, 1, 8, 8), (64, 264, 128256, 1, 4, 4), (32, 1032, 28672, 1, 8, 8), (33, 1032, 28672, 1, 4, 4), (10, 1032, 28640, 1, 4, 4),
            (7, 2056, 14500, 2, 8, 4), (40, 2056, 20500, 2, 8, 4)]


# every count of 256-k slabs around the period of three: whole, and with one 128-k tile in the last slab; waves without a block; 1, 2 and 4 token blocks
STREAM_K = [(m, 256 * slabs - cut, *((70, 1, 4, 4) if slabs % 2 else (33000, 1, 8, 8))) for m in (9, 60, 100) for slabs in range(1, 9) for cut in (0, 136)]


@pytest.mark.parametrize("m,k,rows,n_split,waves,waves_swiglu", WIDE_WGS + STREAM_K)
def test_gemm_streams_match_fp64_and_single_rows(env, m, k, rows, n_split, waves, waves_swiglu):
    """Against fp64 (fp32 sums of k terms of size 0.05), and every row has the bits it has beside others; SwiGLU over as many blocks likewise."""
    torch, P = env
    assert P.spec_k_gemm_plan(m, (rows + 31) // 32, k, n_split) == (waves, 0, 0)
    assert P.spec_k_gemm_plan(m, (rows // 2 + 15) // 16, k) == (waves_swiglu, 0, 0)
    g = torch.Generator(device="cuda"); g.manual_seed(case_seed("wide", m, rows) & 0xFFFF)
    x = torch.randn(m, k, device="cuda", generator=g).to(torch.bfloat16)
    w = (torch.randn(rows, k, device="cuda", generator=g) * 0.05).to(torch.bfloat16)
    got = P.spec_k_gemm(x, [w], n_split)
    want = x.double() @ w.double().t()
    assert (got.double().sum(0) - want).abs().max() <= 1e-6 * np.sqrt(k) * max(1.0, float(want.abs().max()))
    gate, up = w[:rows // 2], w[rows // 2:rows // 2 * 2]
    act = P.spec_k_gemm_swiglu(x, gate, up)
    gd, ud = want[:, :rows // 2], want[:, rows // 2:rows // 2 * 2]
    ref = gd * torch.sigmoid(gd) * ud
    assert ((act.double() - ref).abs() <= 2.0 ** -8 * ref.abs() + 1e-5 * np.sqrt(k)).all()
    few = min(rows, 4096)                                     # few blocks: workgroups of four wavefronts
    assert torch.equal(P.spec_k_gemm(x, [w[:few].contiguous()], n_split), got[:, :, :few])
    for i in sorted({0, m // 2, m - 1}):
        assert torch.equal(P.spec_k_gemm(x[i:i + 1].contiguous(), [w], n_split)[:, 0], got[:, i])
        assert torch.equal(P.spec_k_gemm_swiglu(x[i:i + 1].contiguous(), gate, up)[0], act[i])


# m, k, weight rows of the segments, splits, weight rows of the tile: one round of 256 x 192 where 128 x 256 takes two (the 8B QKV projection, whole
# and ragged, K ranges of unequal length among them), and shapes on the other side of the rule
FOLDED = [(2048, 4096, (4096, 1024, 1024), 2, 192), (1999, 1288, (4096, 900, 1022), 2, 192), (1333, 2064, (4100, 1024, 1022), 3, 192),
          (1025, 1032, (7600, 1024), 2, 192), (2048, 2056, (4096,), 4, 256), (300, 776, (700,), 3, 256), (129, 520, (40,), 2, 256)]


@pytest.mark.parametrize("m,k,rows,n_split,tile", FOLDED)
def test_gemm_folded_ranges_have_the_bits_of_the_split_sums(env, m, k, rows, n_split, tile):
    torch, P = env
    g = torch.Generator(device="cuda"); g.manual_seed(case_seed("fold", m, k) & 0xFFFF)
    x = torch.randn(m, k, device="cuda", generator=g).to(torch.bfloat16)
    ws = [(torch.randn(r, k, device="cuda", generator=g) * 0.05).to(torch.bfloat16) for r in rows]
    got, tile_rows = P.spec_k_gemm_folded(x, ws, n_split)
    assert tile_rows == tile
    part = P.spec_k_gemm(x, ws, n_split)
    want = part[0]
    for s in range(1, n_split):
        want = want + part[s]
    assert torch.equal(got, want)


def make_tree(rng, rows, max_depth):
    par = np.full(rows, -1, np.int32)
    dep = np.zeros(rows, np.int32)
    for j in range(1, rows):
        cand = [p for p in range(j) if dep[p] < max_depth]
        par[j] = cand[int(rng.integers(len(cand)))]
        dep[j] = dep[par[j]] + 1
    anc = np.zeros((rows, 16), np.int32)
    for j in range(rows):
        a, q = j, dep[j]
        while a >= 0:
            anc[j, q] = a
            a, q = par[a], q - 1
    return par, dep, anc


def attention_error_ok(got, want, dtype, v_max):
    """got, want: arrays of the same shape.  fp32 storage: 1e-5.  bf16 storage: keys and values are exact, queries and
    probabilities enter the matrix cores as bf16 hi + lo pairs (relative 2^-16), sums are fp32, and the output is
    rounded to bf16 (relative 2^-9 of the element), so per element |err| <= 2^-8 |want| + 2^-12 max|v| and over the
    whole output rms(err) <= 2^-9 rms(want) + 1e-4.  With outputs of 0.03 .. 0.07 (averages over hundreds of
    unit-variance values) this is a few 1e-4: a dropped block of keys changes the output by several 1e-3."""
    err = np.abs(got - want)
    if dtype == "fp32":
        return err.max() < 1e-5
    per_elem = (err <= 2.0 ** -8 * np.abs(want) + 2.0 ** -12 * v_max).all()
    rms_ok = np.sqrt((err ** 2).mean()) <= 2.0 ** -9 * np.sqrt((want ** 2).mean()) + 1e-4
    return bool(per_elem and rms_ok)


ATTN_CASES = [
    # dtype, hq, hkv, hd, base, rows, tree?, query scale
    ("fp32", 4, 4, 64, 32, 16, True),
    ("fp32", 4, 2, 64, 0, 7, True),
    ("fp32", 8, 1, 128, 65, 16, True),
    ("fp32", 4, 4, 64, 250, 16, True),          # rows straddle the 256-position part boundary
    ("fp32", 4, 4, 64, 0, 64, False),           # prefill chunk from an empty cache
    ("bf16", 8, 8, 128, 511, 60, True),
    ("bf16", 8, 2, 128, 700, 60, True),
    ("bf16", 8, 1, 128, 63, 1, True),           # a single row (plain decoding)
    ("bf16", 4, 4, 128, 192, 64, False),        # chain crossing a part boundary
    ("fp32", 2, 1, 64, 1010, 24, True),         # rows straddle position 1024, where the parts become 256 keys long
    ("fp32", 2, 2, 64, 1500, 8, True),          # several of the longer parts, the last one ragged (vector path)
    ("bf16", 4, 2, 128, 1290, 40, True),        # the same on the matrix-core path
    ("bf16", 4, 2, 128, 1290, 40, True, 6.0),   # peaked scores: a few keys carry the row, outputs of order one
    ("bf16", 8, 1, 128, 2600, 12, True),        # 8 query heads per kv head (the 70B head layout), several far parts
    ("bf16", 2, 2, 64, 1100, 33, True, 6.0),    # head dim 64 on the matrix-core path
]


@pytest.mark.parametrize("case", ATTN_CASES, ids=lambda c: "-".join(str(x) for x in c))
def test_attention_matches_oracle(env, case):
    torch, P = env
    dtype, hq, hkv, hd, base, rows, is_tree = case[:7]
    q_scale = case[7] if len(case) > 7 else 1.0
    rng = np.random.default_rng(case_seed(*case))
    slots = base + rows
    q = rand_storage(rng, (rows, hq * hd), dtype, q_scale)
    kc = rand_storage(rng, (slots, hkv * hd), dtype)
    vc = rand_storage(rng, (slots, hkv * hd), dtype)
    if is_tree:
        par, dep, anc = make_tree(rng, rows, 6)
    else:
        dep, anc = np.arange(rows, dtype=np.int32), None
    out = P.spec_k_attention(to_dev(torch, q, "fp32"), to_dev(torch, kc, dtype), to_dev(torch, vc, dtype), base,
                             torch.from_numpy(dep).cuda(), None if anc is None else torch.from_numpy(anc).cuda(), hq, hkv, hd)
    torch.cuda.synchronize()
    got = out.float().cpu().numpy().reshape(rows, hq, hd).astype(np.float64)
    g = hq // hkv
    k3, v3 = kc.reshape(slots, hkv, hd).astype(np.float64), vc.reshape(slots, hkv, hd).astype(np.float64)
    q3 = q.reshape(rows, hq, hd).astype(np.float64)
    want = np.zeros_like(got)
    for i in range(rows):
        vis = list(range(base)) + ([base + a for a in anc[i, :dep[i] + 1]] if is_tree else list(range(base, base + i + 1)))
        for h in range(hq):
            want[i, h] = attention_row(q3[i, h], k3[vis, h // g], v3[vis, h // g])
    assert attention_error_ok(got, want, dtype, np.abs(vc).max())


def test_attention_tree_row_equals_compacted_chain_row(env):
    """Bit-exactness by construction: a tree row gives the same bits as the same query over a cache in
    which its path has been moved to consecutive slots (what plain decoding sees after compaction)."""
    torch, P = env
    rng = np.random.default_rng(9)
    hq, hkv, hd, base, rows = 8, 2, 128, 300, 24
    par, dep, anc = make_tree(rng, rows, 5)
    q = to_dev(torch, rand_storage(rng, (rows, hq * hd), "bf16"), "fp32")
    kc = to_dev(torch, rand_storage(rng, (base + rows, hkv * hd), "bf16"), "bf16")
    vc = to_dev(torch, rand_storage(rng, (base + rows, hkv * hd), "bf16"), "bf16")
    tree_out = P.spec_k_attention(q, kc, vc, base, torch.from_numpy(dep).cuda(), torch.from_numpy(anc).cuda(), hq, hkv, hd)
    for i in (0, 5, rows - 1):
        path = [base + a for a in anc[i, :dep[i] + 1]]
        kc2, vc2 = kc.clone(), vc.clone()
        for d_, s in enumerate(path):
            kc2[base + d_], vc2[base + d_] = kc[s], vc[s]
        one = P.spec_k_attention(q[i:i + 1].contiguous(), kc2, vc2, base + int(dep[i]), torch.zeros(1, dtype=torch.int32).cuda(),
                                 None, hq, hkv, hd)
        assert torch.equal(one[0], tree_out[i])


@pytest.mark.parametrize("hq,hkv,hd,base,rows", [(16, 16, 64, 95, 90), (8, 4, 64, 200, 160), (8, 8, 128, 100, 90), (4, 4, 64, 380, 140)])
def test_fp32_attention_rows_alone_have_the_bits_of_many(env, hq, hkv, hd, base, rows):
    # few rows over up to 512 keys: one launch whose wavefronts take a part each; many rows, or more keys: partial outputs in memory and a merge.  Rows
    # across the edges of the 128-key parts and of their 64-key halves
    torch, P = env
    rng = np.random.default_rng(hq + base)
    q = to_dev(torch, rand_storage(rng, (rows, hq * hd), "fp32"), "fp32")
    kc = to_dev(torch, rand_storage(rng, (base + rows, hkv * hd), "fp32"), "fp32")
    vc = to_dev(torch, rand_storage(rng, (base + rows, hkv * hd), "fp32"), "fp32")
    dep = torch.arange(rows, dtype=torch.int32, device="cuda")
    run = lambda a, b: P.spec_k_attention(q[a:b].contiguous(), kc, vc, base, dep[a:b].contiguous(), None, hq, hkv, hd)
    whole = run(0, rows)
    for a in range(0, rows, 5):
        assert torch.equal(run(a, min(a + 5, rows)), whole[a:a + 5])


@pytest.mark.parametrize("rows,vocab,k", [(1, 1024, 4), (4, 1024, 4), (10, 32000, 10), (10, 128256, 10), (3, 5000, 16), (16, 4097, 7)])
def test_topk_logprob_matches_oracle(env, rows, vocab, k):
    torch, P = env
    rng = np.random.default_rng(vocab + rows)
    logits = (rng.standard_normal((rows, vocab)) * 1.3).astype(np.float32)
    logits[0, 7] = logits[0, 900] = logits[0].max() + 1.0          # a tie for first place: lower index wins
    if rows > 1:
        logits[-1, vocab - 1] = logits[-1].max() + 2.0             # the last (ragged-slice) entry wins
    tok, lp = P.spec_k_topk_logprob(torch.from_numpy(logits).cuda(), k)
    torch.cuda.synchronize()
    tok, lp = tok.cpu().numpy(), lp.cpu().numpy()
    want_lp = log_softmax(logits.astype(np.float64))
    for r in range(rows):
        want = top_k(logits[r], k)
        assert list(tok[r]) == list(want)
        assert np.abs(lp[r] - want_lp[r, want]).max() < 5e-6
    assert tok[0, 0] == 7 and tok[0, 1] == 900 and (rows == 1 or tok[-1, 0] == vocab - 1)


@pytest.mark.parametrize("rows,vocab,k", [(2, 16, 16), (3, 1023, 16), (4, 1024, 16), (4, 1025, 16), (1, 300, 1)])
def test_topk_logprob_around_the_short_slice(env, rows, vocab, k):
    """Up to 1024 tokens a thread holds four of them, beyond that sixteen."""
    torch, P = env
    logits = np.random.default_rng(vocab).standard_normal((rows, vocab)).astype(np.float32)
    logits[0, vocab // 2] = logits[0, vocab - 1] = 9.0                # equal: lower index first
    tok, lp = (t.cpu().numpy() for t in P.spec_k_topk_logprob(torch.from_numpy(logits).cuda(), k))
    want_lp = log_softmax(logits.astype(np.float64))
    for r in range(rows):
        want = top_k(logits[r], k)
        assert list(tok[r][:k]) == list(want) and np.abs(lp[r][:k] - want_lp[r, want]).max() < 5e-6


@pytest.mark.parametrize("name,rows,k,n_split", [("70b-down", 8192, 28672, 4), ("70b-gateup-slice", 4096, 8192, 1), ("13b-qkv-slice", 5120, 5120, 2)])
def test_gemm_large_shapes_sampled_against_oracle(env, name, rows, k, n_split):
    """Matrix shapes of the largest configurations, M = 60: sampled output columns against fp64 dot products."""
    torch, P = env
    g = torch.Generator(device="cuda"); g.manual_seed(5)
    x = (torch.randn(60, k, device="cuda", generator=g)).to(torch.bfloat16)
    w = (torch.randn(rows, k, device="cuda", generator=g) * 0.02).to(torch.bfloat16)
    got = P.spec_k_gemm(x, [w], n_split).sum(dim=0).cpu().numpy().astype(np.float64)
    cols = [0, 1, 31, 32, rows // 2 + 5, rows - 33, rows - 1]
    xs = x.float().cpu().numpy().astype(np.float64)
    for c in cols:
        want = xs @ w[c].float().cpu().numpy().astype(np.float64)
        assert np.abs(got[:, c] - want).max() < 2e-3


@pytest.mark.parametrize("vocab,k", [(40, 16), (262144, 16), (262145, 16), (300000, 11)])
def test_topk_logprob_merge_of_slices(env, vocab, k):
    """One slice, 64 (a list per lane) and more (several): rows whose best entries sit in one slice, are spread one per slice, tie across
    slices, and a row of three finite entries (the rest follow by index)."""
    torch, P = env
    rng = np.random.default_rng(vocab)
    logits = rng.standard_normal((4, vocab)).astype(np.float32)
    logits[0, vocab - 20:] += 10.0
    logits[1, ::4096] += 12.0
    logits[2] = np.round(logits[2])
    logits[3] = -np.inf
    logits[3, [vocab - 1, vocab // 2, 5]] = [1.0, 2.0, 1.0]
    tok, lp = P.spec_k_topk_logprob(torch.from_numpy(logits).cuda(), k)
    torch.cuda.synchronize()
    tok, lp = tok.cpu().numpy(), lp.cpu().numpy()
    for r in range(4):
        want = np.lexsort((np.arange(vocab), -logits[r].astype(np.float64)))[:k]
        assert list(tok[r]) == list(want)
        x = logits[r].astype(np.float64)
        want_lp = x - x.max() - np.log(np.exp(x - x.max()).sum())
        fin = np.isfinite(want_lp[want])
        assert np.abs(lp[r][fin] - want_lp[want][fin]).max() < 5e-6 and np.isneginf(lp[r][~fin]).all()


@pytest.mark.parametrize("q_scale", [1.0, 6.0], ids=["flat", "peaked"])
def test_attention_long_context_matches_oracle(env, q_scale):
    """Long-KV verify of the LLaMA3-8B configuration: 4100 cached keys (eight 128-key parts and thirteen 256-key parts
    on the matrix cores), GQA 4:1, sampled rows and heads; near-uniform and peaked score distributions."""
    torch, P = env
    rng = np.random.default_rng(77)
    hq, hkv, hd, base, rows = 8, 2, 128, 4100, 60
    par, dep, anc = make_tree(rng, rows, 6)
    q = rand_storage(rng, (rows, hq * hd), "bf16", q_scale)
    kc = rand_storage(rng, (base + rows, hkv * hd), "bf16")
    vc = rand_storage(rng, (base + rows, hkv * hd), "bf16")
    out = P.spec_k_attention(to_dev(torch, q, "fp32"), to_dev(torch, kc, "bf16"), to_dev(torch, vc, "bf16"), base,
                             torch.from_numpy(dep).cuda(), torch.from_numpy(anc).cuda(), hq, hkv, hd)
    got_all = out.float().cpu().numpy().reshape(rows, hq, hd).astype(np.float64)
    k3, v3 = kc.reshape(-1, hkv, hd).astype(np.float64), vc.reshape(-1, hkv, hd).astype(np.float64)
    q3 = q.reshape(rows, hq, hd).astype(np.float64)
    got, want = [], []
    for i in (0, 1, 17, 40, 59):
        vis = list(range(base)) + [base + a for a in anc[i, :dep[i] + 1]]
        for h in (0, 3, 4, 7):
            want.append(attention_row(q3[i, h], k3[vis, h // 4], v3[vis, h // 4]))
            got.append(got_all[i, h])
    assert attention_error_ok(np.array(got), np.array(want), "bf16", np.abs(vc).max())


@pytest.mark.parametrize("rows,hq,hkv,hd,base,order", [(257, 4, 4, 128, 0, "chain"), (256, 8, 8, 64, 63, "chain"), (300, 8, 1, 128, 64, "chain"),
                                                       (289, 16, 8, 128, 1000, "chain"), (260, 4, 2, 64, 5, "reversed"), (270, 2, 1, 128, 130, "scattered"),
                                                       # launches large enough for one walk over all keys
                                                       (300, 32, 4, 128, 0, "chain"), (257, 64, 8, 64, 1000, "reversed"), (270, 64, 64, 128, 130, "scattered")])
def test_attention_of_a_long_chain_matches_fp64(env, rows, hq, hkv, hd, base, order):
    """Hundreds of rows without a tree (prefill), few heads (blocks of 256 rows with partials) and many (one walk over all keys, no
    partials): ragged row tiles and key blocks, grouped heads, head counts with and without the placement over
    eight L2s, empty and long caches, rows that do not stand in order of position (the caller may pass any depths); peaked
    scores so that the running maximum moves."""
    torch, P = env
    rng = np.random.default_rng(case_seed("chain", rows, hq, hd))
    depth = {"chain": np.arange(rows), "reversed": np.arange(rows)[::-1], "scattered": rng.integers(0, rows, rows)}[order].astype(np.int32)
    q = rand_storage(rng, (rows, hq * hd), "bf16", 4.0) * 1.01            # queries are fp32: not exact in bf16
    kc = rand_storage(rng, (base + rows, hkv * hd), "bf16")
    vc = rand_storage(rng, (base + rows, hkv * hd), "bf16")
    out = P.spec_k_attention(to_dev(torch, q, "fp32"), to_dev(torch, kc, "bf16"), to_dev(torch, vc, "bf16"), base,
                             torch.from_numpy(depth.copy()).cuda(), None, hq, hkv, hd)
    got = out.float().cpu().numpy().reshape(rows, hq, hd).astype(np.float64)
    q3 = q.astype(np.float32).reshape(rows, hq, hd).astype(np.float64)
    k3, v3 = kc.reshape(-1, hkv, hd).astype(np.float64), vc.reshape(-1, hkv, hd).astype(np.float64)
    want = np.empty_like(got)
    hidden = np.arange(base + rows)[None] > (base + depth)[:, None]
    for h in range(hq):
        sc = q3[:, h] @ k3[:, h * hkv // hq].T / np.sqrt(hd)
        sc[hidden] = -np.inf
        p = np.exp(sc - sc.max(1, keepdims=True))
        want[:, h] = p @ v3[:, h * hkv // hq] / p.sum(1, keepdims=True)
    assert attention_error_ok(got, want, "bf16", np.abs(vc).max())


@pytest.mark.parametrize("rows,hq,hkv,hd,base,order", [(520, 32, 8, 128, 0, "chain"), (300, 64, 8, 128, 1000, "chain"), (200, 64, 64, 128, 0, "chain"),
                                                       (640, 32, 8, 128, 3500, "chain"), (700, 16, 16, 64, 0, "chain"), (1300, 16, 16, 64, 100, "chain"),
                                                       (513, 40, 40, 128, 15, "reversed"), (777, 32, 4, 64, 130, "scattered")])
def test_attention_row_is_independent_of_the_other_rows(env, rows, hq, hkv, hd, base, order):
    """A bf16 row's bits are those it has alone or among few rows, whichever path a long chain takes (one launch over all keys, or
    blocks of 256 rows with partials): rows with a tail only, with up to and more than seven parts before the tail, near and far
    parts; one row in a tile, half-filled wavefronts; positions out of order."""
    torch, P = env
    g = torch.Generator(device="cuda"); g.manual_seed(case_seed("rows", rows, hq, hd) & 0xFFFF)
    q = torch.randn(rows, hq * hd, device="cuda", generator=g) * 3.0
    kc = torch.randn(base + rows, hkv * hd, device="cuda", generator=g).to(torch.bfloat16)
    vc = torch.randn(base + rows, hkv * hd, device="cuda", generator=g).to(torch.bfloat16)
    dep = torch.arange(rows, dtype=torch.int32, device="cuda")
    if order == "reversed":
        dep = dep.flip(0).contiguous()
    elif order == "scattered":
        dep = torch.randint(0, rows, (rows,), generator=g, device="cuda", dtype=torch.int32)
    run = lambda a, b: P.spec_k_attention(q[a:b].contiguous(), kc, vc, base, dep[a:b].contiguous(), None, hq, hkv, hd)
    whole = run(0, rows).view(torch.int16)
    few = torch.cat([run(a, min(a + 150, rows)) for a in range(0, rows, 150)]).view(torch.int16)
    assert torch.equal(whole, few)
    for i in (0, 15, 16, rows // 2, rows - 1):
        assert torch.equal(run(i, i + 1).view(torch.int16)[0], whole[i])


@pytest.mark.parametrize("shape", ["rising", "falling", "one far peak", "steps"])
@pytest.mark.parametrize("rows,hq,hkv,hd,base", [(3, 4, 1, 128, 1500), (260, 32, 8, 128, 300), (260, 32, 32, 64, 300)])
def test_attention_where_references_move(env, shape, rows, hq, hkv, hd, base):
    """Scores that climb, fall or jump by far more than 2^8 along the keys, so that the reference of a part moves again and again, or never from
    its first block, and that of the row between parts: against fp64, and a row of many has the bits it has alone."""
    torch, P = env
    n = base + rows
    g = torch.Generator(device="cuda"); g.manual_seed(case_seed("move", shape, rows, hd) & 0xFFFF)
    pos = torch.arange(n, device="cuda", dtype=torch.float64) / n
    level = {"rising": 60 * pos, "falling": -60 * pos, "one far peak": 50.0 * (torch.arange(n, device="cuda") == 33), "steps": 9.0 * (torch.arange(n, device="cuda") // 48 % 5)}[shape]
    direction = torch.randn(hkv * hd, device="cuda", generator=g).sign()
    kc = (torch.randn(n, hkv * hd, device="cuda", generator=g) * 0.3 + (level / hd ** 0.5)[:, None].float() * direction).to(torch.bfloat16)
    vc = torch.randn(n, hkv * hd, device="cuda", generator=g).to(torch.bfloat16)
    q = direction.view(hkv, 1, hd).expand(hkv, hq // hkv, hd).reshape(1, hq * hd).repeat(rows, 1) * (1 + 0.1 * torch.randn(rows, 1, device="cuda", generator=g))
    dep = torch.arange(rows, dtype=torch.int32, device="cuda")
    run = lambda a, b: P.spec_k_attention(q[a:b].contiguous(), kc, vc, base, dep[a:b].contiguous(), None, hq, hkv, hd)
    got = run(0, rows)
    for i in (0, rows // 2, rows - 1):
        assert torch.equal(run(i, i + 1)[0], got[i])
    k3, v3 = kc.double().view(n, hkv, hd).repeat_interleave(hq // hkv, 1), vc.double().view(n, hkv, hd).repeat_interleave(hq // hkv, 1)
    sc = torch.bmm(q.double().view(rows, hq, hd).transpose(0, 1).contiguous(), k3.permute(1, 2, 0).contiguous()) / hd ** 0.5
    sc.masked_fill_(torch.arange(n, device="cuda")[None, None] > (base + dep)[None, :, None], -np.inf)
    want = torch.bmm(torch.softmax(sc, -1), v3.transpose(0, 1).contiguous()).transpose(0, 1).contiguous().view(rows, hq, hd)
    # queries and probabilities enter as hi + lo pairs, a score's relative error of 2^-16 is an absolute one of 60 * 2^-16 in the exponent
    assert ((got.double().view_as(want) - want).abs() <= 2.0 ** -8 * want.abs() + 2.0 ** -9 * float(vc.double().abs().max())).all()
