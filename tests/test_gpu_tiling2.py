"""GPU parity of the second tiling of the many-token kernel (2-D grid of wavefronts, expansion shared through LDS,
persistent workgroups) and of its split of K across workgroups (Sec. 1: both regimes have to be served; Sec. 3, Eq. 10,
Eq. 4, Eq. 11: the layer itself), against the CPU oracle on the same seeded inputs: every workgroup tile, ragged edges,
persistent grids smaller than the tile count (several tiles per workgroup), group sizes of one or more chunks, the -8
marks, the exact-integer case bit for bit, power-of-two scales through the block-scaled MFMA, and w4a8_linear with a
workspace on the shapes w4a8_linear_workspace_bytes() names.  Tolerances as in test_gpu_parity.py."""
import numpy as np
import pytest
import torch

from oracle import w4a8_oracle as o
from paper_2505_14638_amd import binding as B
from paper_2505_14638_amd import synthetic as syn

from test_gpu_parity import bf16_bits, check_outputs, dev, host, say

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
POW2_PATH = 2 + 16 * 3
TILES = (0, 1, 2, 3, 4, 5)


def run_variant(x8_d, sx_d, packed, scales, n, g, path, p0, p1):
    m = x8_d.shape[0]
    y32 = torch.full((m, n), float("nan"), dtype=torch.float32, device=DEV)
    y16 = torch.full((m, n), float("nan"), dtype=torch.bfloat16, device=DEV)
    B.linear_variant(x8_d, sx_d, packed, scales, n, g, y32, path, p0, p1)
    B.linear_variant(x8_d, sx_d, packed, scales, n, g, y16, path, p0, p1)
    return host(y32), bf16_bits(y16)


def realistic(seed, m, k, n, g, frac=0.02):
    rng = np.random.default_rng(seed)
    w = syn.make_weights(rng, n, k)
    x = syn.make_activations(rng, m, k, frac, 20.0)
    s_x = syn.static_act_scale(x)
    q, s_w = o.rtn_quantize_weights(w, g)
    x8 = o.quantize_act(x, s_x)
    ref, a = o.linear_ref(x8, s_x, q, s_w, g)
    packed, scales = B.pack_weights(dev(w), g, B.LAYOUT_TILED)
    return x8, s_x, packed, scales, ref, a


def integer_case(seed, m, k, n, g, minus_eight):
    """Small-integer activations and power-of-two scales: every partial sum is exact in float32 in any order, so the
    float32 output must equal the integer matmul bit for bit (also across a split of K)."""
    rng = np.random.default_rng(seed)
    ng = k // g
    xi = rng.integers(-4, 5, size=(m, k))
    x8 = o.e4m3_encode(xi.astype(np.float32))
    q = rng.integers(-7, 8, size=(n, k)).astype(np.int8)
    if minus_eight:
        marked = rng.random((n, ng)) < 0.25
        marked[:16] = False
        for nn, gg in zip(*np.nonzero(marked)):
            q[nn, gg * g + rng.choice(g, size=rng.integers(1, 4), replace=False)] = -8
    e = rng.integers(-1, 2, size=(n, ng))
    s_w = np.ldexp(1.0, e).astype(np.float32)
    part = np.einsum("mgk,ngk->mng", xi.reshape(m, ng, g).astype(np.int64), q.reshape(n, ng, g).astype(np.int64))
    want = (0.5 * (part * np.ldexp(1.0, e)[None]).sum(axis=2)).astype(np.float32)
    packed, scales = B.pack_weights(dev(q), g, B.LAYOUT_TILED, dev(s_w))
    return x8, packed, scales, want


@pytest.mark.parametrize("tile", TILES)
@pytest.mark.parametrize("m,k,n,g,p1", [
    (300, 1024, 520, 512, 0), (513, 256, 144, 256, 0), (70, 128, 20, 128, 0), (257, 640, 130, 128, 0),
    # persistent grids of 8 and 16 workgroups: several tiles per workgroup, the next tile's start inside the epilogue
    (700, 384, 1100, 128, 1 | (8 << 8)), (1300, 640, 600, 128, 3 | (16 << 8)),
])
def test_every_tile_ragged_against_the_oracle(gpu_lib, tile, m, k, n, g, p1):
    x8, s_x, packed, scales, ref, a = realistic([71, m, k, n], m, k, n, g)
    y32, y16 = run_variant(dev(x8), dev(np.array([s_x])), packed, scales, n, g, 2, tile, p1)
    check_outputs(y32, y16, ref, a, f"second tiling, tile {tile}, {m}x{k}x{n} g{g} p1={p1}")


@pytest.mark.parametrize("tile", TILES)
@pytest.mark.parametrize("m,g,minus_eight,p1", [(200, 128, False, 0), (300, 256, True, 0), (600, 128, True, 2 | (8 << 8))])
def test_every_tile_exact_integer_case_bit_for_bit(gpu_lib, tile, m, g, minus_eight, p1):
    k, n = 2048, 304
    x8, packed, scales, want = integer_case([73, m, g], m, k, n, g, minus_eight)
    y32, _ = run_variant(dev(x8), dev(np.array([0.5], np.float32)), packed, scales, n, g, 2, tile, p1)
    assert np.array_equal(y32, want)


@pytest.mark.parametrize("tile", TILES)
@pytest.mark.parametrize("k,g,minus_eight", [(128, 128, True), (256, 128, False), (384, 128, True), (512, 256, True), (640, 128, False),
                                             (768, 384, True), (896, 896, False)])
def test_loops_of_one_to_seven_chunks_bit_for_bit(gpu_lib, tile, k, g, minus_eight):
    """The loops hold two chunks ahead in registers or LDS: fewer chunks than that, one more, odd and even counts; ragged tokens and
    channels, one workgroup and a persistent grid of eight that takes several tiles each."""
    for m, p1 in ((65, 0), (530, 1 | (8 << 8))):
        n = 300
        x8, packed, scales, want = integer_case([79, m, k, g], m, k, n, g, minus_eight)
        y32, _ = run_variant(dev(x8), dev(np.array([0.5], np.float32)), packed, scales, n, g, 2, tile, p1)
        assert np.array_equal(y32, want), (m, p1)


@pytest.mark.parametrize("tile", (1, 4, 5))
def test_power_of_two_scales_on_the_second_tiling(gpu_lib, tile):
    m, k, n, g = 520, 1024, 300, 128
    rng = np.random.default_rng([75, tile])
    w = syn.make_weights(rng, n, k) * np.exp(rng.uniform(-3.0, 3.0, size=(n, 1))).astype(np.float32)
    x = syn.make_activations(rng, m, k, 0.02, 20.0)
    s_x = syn.static_act_scale(x)
    x8 = o.quantize_act(x, s_x)
    q, s = o.rtn_quantize_weights_pow2(w, g)
    ref, a = o.linear_ref(x8, s_x, q, s, g)
    packed, scales = B.pack_weights(dev(w), g, B.LAYOUT_TILED, pow2=True)
    y32, y16 = run_variant(dev(x8), dev(np.array([s_x])), packed, scales, n, g, POW2_PATH, tile, 0)
    check_outputs(y32, y16, ref, a, f"power-of-two scales, tile {tile}")


@pytest.mark.parametrize("k", [128, 1536, 1664])
@pytest.mark.parametrize("fmt", ["two_level", "asym", "asym_two_level"])
def test_256_x_128_tiles_on_either_loop_hold_the_same_bits(gpu_lib, fmt, k):
    """Formats with a table per channel: up to twelve chunks on one loop, from thirteen on on the other.  Every tile sums in the same order, so 512 x 128
    tiles (the one loop at any size) and 128 x 128 (the other) hold the same bits; -8 in a third of the groups of the signed format."""
    m, n, g = 530, 300, 128
    gen = torch.Generator(device=DEV).manual_seed(84)
    sx_d = dev(np.array([0.01], np.float32))
    x8_d = B.quantize_act(torch.randn((m, k), generator=gen, device=DEV), sx_d)
    s = torch.rand((n, k // g), generator=gen, device=DEV) + 0.5
    w_out = torch.rand(n, generator=gen, device=DEV) + 0.5
    if fmt == "two_level":
        low = torch.where(torch.rand((n, k // g), generator=gen, device=DEV) < 0.3, -8, -7).repeat_interleave(g, dim=1)
        q = torch.randint(-8, 8, (n, k), generator=gen, device=DEV).maximum(low).to(torch.int8)
        packed, scales = B.pack_weights(q, g, B.LAYOUT_TILED, s)
    else:
        u = torch.randint(0, 16, (n, k), generator=gen, device=DEV, dtype=torch.uint8)
        packed, scales = B.pack_weights_asym(u, g, s, torch.randint(0, 16, (n, k // g), generator=gen, device=DEV, dtype=torch.uint8))
    for dtype in (torch.float32, torch.bfloat16):
        y = {}
        for tile, p1 in ((0, 0), (5, 0), (2, 0), (2, 1 | (8 << 8))):
            y[tile, p1] = torch.full((m, n), float("nan"), dtype=dtype, device=DEV)
            if fmt == "two_level":
                B.linear_two_level_variant(x8_d, sx_d, packed, scales, w_out, n, g, y[tile, p1], tile, p1)
            else:
                B.linear_asym_variant(x8_d, sx_d, packed, scales, w_out if fmt == "asym_two_level" else None, n, g, y[tile, p1], 2, tile, p1)
        want = y.pop((0, 0))
        assert torch.isfinite(want.float()).all()
        for key, got in y.items():
            assert torch.equal(got, want), key


def test_default_path_takes_the_second_tiling_on_large_grids(gpu_lib):
    """M = 2048 on a 4096-channel layer (activations as in the benchmark configs: 1 % of the channels x 20): w4a8_linear
    routes to the second tiling -- the same bits as the explicit variant, and as the first tiling (one weight band per
    wavefront), whose sums run in the same order."""
    m, k, n, g = 2048, 1024, 4096, 128
    x8, s_x, packed, scales, ref, a = realistic([77], m, k, n, g, frac=0.01)
    sx_d = dev(np.array([s_x]))
    y = B.linear(dev(x8), sx_d, packed, scales, n, g, B.LAYOUT_TILED, out_dtype=torch.float32)
    y32, y16 = run_variant(dev(x8), sx_d, packed, scales, n, g, 2, 4, 0)
    first, _ = run_variant(dev(x8), sx_d, packed, scales, n, g, 1, 16, 1)
    assert np.array_equal(host(y), y32) and np.array_equal(first, y32)
    check_outputs(y32, y16, ref, a, "default path, 2048 x 1024 x 4096")


# ------------------------------------------------------------------------------------------------ K ranges across workgroups
def run_splitk(x8_d, sx_d, packed, scales, n, g, tile, ksplit):
    m = x8_d.shape[0]
    ws = torch.empty(ksplit * m * ((n + 63) // 64 * 64) * 4, dtype=torch.uint8, device=DEV)
    y32 = torch.full((m, n), float("nan"), dtype=torch.float32, device=DEV)
    y16 = torch.full((m, n), float("nan"), dtype=torch.bfloat16, device=DEV)
    B.linear_splitk_variant(x8_d, sx_d, packed, scales, n, g, y32, tile, ksplit, ws)
    B.linear_splitk_variant(x8_d, sx_d, packed, scales, n, g, y16, tile, ksplit, ws)
    return host(y32), bf16_bits(y16)


@pytest.mark.parametrize("tile,ksplit", [(5, 2), (5, 3), (5, 8), (3, 2), (3, 5), (1, 4)])
@pytest.mark.parametrize("m,k,n,g", [(100, 2048, 200, 128), (65, 1152, 136, 128), (300, 1024, 520, 512)])
def test_split_k_ragged_against_the_oracle(gpu_lib, tile, ksplit, m, k, n, g):
    """K ranges that do not divide the chunk count evenly, groups spanning several chunks (a range may end inside a
    group: the group's scale then multiplies two partial sums), ragged tokens and channels."""
    x8, s_x, packed, scales, ref, a = realistic([79, m, k, n], m, k, n, g)
    y32, y16 = run_splitk(dev(x8), dev(np.array([s_x])), packed, scales, n, g, tile, ksplit)
    check_outputs(y32, y16, ref, a, f"split K, tile {tile}, {ksplit} ranges, {m}x{k}x{n} g{g}")


@pytest.mark.parametrize("tile,ksplit", [(5, 2), (5, 7), (3, 16), (1, 3)])
def test_split_k_exact_integer_case_bit_for_bit(gpu_lib, tile, ksplit):
    m, k, n, g = 130, 2048, 304, 128
    x8, packed, scales, want = integer_case([81, tile, ksplit], m, k, n, g, True)
    y32, _ = run_splitk(dev(x8), dev(np.array([0.5], np.float32)), packed, scales, n, g, tile, ksplit)
    assert np.array_equal(y32, want)


@pytest.mark.parametrize("ksplit", [2, 5])
@pytest.mark.parametrize("m,k,n,g", [(100, 2048, 200, 128), (65, 1152, 136, 128), (300, 1024, 520, 512)])
def test_split_k_ragged_on_256_x_128_tiles(gpu_lib, ksplit, m, k, n, g):
    """The tile that w4a8_linear splits 400 and 512 tokens of a down projection with: uneven ranges, ranges that begin inside a group."""
    test_split_k_ragged_against_the_oracle(gpu_lib, 2, ksplit, m, k, n, g)


@pytest.mark.parametrize("ksplit", [2, 5])
def test_split_k_exact_integer_case_on_256_x_128_tiles(gpu_lib, ksplit):
    test_split_k_exact_integer_case_bit_for_bit(gpu_lib, 2, ksplit)


@pytest.mark.parametrize("m", [48, 96, 128, 400])
def test_linear_with_workspace_on_the_down_projection(gpu_lib, m):
    """The Llama-3-8B down projection (K = 14336, N = 4096) at batch sizes where w4a8_linear asks for a workspace (from 41
    tokens on; at 48 the layer without a workspace runs on the few-token kernel): sampled
    token rows x all channels against the oracle, bf16 == RNE(float32), and the same bits on a second call (the order
    of the ranges in the sum is fixed)."""
    k, n = syn.LLAMA3_8B["down"]
    g = 128
    need = B.linear_workspace_bytes(m, k, n, g)
    assert need > 0
    rng = np.random.default_rng([83, m])
    w = syn.make_weights(rng, n, k)
    x = syn.make_activations(rng, m, k, 0.01, 20.0)
    s_x = syn.static_act_scale(x)
    q, s_w = o.rtn_quantize_weights(w, g)
    x8 = o.quantize_act(x, s_x)
    rows = np.unique(np.concatenate([[0, m - 1], rng.integers(0, m, size=14)]))
    ref, a = o.linear_ref(x8[rows], s_x, q, s_w, g)
    packed, scales = B.pack_weights(dev(w), g, B.LAYOUT_TILED)
    ws = torch.empty(need, dtype=torch.uint8, device=DEV)
    sx_d, x8_d = dev(np.array([s_x])), dev(x8)
    y32 = host(B.linear(x8_d, sx_d, packed, scales, n, g, B.LAYOUT_TILED, out_dtype=torch.float32, workspace=ws))
    y16 = bf16_bits(B.linear(x8_d, sx_d, packed, scales, n, g, B.LAYOUT_TILED, out_dtype=torch.bfloat16, workspace=ws))
    check_outputs(y32[rows], y16[rows], ref, a, f"down projection with workspace, M = {m}")
    again = host(B.linear(x8_d, sx_d, packed, scales, n, g, B.LAYOUT_TILED, out_dtype=torch.float32, workspace=ws))
    assert np.array_equal(again.view(np.uint32), y32.view(np.uint32))
    # without a workspace the layer takes the unsplit kernels: same tolerance, different order of the sum
    plain = host(B.linear(x8_d, sx_d, packed, scales, n, g, B.LAYOUT_TILED, out_dtype=torch.float32))
    ok, worst = o.within_tolerance(plain[rows], ref, a)
    say(f"  without workspace: worst err/bound = {worst:.3e}")
    assert ok


def test_linear_with_workspace_at_k_8192(gpu_lib):
    """K = 8192 takes K ranges across workgroups when that gives four or more of them: a narrow layer at 100 tokens through
    w4a8_linear with the workspace it asks for, every output against the oracle."""
    m, k, n, g = 100, 8192, 2048, 128
    need = B.linear_workspace_bytes(m, k, n, g)
    assert need > 0 and B.linear_launch_shape(m, k, n, g, True)[0] == 3 and B.linear_workspace_bytes(m, 4096, n, g) == 0
    x8, s_x, packed, scales, ref, a = realistic([85], m, k, n, g, frac=0.01)
    ws = torch.empty(need, dtype=torch.uint8, device=DEV)
    sx_d, x8_d = dev(np.array([s_x])), dev(x8)
    y32 = host(B.linear(x8_d, sx_d, packed, scales, n, g, B.LAYOUT_TILED, out_dtype=torch.float32, workspace=ws))
    y16 = bf16_bits(B.linear(x8_d, sx_d, packed, scales, n, g, B.LAYOUT_TILED, out_dtype=torch.bfloat16, workspace=ws))
    check_outputs(y32, y16, ref, a, "K = 8192 with workspace")


# ------------------------------------------------------------------------------------- rows that no 16-byte store is aligned to
def into_odd_rows(m, n, dtype, off, pad):
    """A buffer of odd row stride whose payload starts `off` elements in, filled with a byte pattern; (buffer, payload view)."""
    size = torch.empty(0, dtype=dtype).element_size()
    buf = torch.full((m, (n + pad) * size), 0x5A, dtype=torch.uint8, device=DEV).view(dtype)
    return buf, buf[:, off : off + n]


@pytest.mark.parametrize("path,p0,p1", [(2, t, 0) for t in TILES] + [(1, 16, 1), (1, 8, 2), (1, 4, 4)])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_rows_at_odd_addresses_hold_the_same_bits(gpu_lib, path, p0, p1, dtype):
    """Rows at element-aligned addresses hold the bits that 16-byte aligned ones do (the last band ragged: element by
    element), and what lies around them stays as it was."""
    m, k, n, g = 130, 1024, 203, 128
    x8, s_x, packed, scales, _, _ = realistic([79, m, k, n], m, k, n, g)
    x8_d, sx_d = dev(x8), dev(np.array([s_x]))
    want = torch.empty((m, 256), dtype=dtype, device=DEV)[:, :n]
    B.linear_variant(x8_d, sx_d, packed, scales, n, g, want, path, p0, p1)
    for off, pad in ((0, 0), (1, 2), (3, 6)):
        buf, out = into_odd_rows(m, n, dtype, off, pad)
        before = buf.clone()
        B.linear_variant(x8_d, sx_d, packed, scales, n, g, out, path, p0, p1)
        assert torch.equal(out, want), f"offset {off}"
        out.copy_(before[:, off : off + n])
        assert torch.equal(buf.view(torch.uint8), before.view(torch.uint8)), f"written outside the rows, offset {off}"


@pytest.mark.parametrize("m,k,f", [(8, 512, 160), (100, 1024, 240), (1100, 4096, 6144)])
def test_silu_mul_rows_a_megabyte_apart(gpu_lib, m, k, f):
    """The fused gate|up layer takes any row stride of its output, on whichever kernel the sizes lead to."""
    assert B.linear_launch_shape(m, k, 2 * f, 128)[0] == {8: 0, 100: 1, 1100: 2}[m]
    gen = torch.Generator(device=DEV).manual_seed(82)
    sx_d, next_s = dev(np.array([0.01], np.float32)), dev(np.array([0.02], np.float32))
    x8_d = B.quantize_act(torch.randn((m, k), generator=gen, device=DEV), sx_d)
    packed, scales = B.pack_weights(torch.randn((2 * f, k), generator=gen, device=DEV) * 0.02, 128, B.LAYOUT_TILED)
    want = B.linear_silu_mul_fp8_out(x8_d, sx_d, packed, scales, f, 128, next_s)
    far = torch.zeros((m, (1 << 20) + 16), dtype=torch.uint8, device=DEV)
    B.linear_silu_mul_fp8_out(x8_d, sx_d, packed, scales, f, 128, next_s, out=far[:, :f])
    assert torch.equal(far[:, :f], want) and int(far[:, f:].max()) == 0


@pytest.mark.parametrize("m,k,n,path", [(100, 1024, 480, 1), (600, 1024, 8224, 1), (700, 1024, 16416, 2), (1000, 2048, 6176, 2)])
def test_fp8_rows_at_odd_addresses_hold_the_same_bits(gpu_lib, m, k, n, path):
    """The E4M3 and the SiLU*mul output of either tiling (256 x 256 and 256 x 128 tiles of the second)."""
    g = 128
    assert B.linear_launch_shape(m, k, n, g)[0] == path
    gen = torch.Generator(device=DEV).manual_seed(80)
    sx_d, next_s = dev(np.array([0.01], np.float32)), dev(np.array([0.02], np.float32))
    x8_d = B.quantize_act(torch.randn((m, k), generator=gen, device=DEV), sx_d)
    packed, scales = B.pack_weights(torch.randn((n, k), generator=gen, device=DEV) * 0.02, g, B.LAYOUT_TILED)
    for call, width in ((B.linear_fp8_out, n), (B.linear_silu_mul_fp8_out, n // 2)):
        size = n if width == n else n // 2
        want = call(x8_d, sx_d, packed, scales, size, g, next_s, out=torch.empty((m, width), dtype=torch.uint8, device=DEV))
        buf, out = into_odd_rows(m, width, torch.uint8, 5, 9)
        before = buf.clone()
        call(x8_d, sx_d, packed, scales, size, g, next_s, out=out)
        assert torch.equal(out, want)
        out.copy_(before[:, 5 : 5 + width])
        assert torch.equal(buf, before)


# ------------------------------------------------------------------------------------- FP8 outputs of the second tiling
def same_e4m3(a, b):
    """The same bytes, a NaN being one with either sign."""
    nan = (a & 0x7F) == 0x7F
    return torch.equal(nan, (b & 0x7F) == 0x7F) and torch.equal(a.masked_fill(nan, 0x7F), b.masked_fill(nan, 0x7F))


@pytest.mark.parametrize("tile,m,k,n", [(0, 257, 128, 30048), (1, 520, 128, 15488), (2, 390, 896, 15488), (4, 390, 128, 34208)])
def test_fp8_outputs_of_every_tile_equal_the_unfused_sequence(gpu_lib, tile, m, k, n):
    """Ragged sizes that the launch choice sends to each tile: w4a8_linear_fp8_out against linear (bf16) then quantize_act, and
    w4a8_linear_silu_mul_fp8_out against linear, silu_mul, quantize_act -- kernels of their own, which divide the general way.  Ordinary
    scales and ones outside 2^-30 .. 2^30, quotients far beyond 448, gates of hundreds and beyond 2^60, infinities, NaN, a scale of zero."""
    g = 128
    assert B.linear_launch_shape(m, k, n, g)[:2] == (2, tile)
    gen = torch.Generator(device=DEV).manual_seed(83)
    x8_d = B.quantize_act(torch.randn((m, k), generator=gen, device=DEV), dev(np.array([0.05], np.float32)))
    x8_d[::37] = 0                                               # outputs of zero: NaN under an infinite activation scale
    w = torch.randn((n, k), generator=gen, device=DEV) * 0.02
    packed, scales = B.pack_weights(w, g, B.LAYOUT_TILED)
    paired, paired_s = B.pack_weights(B.interleave_gate_up(w), g, B.LAYOUT_TILED)
    seen = set()
    for s_x in (0.05, 2.0, 2.0 ** -45, 2.0 ** 45, 2.0 ** 62, 3e38, float("inf")):
        sx_d = dev(np.array([s_x], np.float32))
        y16 = B.linear(x8_d, sx_d, packed, scales, n, g, B.LAYOUT_TILED, out_dtype=torch.bfloat16)
        h16 = B.silu_mul(y16)
        for src, call, args in ((y16, B.linear_fp8_out, (packed, scales, n)), (h16, B.linear_silu_mul_fp8_out, (paired, paired_s, n // 2))):
            finite = src.float()[torch.isfinite(src.float())]
            amax = float(finite.abs().max()) if finite.numel() else 1.0
            for y_scale in (amax / 600.0, amax / 1e6, 1.0, 0.0):  # some saturate, most do, whatever comes, a division by zero
                ys_d = dev(np.array([max(y_scale, 1e-44) if y_scale else 0.0], np.float32))
                want = B.quantize_act(src, ys_d)
                got = call(x8_d, sx_d, *args, g, ys_d)
                assert same_e4m3(got, want), (call.__name__, s_x, y_scale)
                seen |= {int((want & 0x7F).min()), int((want & 0x7F).max())}
    assert {0x00, 0x7E, 0x7F} <= seen


@pytest.mark.parametrize("tile,m", [(4, 130), (1, 200)])
def test_every_bf16_gate_through_the_fused_epilogue(gpu_lib, tile, m):
    """All 65536 bf16 values as gates (one channel each, by its group scale and the sign of its code) under several up values and output scales: the bytes
    of linear, silu_mul (the general division) and quantize_act."""
    f, k = 65536, 128
    assert B.linear_launch_shape(m, k, 2 * f, 128)[:2] == (2, tile)
    values = torch.arange(f, dtype=torch.int32, device=DEV)
    gates = (values << 16).view(torch.float32)
    x8_d = torch.zeros((m, k), dtype=torch.uint8, device=DEV)
    x8_d[:, 0] = 0x38                                            # 1.0
    one = dev(np.array([1.0], np.float32))
    for shift in range(3):
        ups = torch.tensor([1.0, 1.171875, 0.0078125, 3.140625, 201.0, 1.0e-3, 1.3046875], device=DEV)[(values + shift * 2) % 7]
        codes = torch.zeros((2 * f, k), dtype=torch.int8, device=DEV)
        codes[:f, 0] = 1 - 2 * (values >> 15).to(torch.int8)
        codes[f:, 0] = 1
        s = torch.cat([gates.abs(), ups])[:, None].contiguous()
        packed, scales = B.pack_weights(codes, 128, B.LAYOUT_TILED, s)
        paired, paired_s = B.pack_weights(B.interleave_gate_up(codes), 128, B.LAYOUT_TILED, B.interleave_gate_up(s))
        gu = B.linear(x8_d, one, packed, scales, 2 * f, 128, B.LAYOUT_TILED, out_dtype=torch.bfloat16)
        got_gates = gu[0, :f].float()
        nan = torch.isnan(gates)
        assert torch.equal(torch.isnan(got_gates), nan) and torch.equal(got_gates[~nan], gates[~nan])
        h = B.silu_mul(gu)
        for y_scale in (1.0, 0.01, 100.0, 1e-4, 1e30):
            ys_d = dev(np.array([y_scale], np.float32))
            got = B.linear_silu_mul_fp8_out(x8_d, one, paired, paired_s, f, 128, ys_d)
            assert same_e4m3(got, B.quantize_act(h, ys_d)), (shift, y_scale)
