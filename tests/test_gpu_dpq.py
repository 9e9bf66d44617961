"""GPU parity of the offline calibration: the Group-Aware Reordering permutation (Sec. 3.2, App. A.3) and Dual
Precision Quantization (Alg. 1) -- codes, group scales and zero-points bit-exact against the oracle, which takes the
same float32 steps -- and the calibrated weights through packing and the literal inference layer."""
import numpy as np
import pytest
import torch

from oracle import w4a8_oracle as o
from paper_2505_14638_amd import binding as B
from paper_2505_14638_amd import synthetic as syn

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def host(t):
    torch.cuda.synchronize()
    return t.cpu().numpy()


def calibration_inputs(rng, t, k):
    """Synthetic calibration activations: unequal feature magnitudes, mild correlations, a few outlier channels."""
    base = rng.standard_normal((t, k))
    mix = np.eye(k) + 0.3 * rng.standard_normal((k, k)) / np.sqrt(k)
    x = (base @ mix) * np.exp(rng.uniform(-1.0, 1.0, size=k))[None, :]
    x[:, rng.choice(k, size=max(1, k // 100), replace=False)] *= 20.0
    return x


@pytest.mark.parametrize("k,g", [(1024, 128), (512, 256), (384, 384)])
def test_gar_permutation_bit_exact(gpu_lib, k, g):
    rng = np.random.default_rng([81, k, g])
    d = rng.random(k).astype(np.float32)
    d[rng.choice(k, size=k // 8, replace=False)] = d[0]           # ties, inside groups and between group maxima
    if k > g:
        d[g:2 * g] = np.minimum(d[g:2 * g], d[:g].max())
        d[g + 3] = d[:g].max()
    got = host(B.gar_permutation(dev(d), g))
    assert np.array_equal(got, o.gar_permutation(d, g))


@pytest.mark.parametrize("n,k,g,per_channel,reorder", [(40, 256, 128, True, False), (150, 512, 256, True, True),
                                                       (70, 384, 128, False, True), (129, 640, 128, True, True)])
def test_dpq_bit_exact(gpu_lib, n, k, g, per_channel, reorder):
    rng = np.random.default_rng([82, n, k, g])
    w = syn.make_weights(rng, n, k)
    x = calibration_inputs(rng, 2 * k, k)
    perm = o.gar_permutation(np.diag(x.T @ x), g) if reorder else None
    u = o.hessian_inverse_factor(x[:, perm] if reorder else x).astype(np.float32)
    s_w = (np.abs(w).max(axis=1) / np.float32(448.0)).astype(np.float32) if per_channel else \
        np.array([np.abs(w).max() / np.float32(448.0)], dtype=np.float32)
    want = o.dpq_quantize(w, u, s_w, g, perm=perm)
    got = B.dpq_calibrate(dev(w), dev(u), dev(s_w), g, dev(perm.astype(np.int32)) if reorder else None)
    codes, scales, zeros = (host(t) for t in got)
    assert np.array_equal(scales, want[1]) and np.array_equal(zeros, want[2])
    assert np.array_equal(codes, want[0])
    # compensation took place: the codes differ from the uncompensated double quantization
    plain = o.dpq_quantize(w, np.eye(k, dtype=np.float32), s_w, g)
    assert np.mean(codes != plain[0]) > 0.05


@pytest.mark.parametrize("n,k,g,grid,shrink,reorder", [(40, 256, 128, 20, 0.8, False), (70, 512, 256, 37, 0.5, True),
                                                        (33, 384, 128, 5, 0.9, True), (17, 256, 128, 2, 0.3, False)])
def test_dpq_with_the_mse_scale_search_bit_exact(gpu_lib, n, k, g, grid, shrink, reorder):
    """Alg. 1 with the scale search of Sec. 3.3: candidates split over the lanes of a row on the GPU, scanned one after
    the other in the oracle -- the same float32 scores, the same first minimum, the same codes and parameters."""
    rng = np.random.default_rng([87, n, k, g])
    w = syn.make_weights(rng, n, k)
    w[np.arange(n), rng.integers(0, k, n)] *= 5.0                          # a stretched range in one group per row
    x = calibration_inputs(rng, 2 * k, k)
    perm = o.gar_permutation(np.diag(x.T @ x), g) if reorder else None
    u = o.hessian_inverse_factor(x[:, perm] if reorder else x).astype(np.float32)
    s_w = (np.abs(w).max(axis=1) / np.float32(448.0)).astype(np.float32)
    want = o.dpq_quantize(w, u, s_w, g, perm=perm, mse_grid=grid, mse_max_shrink=shrink)
    got = B.dpq_calibrate(dev(w), dev(u), dev(s_w), g, dev(perm.astype(np.int32)) if reorder else None, mse_grid=grid,
                          mse_max_shrink=shrink)
    codes, scales, zeros = (host(t) for t in got)
    assert np.array_equal(scales, want[1]) and np.array_equal(zeros, want[2])
    assert np.array_equal(codes, want[0])
    plain = o.dpq_quantize(w, u, s_w, g, perm=perm)
    assert np.mean(scales != plain[1]) > 0.1                               # the search did move scales


def test_calibrated_weights_through_packing_and_inference(gpu_lib):
    """Calibration -> w4a8_pack_weights_asym -> w4a8_linear_asym_two_level: the layer on calibrated weights is closer
    to the unquantized layer, on the calibration inputs, than the layer on uncompensated weights; and the inference
    output matches the oracle's literal layer on the same codes."""
    rng = np.random.default_rng(83)
    n, k, g, t = 96, 512, 128, 1024
    w = syn.make_weights(rng, n, k)
    x = calibration_inputs(rng, t, k)
    s_x = syn.static_act_scale(x.astype(np.float32))
    x8 = o.quantize_act(x.astype(np.float32), s_x)
    xq = o.e4m3_decode(x8) * float(s_x)                                   # the activations inference sees
    s_w = (np.abs(w).max(axis=1) / np.float32(448.0)).astype(np.float32)
    h_diag = np.diag(xq.T @ xq).astype(np.float32)
    perm = host(B.gar_permutation(dev(h_diag), g))
    u = o.hessian_inverse_factor(xq[:, perm]).astype(np.float32)
    full = xq @ w.astype(np.float64).T
    errs = {}
    for name, (uf, pm) in {"plain": (np.eye(k, dtype=np.float32), None), "dpq_gar": (u, perm)}.items():
        codes, scales, zeros = B.dpq_calibrate(dev(w), dev(uf), dev(s_w), g, dev(pm) if pm is not None else None)
        packed, params = B.pack_weights_asym(codes, g, scales, zeros)
        y = host(B.linear_asym_two_level(dev(x8), dev(np.array([s_x], np.float32)), packed, params, dev(s_w), n, g,
                                         out_dtype=torch.float32))
        ref, w8 = o.linear_ref_asym_paper_literal(x8, s_x, host(codes), host(zeros), host(scales), s_w, g)
        a = float(s_x) * (np.abs(o.e4m3_decode(x8)) @ np.abs(o.e4m3_decode(w8)).T) * s_w.astype(np.float64)[None, :]
        ok, worst = o.within_tolerance(y, ref, a, floor=2.0 ** -4)
        assert ok, (name, worst)
        errs[name] = float(np.linalg.norm(y - full) ** 2)
    print(f"  layer error on the calibration inputs: uncompensated {errs['plain']:.4e}, DPQ + GAR {errs['dpq_gar']:.4e}", flush=True)
    assert errs["dpq_gar"] < 0.9 * errs["plain"]


@pytest.mark.parametrize("n,k,g,grid", [(1, 128, 128, 0), (63, 256, 128, 0), (65, 384, 128, 3), (130, 256, 256, 0), (130, 256, 256, 20),
                                        (65, 384, 128, 20), (3, 256, 256, 300), (9, 384, 384, 100), (70, 512, 256, 2),
                                        (2079, 256, 128, 13), (2080, 256, 128, 13)])
def test_dpq_general_division_and_tile_edges(gpu_lib, n, k, g, grid):
    """Rows around the 64 of a tile, and in some rows what the short division does not take -- zero weights, weights and
    scales near the ends of float32's range, a diagonal entry of U beyond 2^30 -- beside rows it does: bit exact.  The search
    in a launch of its own (wide groups; more than 12 candidates and fewer than 160 rows for each) and beside the walk."""
    rng = np.random.default_rng([93, n, k])
    w = syn.make_weights(rng, n, k)
    w[::5, ::7] = 0.0
    w[2::9] *= np.float32(1e-25)
    w[3::11] *= np.float32(1e25)
    x = calibration_inputs(rng, 2 * k, k)
    u = o.hessian_inverse_factor(x).astype(np.float32)
    if n > 64:
        u[k - 70, k - 70] = np.float32(2.0 ** 31)
    s_w = (np.abs(w).max(axis=1) / np.float32(448.0)).astype(np.float32)
    want = o.dpq_quantize(w, u, s_w, g, mse_grid=grid)
    codes, scales, zeros = (host(t) for t in B.dpq_calibrate(dev(w), dev(u), dev(s_w), g, None, mse_grid=grid))
    assert np.array_equal(scales, want[1]) and np.array_equal(zeros, want[2]) and np.array_equal(codes, want[0])


@pytest.mark.parametrize("n,k,g", [(40, 256, 128), (130, 512, 256)])
def test_dpq_products_below_the_normal_range(gpu_lib, n, k, g):
    """Rows so small that an error times U is a subnormal number: the matrix unit has to round it, not to flush it."""
    rng = np.random.default_rng([96, n, k, g])
    w = syn.make_weights(rng, n, k)
    w[::2] *= np.float32(1e-33)
    w[1::2] *= np.float32(1e-34)
    u = o.hessian_inverse_factor(calibration_inputs(rng, 2 * k, k)).astype(np.float32)
    s_w = (np.abs(w).max(axis=1) / np.float32(448.0)).astype(np.float32)
    off = np.abs(u[np.triu_indices(k, 1)])
    assert s_w.min() > 2.0 ** -126 * 0.5 and np.mean(s_w.max() * off.astype(np.float64) < 2.0 ** -126) > 0.5
    want = o.dpq_quantize(w, u, s_w, g)
    codes, scales, zeros = (host(t) for t in B.dpq_calibrate(dev(w), dev(u), dev(s_w), g))
    assert np.array_equal(codes, want[0]) and np.array_equal(scales, want[1]) and np.array_equal(zeros, want[2])
    # the updates count: without them the codes are others
    assert np.mean(codes != o.dpq_quantize(w, np.eye(k, dtype=np.float32), s_w, g)[0]) > 0.02


def test_scale_search_launches_with_columns_beside_the_walk(gpu_lib):
    """2100 rows x 2560 features, 20 candidates, in reordered columns: the launch before a search brings 15 blocks of columns up
    to date, the others go with the walk.  Rows are independent: some of them against the oracle, bit for bit."""
    rng = np.random.default_rng(97)
    n, k, g = 2100, 2560, 128
    w = syn.make_weights(rng, n, k)
    u = (np.triu(rng.standard_normal((k, k)) * 0.02, 1) + np.diag(rng.uniform(0.5, 1.5, size=k))).astype(np.float32)
    s_w = (np.abs(w).max(axis=1) / np.float32(448.0)).astype(np.float32)
    perm = o.gar_permutation(rng.random(k).astype(np.float32), g)
    got = B.dpq_calibrate(dev(w), dev(u), dev(s_w), g, dev(perm.astype(np.int32)), mse_grid=20, mse_max_shrink=0.7)
    rows = np.array([0, 63, 64, 1000, 2099])
    want = o.dpq_quantize(w[rows], u, s_w[rows], g, perm=perm, mse_grid=20, mse_max_shrink=0.7)
    for a, b in zip(got, want):
        assert np.array_equal(host(a)[rows], b)


def median_ms(call):
    times = []
    for _ in range(9):
        start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        start.record()
        call()
        end.record()
        end.synchronize()
        times.append(start.elapsed_time(end))
    return sorted(times)[4]


@pytest.mark.parametrize("g", [128, 1024])
def test_scale_search_takes_less_time_than_the_walk(gpu_lib, g):
    """100 candidates on 256 rows: 1.2 times the calibration without a search at either group size, 4 and 11 times with four
    lanes scoring a row's candidates; with 32 lanes it was 2.1."""
    n, k = 256, 1024
    gen = torch.Generator(device=DEV).manual_seed(95)
    w = torch.randn((n, k), generator=gen, device=DEV)
    u = torch.triu(torch.randn((k, k), generator=gen, device=DEV) * 0.02, 1) + torch.eye(k, device=DEV)
    s_w = w.abs().amax(dim=1) / 448.0

    without, searched = (median_ms(lambda: B.dpq_calibrate(w, u, s_w, g, None, mse_grid=grid)) for grid in (0, 100))
    print(f"  groups of {g}: {without:.3f} ms without, {searched:.3f} ms with 100 candidates", flush=True)
    assert searched < 2.0 * without


@pytest.mark.parametrize("k,g", [(128, 128), (2176, 128), (133120, 128)])
def test_gar_permutation_ties_signs_and_many_groups(gpu_lib, k, g):
    """One group, and more groups than the kernel holds maxima of at a time; ties, zeros of both signs, negative values."""
    rng = np.random.default_rng([94, k])
    d = np.round(rng.standard_normal(k) * 4).astype(np.float32)
    d[::3] *= np.float32(-0.0)
    assert np.array_equal(host(B.gar_permutation(dev(d), g)), o.gar_permutation(d, g))


@pytest.mark.parametrize("t,k,dtype", [(1, 64, "f32"), (100, 200, "f32"), (1000, 384, "bf16"), (4096, 1024, "f32")])
def test_hessian_accumulate(gpu_lib, t, k, dtype):
    """H = X^T X over two batches (float32 accumulation on the GPU) against the float64 product of the same values:
    each entry within 2e-5 of sqrt(H_ii H_jj) (about a hundred float32 roundings of terms no larger than that)."""
    rng = np.random.default_rng([84, t, k])
    x = calibration_inputs(rng, 2 * t, k).astype(np.float32)
    if dtype == "bf16":
        x = o.bf16_bits_to_f32(syn.f32_to_bf16_bits(x))
        xd = torch.from_numpy(x).to(DEV).to(torch.bfloat16)
    else:
        xd = torch.from_numpy(x).to(DEV)
    wide = torch.full((t, k + 7), 1e6, dtype=xd.dtype, device=DEV)
    wide[:, :k] = xd[t:]
    h = B.hessian_accumulate(xd[:t])
    h = B.hessian_accumulate(wide[:, :k], h)                              # second batch with a row stride
    got = host(h).astype(np.float64)
    want = x.astype(np.float64).T @ x.astype(np.float64)
    d = np.sqrt(np.diag(want))
    assert np.all(np.abs(got - want) <= 2e-5 * np.outer(d, d) + 1e-30)
    assert np.array_equal(got, got.T)                                     # the same products in the same order


@pytest.mark.parametrize("t,k,dtype", [(45, 3466, "bf16"), (33, 3461, "bf16"), (64, 130, "bf16"), (7, 33, "bf16"), (17, 70, "f32"),
                                       (50, 257, "f32"), (4096, 256, "bf16"), (512, 3458, "bf16"), (545, 3458, "bf16")])
def test_hessian_accumulate_tile_edges(gpu_lib, t, k, dtype):
    """Remainders of the tiles (64 and, on bf16 layers of 3457 features and more, 128 wide from 33 tokens on, with even strides
    from 513) and of the token slices (16 / 32), even and odd row strides, against float64.  An entry is a sum of t products,
    each at most sqrt(H_ii H_jj) in sum of magnitudes: every rounding, and every product the bf16 matrix unit cuts off 24
    bits below the largest of its octet, costs at most 2^-24 of that, one per token and one for the batch that is added."""
    rng = np.random.default_rng([91, t, k])
    x = calibration_inputs(rng, 2 * t, k) if k < 1000 else rng.standard_normal((2 * t, k))
    xd = torch.from_numpy(x.astype(np.float32)).to(DEV)
    if dtype == "bf16":
        xd = xd.to(torch.bfloat16)
    x = host(xd.float()).astype(np.float64)
    wide = torch.full((t, k + 7), 1e6, dtype=xd.dtype, device=DEV)
    wide[:, :k] = xd[t:]
    got = host(B.hessian_accumulate(wide[:, :k], B.hessian_accumulate(xd[:t]))).astype(np.float64)
    want = x.T @ x
    d = np.sqrt(np.diag(want))
    assert np.all(np.abs(got - want) <= (2 * t + 1) * 2.0 ** -24 * np.outer(d, d) + 1e-30)
    assert np.array_equal(got, got.T)


@pytest.mark.parametrize("t", [544, 545, 575])
def test_hessian_accumulate_whole_slices_and_a_tail(gpu_lib, t):
    """128 x 128 tiles with features past the end in the last ones, whole slices of 32 tokens and none, one or 31 left over; inputs, strides and
    tolerance of test_hessian_accumulate_tile_edges."""
    test_hessian_accumulate_tile_edges(gpu_lib, t, 3466, "bf16")


@pytest.mark.parametrize("t,k", [(50, 70), (3, 128)])
def test_hessian_accumulate_float32_is_a_chain_of_fmas(gpu_lib, t, k):
    """float32 activations: every entry is the bits of one FMA per token, in their order.  Integers below 2^15: a product and
    its sum with an accumulator below 2^37 are exact in float64, so rounding that once to float32 is the FMA."""
    rng = np.random.default_rng([96, t, k])
    x = rng.integers(-(1 << 15) + 1, 1 << 15, size=(t, k)).astype(np.float32)
    want = np.zeros((k, k), np.float32)
    for row in x.astype(np.float64):
        want = (want.astype(np.float64) + np.outer(row, row)).astype(np.float32)
    assert np.array_equal(host(B.hessian_accumulate(dev(x))), want)


def test_hessian_accumulate_of_few_tokens_takes_no_longer_in_bf16(gpu_lib):
    """Reading and writing H is most of the time: 39 us for either type on 5120 features; on 128 x 128 tiles bf16 took 69."""
    k = 5120
    h = torch.zeros((k, k), device=DEV)
    f32, bf16 = (median_ms(lambda: B.hessian_accumulate(x, h)) for x in (torch.zeros((16, k), device=DEV, dtype=d) for d in (torch.float32, torch.bfloat16)))
    print(f"  16 tokens: float32 {f32 * 1e3:.1f} us, bf16 {bf16 * 1e3:.1f} us", flush=True)
    assert bf16 < 1.4 * f32


@pytest.mark.parametrize("k,reorder,damp", [(128, False, 0.01), (512, True, 0.01), (1024, True, 0.05), (1152, False, 0.01)])
def test_hessian_inverse_factor(gpu_lib, k, reorder, damp):
    """Dampening + Cholesky (Sec. 3.3) on the GPU (float64 inside) against the oracle's float64 route through the
    explicit inverse, from the same float32 Hessian: float32 rounding of the result plus a conditioning allowance."""
    rng = np.random.default_rng([85, k])
    x = calibration_inputs(rng, 2 * k, k)
    h = (x.T @ x).astype(np.float32)
    h = np.maximum(h, h.T)                                                # symmetric after the rounding to float32
    perm = o.gar_permutation(np.diag(h), 128) if reorder else None
    want = o.hessian_inverse_factor_from_h(h, damp, perm)
    u, info = B.hessian_inverse_factor(dev(h), damp, dev(perm.astype(np.int32)) if reorder else None)
    got = host(u).astype(np.float64)
    assert int(host(info)[0]) == 0
    assert np.all(np.tril(got, -1) == 0.0) and np.all(np.diag(got) > 0)
    assert np.all(np.abs(got - want) <= 2.0 ** -23 * np.abs(want) + 1e-9 * np.abs(want).max())
    hd = (h if perm is None else h[perm][:, perm]).astype(np.float64)
    hd = hd + np.eye(k) * damp * np.trace(hd) / k
    assert np.abs(got.T @ got @ hd - np.eye(k)).max() < 1e-3            # float32 entries of U: ~cond * 2^-24


@pytest.mark.parametrize("k", [256, 384, 640, 896])
def test_hessian_inverse_factor_few_pairs_of_tile_columns(gpu_lib, k):
    """4, 6, 10 and 14 tiles: the inverse, one pair of tile columns behind the factorization, starts and ends.  Tolerance as in
    test_hessian_inverse_factor: float32 rounding of the result plus a conditioning allowance."""
    rng = np.random.default_rng([92, k])
    x = calibration_inputs(rng, 2 * k, k)
    h = (x.T @ x).astype(np.float32)
    h = np.maximum(h, h.T)
    want = o.hessian_inverse_factor_from_h(h, 0.01, None)
    u, info = B.hessian_inverse_factor(dev(h), 0.01)
    got = host(u).astype(np.float64)
    assert int(host(info)[0]) == 0 and np.all(np.tril(got, -1) == 0.0)
    assert np.all(np.abs(got - want) <= 2.0 ** -23 * np.abs(want) + 1e-9 * np.abs(want).max())


def test_hessian_inverse_factor_reports_a_matrix_that_is_not_positive_definite(gpu_lib):
    k = 256
    h = np.eye(k, dtype=np.float32)
    h[100, 100] = -1.0
    _, info = B.hessian_inverse_factor(dev(h), 0.0)
    assert int(host(info)[0]) == k - 100                                  # 1 + index counted from the end: 155 + 1


def test_calibration_pipeline_on_the_gpu(gpu_lib):
    """Activations -> Hessian -> reordering -> factor -> Alg. 1, every step on the GPU, against the oracle run on the
    GPU's float32 Hessian: the permutation is identical; the factor agrees to float32 rounding, so all but a few codes
    (a decision next to a tie can flip, and its compensation moves a few later ones) are identical and the layer error
    is the same."""
    rng = np.random.default_rng(86)
    n, k, g, t = 64, 512, 128, 2048
    w = syn.make_weights(rng, n, k)
    x = calibration_inputs(rng, t, k).astype(np.float32)
    s_w = (np.abs(w).max(axis=1) / np.float32(448.0)).astype(np.float32)
    h_d = B.hessian_accumulate(dev(x))
    perm_d = B.gar_permutation(torch.diagonal(h_d).contiguous(), g)
    u_d, info = B.hessian_inverse_factor(h_d, 0.01, perm_d)
    codes, scales, zeros = (host(a) for a in B.dpq_calibrate(dev(w), u_d, dev(s_w), g, perm_d))
    assert int(host(info)[0]) == 0
    h = host(h_d)
    perm = o.gar_permutation(np.diag(h), g)
    assert np.array_equal(host(perm_d), perm)
    u = o.hessian_inverse_factor_from_h(h, 0.01, perm).astype(np.float32)
    want = o.dpq_quantize(w, u, s_w, g, perm=perm)
    same = float(np.mean(codes == want[0]))
    print(f"  codes identical to the oracle's: {same:.5f}", flush=True)
    assert same > 0.995 and np.mean(zeros == want[2]) > 0.99

    def layer_error(c, s, z):
        _, w8 = o.linear_ref_asym_paper_literal(np.zeros((1, k), np.uint8), 1.0, c, z, s, np.ones(n), g)
        return float(np.linalg.norm((w.astype(np.float64) - o.e4m3_decode(w8) * s_w.astype(np.float64)[:, None]) @ x.T.astype(np.float64)) ** 2)
    e_gpu, e_ref = layer_error(codes, scales, zeros), layer_error(*want)
    plain = o.dpq_quantize(w, np.eye(k, dtype=np.float32), s_w, g)
    e_plain = layer_error(*plain)
    print(f"  layer error: GPU pipeline {e_gpu:.4e}, oracle {e_ref:.4e}, uncompensated {e_plain:.4e}", flush=True)
    assert abs(e_gpu - e_ref) < 0.02 * e_ref and e_gpu < 0.9 * e_plain


def test_calibration_at_the_size_bench_times_sampled_rows(gpu_lib):
    """A 4096 x 4096 layer with 8192 calibration tokens, the shapes of bench.py's calibration leg.  The factor from the
    GPU against the oracle's at full size; then Alg. 1 with GAR and the scale search on all 4096 rows on the GPU against
    the oracle on 12 sampled rows (rows are independent), bit for bit, both on the oracle's factor."""
    rng = np.random.default_rng(88)
    n = k = 4096
    g, t = 128, 8192
    print("  inputs", flush=True)
    w = syn.make_weights(rng, n, k)
    x = syn.make_activations(rng, t, k, 0.01, 20.0) * np.exp(rng.uniform(-1.0, 1.0, size=k)).astype(np.float32)[None, :]
    s_w = (np.abs(w).max(axis=1) / np.float32(448.0)).astype(np.float32)
    h_d = B.hessian_accumulate(dev(x.astype(np.float32)))
    perm_d = B.gar_permutation(torch.diagonal(h_d).contiguous(), g)
    u_d, info = B.hessian_inverse_factor(h_d, 0.01, perm_d)
    h, perm = host(h_d), host(perm_d)
    assert int(host(info)[0]) == 0 and np.array_equal(perm, o.gar_permutation(np.diag(h), g))
    print("  oracle factor", flush=True)
    u = o.hessian_inverse_factor_from_h(h, 0.01, perm)
    got_u = host(u_d).astype(np.float64)
    assert np.all(np.abs(got_u - u) <= 2.0 ** -23 * np.abs(u) + 1e-9 * np.abs(u).max())
    u32 = u.astype(np.float32)
    print("  Alg. 1 on the GPU", flush=True)
    codes, scales, zeros = (host(a) for a in B.dpq_calibrate(dev(w), dev(u32), dev(s_w), g, perm_d, mse_grid=8, mse_max_shrink=0.6))
    rows = np.sort(np.concatenate([[0, n - 1], rng.choice(n - 2, 10, replace=False) + 1]))
    print("  Alg. 1 in the oracle, 12 rows", flush=True)
    want = o.dpq_quantize(w[rows], u32, s_w[rows], g, perm=perm, mse_grid=8, mse_max_shrink=0.6)
    assert np.array_equal(scales[rows], want[1]) and np.array_equal(zeros[rows], want[2])
    assert np.array_equal(codes[rows], want[0])


@pytest.mark.parametrize("at", [0, 15, 16, 31, 47, 48, 63, 64, 79, 112, 127, 191])
def test_hessian_inverse_factor_reports_the_first_bad_pivot_of_every_block(gpu_lib, at):
    """A pivot that is not positive in each 16 x 16 diagonal block of a tile and at their edges, with couplings to the columns before it and a
    second one behind: `at` counts in the factorization's order, from the last column."""
    k = 256
    rng = np.random.default_rng([93, at])
    x = calibration_inputs(rng, 2 * k, k)
    h = (x.T @ x).astype(np.float32)
    h = np.maximum(h, h.T)
    h[k - 1 - at, k - 1 - at] = -1.0
    h[k - 1 - min(at + 40, k - 1), k - 1 - min(at + 40, k - 1)] = -1.0
    _, info = B.hessian_inverse_factor(dev(h), 0.0)
    assert int(host(info)[0]) == at + 1


@pytest.mark.parametrize("scale", [1e-30, 1e30])
def test_hessian_inverse_factor_scales(gpu_lib, scale):
    """U scales with 1 / sqrt of the Hessian at the ends of float32.  Tolerance as in test_hessian_inverse_factor."""
    k = 256
    x = calibration_inputs(np.random.default_rng(94), 2 * k, k)
    h = (x.T @ x)
    h = (h / np.abs(h).max() * scale).astype(np.float32)
    h = np.maximum(h, h.T)
    want = o.hessian_inverse_factor_from_h(h.astype(np.float64) / scale, 0.01, None) / np.sqrt(scale)
    u, info = B.hessian_inverse_factor(dev(h), 0.01)
    assert int(host(info)[0]) == 0
    assert np.all(np.abs(host(u).astype(np.float64) - want) <= 2.0 ** -22 * np.abs(want) + 1e-9 * np.abs(want).max())


def test_hessian_inverse_factor_special_cases(gpu_lib):
    """A diagonal Hessian without dampening has the closed form U = diag(1 / sqrt(h_ii)); the identity permutation is
    the same as none; a reversal of the columns gives the factor of the reversed matrix."""
    rng = np.random.default_rng(89)
    k = 256
    d = rng.uniform(0.5, 4.0, k).astype(np.float32)
    u, info = B.hessian_inverse_factor(dev(np.diag(d)), 0.0)
    assert int(host(info)[0]) == 0
    assert np.allclose(host(u), np.diag(1.0 / np.sqrt(d.astype(np.float64))), rtol=2e-7, atol=0)
    x = calibration_inputs(rng, 2 * k, k)
    h = (x.T @ x).astype(np.float32)
    h = np.maximum(h, h.T)
    u0 = host(B.hessian_inverse_factor(dev(h), 0.01)[0])
    u1 = host(B.hessian_inverse_factor(dev(h), 0.01, dev(np.arange(k, dtype=np.int32)))[0])
    assert np.array_equal(u0, u1)
    rev = np.arange(k - 1, -1, -1, dtype=np.int32)
    u2 = host(B.hessian_inverse_factor(dev(h), 0.01, dev(rev))[0])
    u3 = host(B.hessian_inverse_factor(dev(np.ascontiguousarray(h[::-1, ::-1])), 0.01)[0])
    assert np.array_equal(u2, u3)


@pytest.mark.parametrize("n", [9000, 17000])
def test_dpq_many_rows_sampled(gpu_lib, n):
    """Layers with more than 8192 / 16384 rows run the block kernel with 16 / 8 lanes per row (and, beyond 16384, with U
    read from global memory): the same bits as the oracle on sampled rows, scale search included."""
    rng = np.random.default_rng([90, n])
    k, g = 256, 128
    w = syn.make_weights(rng, n, k)
    x = calibration_inputs(rng, 2 * k, k)
    perm = o.gar_permutation(np.diag(x.T @ x), g)
    u = o.hessian_inverse_factor(x[:, perm]).astype(np.float32)
    s_w = (np.abs(w).max(axis=1) / np.float32(448.0)).astype(np.float32)
    got = B.dpq_calibrate(dev(w), dev(u), dev(s_w), g, dev(perm.astype(np.int32)), mse_grid=6, mse_max_shrink=0.5)
    codes, scales, zeros = (host(t) for t in got)
    rows = np.sort(np.concatenate([[0, n - 1], rng.choice(n - 2, 30, replace=False) + 1]))
    want = o.dpq_quantize(w[rows], u, s_w[rows], g, perm=perm, mse_grid=6, mse_max_shrink=0.5)
    assert np.array_equal(scales[rows], want[1]) and np.array_equal(zeros[rows], want[2])
    assert np.array_equal(codes[rows], want[0])
