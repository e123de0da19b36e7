"""GPU tests of the 17 to 144 row kernel and of the two dequantization routes
(needs an MI355X): the sizes where a workgroup's rounds, tiles and rows end
unevenly, and the ends of the scale range that each route takes, against the
oracle within max(2 bf16 ulp, 1e-3); integer sums and dequantized weights bit
for bit.
"""

import numpy as np
import pytest
import torch

from oracle import qlin_ref as ref
from paper_2607_04244_amd import qlin
from synth import gen

from test_parity import assert_close, dev, host_bits, make, oracle, run

pytestmark = pytest.mark.gpu

SKINNY, AUTO = qlin.PATH_SKINNY, qlin.PATH_AUTO


@pytest.mark.parametrize("M", [17, 32, 33, 48, 49, 64])
@pytest.mark.parametrize("Kb,N", [(1, 16), (4, 48), (5, 16), (8, 208), (9, 32), (12, 16), (13, 80), (20, 12304),
                                  (3, 20480)])
def test_rounds_tiles_and_rows_end_unevenly(M, Kb, N):
    """Groups below, at and past the 8 of a round (the last up to four shared
    by two waves each), one to the most tiles a workgroup holds, full and
    partial m-tiles; both formats, without a K split."""
    for sym in (False, True):
        c = gen.random_case(M * 1000 + Kb * 10 + N + sym, M, 128 * Kb, N)
        lin = make(c, symmetric=sym)
        assert "kernel=k_mid" in lin.plan(M), lin.plan(M)
        assert_close(run(lin, c["x"], SKINNY), oracle(c, symmetric=sym), f"M={M} Kb={Kb} N={N} sym={sym}")
        lin.close()


@pytest.mark.parametrize("M", [17, 48, 64])
@pytest.mark.parametrize("Kb,N", [(1, 8208), (2, 12304), (4, 19456), (5, 4112), (5, 8192), (5, 20480), (6, 8208),
                                  (6, 16400), (7, 12288), (7, 20480), (8, 8208), (11, 8208), (12, 4112)])
def test_last_groups_shared_by_tile(M, Kb, N):
    """Two and more tiles a workgroup: the waves of a pair take every other tile
    of a shared last group, alone (up to 4 groups) or after whole rounds; of 5 to
    7 groups in one round the last ones by four, two and two waves."""
    c = gen.random_case(M * 1000 + Kb * 10 + N, M, 128 * Kb, N)
    lin = make(c)
    assert_close(run(lin, c["x"], SKINNY), oracle(c), f"M={M} Kb={Kb} N={N}")
    lin.close()


@pytest.mark.parametrize("M,K,Ns", [(17, 128, (32784,)), (48, 256, (24592,)), (49, 384, (20480, 16)),
                                    (64, 512, (11280, 9232))])
def test_very_wide_layers_run_as_tiled_blocks(M, K, Ns):
    """More columns than one round of workgroups holds: the tiled kernel, from a
    handle's own plans and for a group."""
    cs = [gen.random_case(M + K + N, M, K, N) for N in Ns]
    lins = [make(c) for c in cs]
    _, plan = qlin.group_plan(lins, M)
    assert "kernel=k_tiled" in plan or torch.cuda.get_device_properties(0).multi_processor_count != 256, plan
    if len(Ns) == 1:
        assert lins[0].plan(M) == plan
        ys = [run(lins[0], cs[0]["x"])]
    else:
        ys = [host_bits(y) for y in qlin.forward_group(lins, dev(cs[0]["x"]))]
    for y, c in zip(ys, cs):
        assert_close(y, oracle(dict(c, x=cs[0]["x"])), f"M={M} K={K} N={Ns}")
    for lin in lins:
        lin.close()


@pytest.mark.parametrize("M", [65, 80, 81, 96, 97, 112, 113, 128, 129, 144])
@pytest.mark.parametrize("Kb,N", [(3, 48), (4, 16), (5, 208), (9, 224), (13, 4112)])
def test_half_group_units_end_unevenly(M, Kb, N):
    """Above 64 rows: half groups below, at and past the 8 of a round, one and
    two tiles a workgroup, full and partial m-tiles; both formats."""
    for sym in (False, True):
        c = gen.random_case(M * 1000 + Kb * 10 + N + sym, M, 128 * Kb, N)
        lin = make(c, symmetric=sym)
        assert "path=tiled kernel=k_mid" in lin.plan(M), lin.plan(M)
        assert_close(run(lin, c["x"]), oracle(c, symmetric=sym), f"M={M} Kb={Kb} N={N} sym={sym}")
        lin.close()


@pytest.mark.parametrize("M,N", [(65, 8208), (80, 12288), (81, 8208), (96, 12288)])
def test_most_tiles_above_64_rows(M, N):
    K = 128 * 20
    c = gen.random_case(M + N, M, K, N)
    lin = make(c)
    # the tiles a workgroup follow from the compute units
    assert "kernel=k_mid" in lin.plan(M) or torch.cuda.get_device_properties(0).multi_processor_count != 256, lin.plan(M)
    assert_close(run(lin, c["x"]), oracle(c), f"M={M} N={N}")
    lin.close()


@pytest.mark.parametrize("M,split", [(17, 2), (33, 3), (64, 5)])
def test_split_integer_sums_are_bit_exact(M, split):
    K, N = 128 * 21, 176
    rng = np.random.default_rng(M)
    Q = rng.integers(0, 16, size=(N, K), dtype=np.uint8)
    xi = rng.integers(-1, 2, size=(M, K))
    x = np.select([xi == 1, xi == -1], [0x3F80, 0xBF80], 0).astype(np.uint16)
    c = dict(K=K, N=N, packed=ref.pack_codes(Q), scales=np.full((N, K // 128), 0x3F80, np.uint16))
    lin = make(c, symmetric=True)
    y_ref = ref.round_output(ref.forward(x, c["packed"], c["scales"], ref.symmetric_zeros(N, K)))
    for _ in range(2):                     # the arrival counters are left at zero
        assert np.array_equal(run(lin, x, SKINNY, split), y_ref)
    lin.close()


# bf16 scales at the ends of the f16 route's range [2^-25, 2^4) and just past them
F16_LO, F16_HI = (127 - 25) << 7, (127 + 3) << 7 | 127


@pytest.mark.parametrize("lo,hi", [(F16_LO, F16_LO + 127), (F16_LO, F16_HI), (F16_LO - 1, F16_HI), (F16_LO, F16_HI + 1),
                                   (27 << 7, 226 << 7)])
@pytest.mark.parametrize("sym", [False, True])
def test_scale_range_of_both_routes(lo, hi, sym):
    """Dequantized weights bit for bit through both routines, and sums through
    every decode kernel, for scales spread over [lo, hi] (bf16 patterns) with
    both ends present and every zero-point in [0, 15].  x is scaled so that the
    outputs are of the order of one."""
    K, N = 512, 64
    rng = np.random.default_rng(lo + hi)
    scales = rng.integers(lo, hi + 1, size=(N, K // 128)).astype(np.uint16)
    scales[0, 0], scales[N - 1, K // 128 - 1] = lo, hi
    packed = rng.integers(0, 2 ** 32, size=(N, K // 8), dtype=np.uint32)
    zeros = gen.f32_to_bf16_bits(rng.integers(0, 16, size=(N, K // 128)).astype(np.float32))
    z = ref.symmetric_zeros(N, K) if sym else zeros
    lin = qlin.QLinear(packed, scales, None if sym else zeros)
    w = ref.dequant_bf16(packed, scales, z)
    for routine in (0, 1):
        assert np.array_equal(host_bits(lin.dequantize(routine)), w), f"routine {routine}"
    top = float(ref.bf16_to_f64(np.array([hi], np.uint16))[0])
    x = gen.f32_to_bf16_bits((rng.standard_normal((40, K)) / (8.0 * top)).astype(np.float32))
    for path, M in ((qlin.PATH_GEMV, 3), (qlin.PATH_REGS, 16), (SKINNY, 16), (SKINNY, 40), (qlin.PATH_TILED, 40)):
        assert_close(run(lin, x[:M], path), ref.forward(x[:M], packed, scales, z), f"path={path} M={M}")
    lin.close()


@pytest.mark.parametrize("M", [1, 16, 40, 130])
def test_group_of_both_routes(M):
    """One launch over members whose scales take different routes."""
    K = 640
    cases = [gen.random_case(700 + i, M, K, N, s_range=r) for i, (N, r) in
             enumerate(((48, (0.002, 0.02)), (272, (20.0, 40.0)), (16, (0.002, 0.02))))]
    lins = [make(c) for c in cases]
    x = cases[0]["x"]
    need, _ = qlin.group_plan(lins, M)
    ys = qlin.forward_group(lins, dev(x), workspace=qlin.new_workspace(need) if need else None)
    torch.cuda.synchronize()
    for c, y in zip(cases, ys):
        assert_close(host_bits(y), oracle(dict(c, x=x)), f"M={M} N={c['N']}")
    for l in lins:
        l.close()


PATHS = [(qlin.PATH_GEMV, 3), (qlin.PATH_REGS, 16), (SKINNY, 16), (SKINNY, 40), (qlin.PATH_TILED, 40), (AUTO, 130)]


@pytest.mark.parametrize("power", [-100, -110])
@pytest.mark.parametrize("path,M", PATHS)
def test_small_activations_on_the_f16_route(path, M, power):
    """Activations of 2^power: the f16 route's sums are 2^12 smaller than the
    outputs until their rounding.  Bound: half a bf16 unit of the output, K
    binary32 roundings of the products' sum, and K products and sums at the
    scaled subnormals' step 2^(-149 + 12)."""
    c = gen.random_case(60 - power, M, 1024, 208)
    x64 = np.random.default_rng(power & 0xFF).standard_normal((M, c["K"])) * 2.0 ** power
    x = gen.f32_to_bf16_bits(x64.astype(np.float32))
    lin = make(c)
    y = ref.bf16_to_f64(run(lin, x, path))
    w = ref.bf16_to_f64(ref.dequant_bf16(c["packed"], c["scales"], c["zeros"]))
    exact, size = ref.bf16_to_f64(x) @ w.T, np.abs(ref.bf16_to_f64(x)) @ np.abs(w).T
    bound = 2.0 ** -8 * np.abs(exact) + c["K"] * (2.0 ** -24 * size + 2.0 ** -137) + 2.0 ** -134
    assert np.all(np.abs(y - exact) <= bound), np.max(np.abs(y - exact) / bound)
    assert np.median(bound / np.abs(exact)) < 2.0 ** -7            # the bound says something
    lin.close()


@pytest.mark.parametrize("sym", [False, True])
def test_vector_kernel_has_one_range_on_both_routes(sym):
    """The GEMV kernel's sums are those of the weights themselves on either
    route: a handle of each, with the same weights in its first columns, gives
    the same bits for activations that put sums among binary32's smallest."""
    K, N = 512, 48
    rng = np.random.default_rng(5)
    packed = rng.integers(0, 2 ** 32, size=(N + 16, K // 8), dtype=np.uint32)
    scales = rng.integers(F16_LO, F16_LO + 256, size=(N + 16, K // 128)).astype(np.uint16)
    scales[N:] = F16_HI + 1                                        # not on the f16 route
    zeros = gen.f32_to_bf16_bits(rng.integers(0, 16, size=scales.shape).astype(np.float32))
    f16 = qlin.QLinear(packed[:N], scales[:N], None if sym else zeros[:N])
    bf16 = qlin.QLinear(packed, scales, None if sym else zeros)
    for power in (0, -90, -104, -108, -112):
        x = gen.f32_to_bf16_bits((rng.standard_normal((4, K)) * 2.0 ** power).astype(np.float32))
        a, b = run(f16, x, qlin.PATH_GEMV), run(bf16, x, qlin.PATH_GEMV)[:, :N]
        assert np.array_equal(a, b), f"2^{power}: {np.count_nonzero(a != b)} differ"
    f16.close()
    bf16.close()


@pytest.mark.parametrize("path,M", PATHS + [(AUTO, 64), (AUTO, 80)])
def test_infinities_and_nans_stay_in_their_rows(path, M):
    """An infinity and a NaN in two rows of x: those rows' outputs are infinite
    or NaN where the exact sums are, the others keep their bits."""
    c = gen.random_case(31, M, 640, 272)
    lin = make(c)
    clean = run(lin, c["x"], path)
    x = c["x"].copy()
    rows = [0, M - 1]
    x[0, 130], x[M - 1, 5] = 0x7F80, 0x7FC0
    y = run(lin, x, path)
    assert np.array_equal(np.delete(y, rows, axis=0), np.delete(clean, rows, axis=0))
    w = ref.bf16_to_f64(ref.dequant_bf16(c["packed"], c["scales"], c["zeros"]))
    got = ref.bf16_to_f64(y)
    assert np.all(np.isnan(got[M - 1]))
    zero = w[:, 130] == 0
    assert np.all(np.isnan(got[0, zero])) and np.array_equal(got[0, ~zero], np.sign(w[~zero, 130]) * np.inf)
    lin.close()
