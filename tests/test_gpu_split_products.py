"""fp32 products of the large tiles (96 x 128 elements and more), which are taken as six bf16 products of the
operands' parts.  Each product is looked at by itself (one nonzero value in a row of A), against float64: no
one is off by more than three units of 2^-24, and they are off to either side alike; values the parts
cannot hold (infinities, the ends of the fp32 range) are multiplied in fp32."""
import ctypes as C

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

F32, STORE = 0, 1
TILES = [(96, 128), (128, 128), (176, 128), (128, 192)]
U = 2.0**-24
BOUND = 3.07


def matmul(tile, a, w):
    """A W^T through one tile shape of the tiled GEMM."""
    import torch
    from paper_2502_09922_amd import binding

    fn = binding.lib.ls_test_tiled_gemm
    fn.argtypes = [C.c_uint32] + [C.c_int] * 4 + [C.c_void_p] * 2 + [C.c_int] * 3 + [C.c_void_p] * 2
    a, w = torch.from_numpy(a).cuda(), torch.from_numpy(w).cuda()
    out = torch.full((a.shape[0], w.shape[0]), float("nan"), device="cuda")
    assert fn(F32, STORE, *tile, 1, a.data_ptr(), w.data_ptr(), a.shape[0], w.shape[0], a.shape[1], out.data_ptr(), None)
    torch.cuda.synchronize()
    return out.cpu().numpy()


def one_per_row(values, k):
    a = np.zeros((len(values), k), np.float32)
    a[np.arange(len(values)), np.arange(len(values)) % k] = values
    return a


def error_of_products(tile, values, w):
    """Error of values[m] * w[n][m % K], in units of 2^-24 of the product."""
    got = matmul(tile, one_per_row(values, w.shape[1]), w).astype(np.float64)
    want = values.astype(np.float64)[:, None] * w.astype(np.float64)[:, np.arange(len(values)) % w.shape[1]].T
    return (got - want) / (np.abs(want) * U)


@pytest.mark.parametrize("tile", TILES)
def test_every_product_keeps_its_bits_and_has_no_bias(tile):
    # what is left out is at most 1 unit (2 x 2^-25); the last addition loses at most 2 (the bf16 matrix
    # instruction drops what an accumulator smaller than the product holds below the result's last bit,
    # towards minus infinity: a whole last bit in the worst case); the additions of the smaller partial
    # sums, 2^-7 of the product, 4 x 2 x 2^-7 together
    rng = np.random.default_rng(1)
    a = rng.standard_normal(2 * tile[0]).astype(np.float32)
    w = rng.standard_normal((tile[1], 64)).astype(np.float32)
    err = error_of_products(tile, a, w)
    print("random mantissas: largest %.2f, mean %+.4f of 2^-24" % (np.abs(err).max(), err.mean()))
    assert np.abs(err).max() <= BOUND
    # away from zero and towards it alike: errors of a standard deviation below 1 unit, so the mean of n of them
    # stays within 5 / sqrt(n)
    signed = err * np.sign(a)[:, None] * np.sign(w)[:, np.arange(len(a)) % 64].T
    assert abs(signed.mean()) <= 5 / np.sqrt(err.size), signed.mean()
    # one sign and one mantissa throughout: 1 + 2^-7 - 2^-23, all bits of the second and third part set
    worst = np.full(tile[0] + 1, np.uint32(0x3F80FFFF)).view(np.float32)
    err = error_of_products(tile, worst, np.full((tile[1], 64), worst[0]))
    print("0x3F80FFFF squared: %.2f of 2^-24" % err.max())
    assert np.abs(err).max() <= BOUND


@pytest.mark.parametrize("tile", TILES)
def test_the_ends_of_the_range_and_infinities(tile):
    rng = np.random.default_rng(2)
    m, n, k = tile[0] + 1, 144, 96
    pairs = ((2.0**-102, 2.0**90), (2.0**-60, 2.0**-40), (2.0**126, 2.0**-30), (2.0**70, 2.0**50), (2.0**-51, 1.0))
    for sa, sw in pairs:
        a = (sa * rng.uniform(1, 2, m)).astype(np.float32)
        w = (sw * rng.uniform(1, 2, (n, k))).astype(np.float32)
        err = error_of_products(tile, a, w)
        assert np.abs(err).max() <= BOUND, (sa, sw, np.abs(err).max())
    # the largest fp32 value, which rounds to an infinity in 8 bits
    top = np.full(m, np.finfo(np.float32).max)
    got = matmul(tile, one_per_row(top, k), np.full((n, k), 0.5, np.float32))
    assert (got == np.float32(top[0] * np.float32(0.5))).all()
    # an infinity in one weight, and one in one row: everything else stays what it is
    a = rng.standard_normal((m, k)).astype(np.float32)
    w = rng.standard_normal((n, k)).astype(np.float32)
    want = a.astype(np.float64) @ w.astype(np.float64).T
    bound = 2 * k * U * (np.abs(a).astype(np.float64) @ np.abs(w).astype(np.float64).T)
    w[7, 33] = np.inf
    a[m - 1, 64] = -np.inf
    got = matmul(tile, a, w)
    rows, cols = np.arange(m) != m - 1, np.arange(n) != 7
    assert (np.abs(got - want)[np.ix_(rows, cols)] <= bound[np.ix_(rows, cols)]).all()
    assert (got[rows, 7] == np.where(a[rows, 33] > 0, np.inf, -np.inf)).all()
    assert (got[m - 1, cols] == np.where(w[cols, 64] > 0, -np.inf, np.inf)).all()


@pytest.mark.parametrize("tile", TILES)
def test_sums_of_one_sign_do_not_drift(tile):
    # n = 6 K / 32 additions; each rounds the sum so far, on average half the result, to 24 bits: errors of
    # 2^-24 / sqrt(3) of it, as likely up as down, add up to sqrt(n / 3) * 2^-24 / sqrt(3) of the result
    rng = np.random.default_rng(4)
    k = 8192
    a = np.abs(rng.standard_normal((tile[0], k))).astype(np.float32)
    w = np.abs(rng.standard_normal((tile[1], k))).astype(np.float32)
    want = a.astype(np.float64) @ w.astype(np.float64).T
    err = np.linalg.norm(matmul(tile, a, w) - want) / np.linalg.norm(want)
    expect = np.sqrt(6 * k / 32) / 3 * U
    print("%.2e, %.1f of what independent roundings give" % (err, err / expect))
    assert err <= 4 * expect


@pytest.mark.parametrize("rows,tiles", [(161, ((176, 128), (96, 128))), (257, ((176, 128), (96, 128))), (500, ((128, 128), (128, 128)))])
def test_prompts_on_the_large_tiles_against_the_oracle(rows, tiles):
    """A layer as wide as the 7B shape's, K of the down projection with half a k-step at its end (688) and cut: what the plan
    takes for the O and the down projection."""
    import synth
    from helpers import check_close, check_delta, make_gpu, make_oracle, to_dev, to_host
    from oracle.stage_oracle import decode_values
    from paper_2502_09922_amd import binding

    fn = binding.lib.ls_test_tiled_plan
    fn.argtypes = [C.c_uint32] + [C.c_int] * 5 + [C.c_size_t, C.POINTER(C.c_int * 3)]
    for k, tile in zip((4096, 688), tiles):  # O and down projection
        plan = (C.c_int * 3)()
        assert fn(F32, 0, rows, 4096, k, 1, 8 * rows * 4096 * 4, C.byref(plan))
        assert tuple(plan[:2]) == tile and plan[2] > 1, list(plan)
    shape = synth.StageShape("f32", 1, 4096, 32, 4, 128, 688, 0)
    lengths = [rows - rows // 3, rows // 3]
    gpu = make_gpu(shape, 3, 0, 1, 2, max(lengths), rows)
    ora = make_oracle(shape, 3, 0, 1, 2, max(lengths))
    x = synth.hidden_states(shape, 4, rows)
    got, want = to_host(gpu.prefill(to_dev(shape, x), lengths)), ora.prefill(x, lengths)
    check_close(got, want, "f32", "prompt")
    check_delta(got, want, decode_values(x), "f32", "prompt")
    gpu.close()
