"""The wave-tile builds that default launches choose among (rg_linear for M > 8, FP32 weights at
M > 4, and any K or alignment the 16-byte kernels do not take) against the oracle, bit for bit.

Every shape below makes the rule choose another build (tests/test_abi.py holds that all are reached): the tiles from 8 x 16 to 64 x 64, with
ragged last tiles in M and N, a short last segment and slab, one and several rounds of
segments, K below one slab, odd K (rows of x and W at every alignment), the bias and pointers off
their 16-byte alignment.  No tolerance: the order fixes every bit.
"""
import numpy as np
import pytest

from tests import gpu_util as gu

pytestmark = pytest.mark.gpu

# one shape per build, from 64 x 64 down to 16 x 16, then K below a slab, long K and many short rows
ALIGNED = [(57, 28818, 776), (49, 12370, 1288), (49, 22599, 776), (49, 8452, 1288), (49, 14341, 1288), (41, 30135, 776),
           (33, 11110, 1288), (33, 27477, 776), (49, 13426, 776), (49, 10663, 776), (25, 4445, 2056), (17, 24777, 776),
           (17, 9299, 1288), (17, 4149, 2056), (9, 24770, 776), (17, 6361, 776), (17, 2055, 2056), (9, 32, 264),
           (10, 70, 8), (333, 1000, 24), (65, 130, 4360), (129, 20954, 264), (17, 2057, 1288)]
ALIGNED_F32 = [(33, 14762, 1288), (33, 10921, 1288), (33, 7053, 1288), (17, 10506, 1288), (17, 6148, 1288), (5, 6361, 2056),
               (5, 4639, 1288), (5, 33, 264), (9, 33, 260), (17, 21688, 268), (65, 130, 4364)]
ANY = [(33, 5753, 1289), (17, 6160, 1289), (17, 6351, 775), (9, 2055, 1289), (1, 4231, 2061), (1, 31, 263), (1, 31, 1),
       (3, 1000, 1001), (9, 20555, 3), (100, 16491, 31), (47, 300, 4099), (8, 77, 513)]


def _inputs(M, N, K, f32, seed):
    rng = np.random.default_rng(seed)
    x = rng.standard_normal((M, K), dtype=np.float32)
    w = (0.02 * rng.standard_normal((N, K), dtype=np.float32)).astype(np.float32)
    return x, w if f32 else (w.view(np.uint32) >> 16).astype(np.uint16)


def _check(M, N, K, f32=False, bias=False, shift=0):
    import torch
    import oracle
    import paper_2609_25624_amd as rg
    rg.rg_linear_set_launch(None)
    gu.log(f"wave-tile rule M={M} N={N} K={K} f32={f32} bias={bias} shift={shift}")
    x, w = _inputs(M, N, K, f32, M + N + K)
    # `shift` elements between the allocation's start and the first row
    xb = torch.zeros(M * K + shift, dtype=torch.float32, device=gu.dev())
    wb = torch.zeros(N * K + shift, dtype=torch.float32 if f32 else torch.int16, device=gu.dev())
    xd, wd = xb[shift:].view(M, K), wb[shift:].view(N, K)
    xd.copy_(torch.from_numpy(x))
    wd.copy_(torch.from_numpy(w if f32 else w.view(np.int16)))
    if bias:
        b = np.random.default_rng(1).standard_normal(N, dtype=np.float32)
        bd = torch.from_numpy(b).to(gu.dev())
        want = oracle.linear_bias(x, w, b)
    elif f32:
        want = oracle.linear_f32w(x, w)
    else:
        want = oracle.linear_fast(x, w)
    for order in (0, 1):                 # the tiles' workgroups forward and reversed
        rg.rg_linear_set_launch(grid_order=order)
        y = torch.full((M, N), 7.0, dtype=torch.float32, device=gu.dev())
        if bias:
            rg.rg_linear_bias(xd, wd, bd, y)
        elif f32:
            rg.rg_linear_f32w(xd, wd, y)
        else:
            rg.rg_linear(xd, wd, y)
        torch.cuda.synchronize()
        gu.assert_bitwise(y.cpu().numpy(), want, f"({M},{N},{K}) order {order}")
    rg.rg_linear_set_launch(None)


@pytest.mark.parametrize("M,N,K", ALIGNED)
def test_bf16_builds(M, N, K):
    _check(M, N, K)


@pytest.mark.parametrize("M,N,K", ALIGNED_F32)
def test_f32_builds(M, N, K):
    _check(M, N, K, f32=True)


@pytest.mark.parametrize("f32", [False, True])
@pytest.mark.parametrize("M,N,K", ANY)
def test_odd_k_builds(M, N, K, f32):
    _check(M, N, K, f32=f32)


@pytest.mark.parametrize("M,N,K,f32,kernel", [
    (9, 300, 28672, False, "skinny"), (16, 1024, 1024, False, "skinny"), (64, 250, 7056, False, "skinny"),
    (33, 40, 2056, False, "skinny"), (13, 64, 32168, False, "skinny"),
    (1906, 4288, 360, False, "tiled"), (2000, 4096, 1032, False, "tiled"), (249, 27072, 304, False, "tiled"),
    (142, 28835, 320, True, "tiled"), (2000, 4096, 1036, True, "tiled"), (487, 11335, 388, True, "tiled"),
    (51, 2310, 1, False, "generic"), (1, 3001, 21, False, "generic"), (7, 555, 7, True, "generic"),
    (3, 901, 11, False, "generic"), (2, 501, 23, True, "generic"), (206, 390, 1, False, "generic")])
def test_defaults_that_other_kernels_lead(M, N, K, f32, kernel):
    import paper_2609_25624_amd as rg
    rg.rg_linear_set_launch(None)
    assert (rg.rg_plan_f32w if f32 else rg.rg_plan)(M, N, K)["kernel_name"] == kernel
    _check(M, N, K, f32=f32)


@pytest.mark.parametrize("M,N,K,shift", [(5, 100, 1003, 0), (12, 300, 512, 1), (70, 500, 264, 3), (2, 40, 256, 1)])
def test_bias_and_shifted_pointers(M, N, K, shift):
    _check(M, N, K, bias=True, shift=shift)


@pytest.mark.parametrize("M,N,K", [(64, 4096, 4096), (16, 6144, 4096), (40, 1030, 4104), (5, 2999, 1003), (333, 1000, 2056)])
def test_cu_masks(M, N, K):
    """The default's tiles on streams that own only some of the compute units."""
    import torch
    import oracle
    import paper_2609_25624_amd as rg
    rg.rg_linear_set_launch(None)
    gu.log(f"wave-tile rule cu masks {rg.rg_plan(M, N, K)}")
    x, w = _inputs(M, N, K, False, 3)
    xd, wd = gu.to_dev(x, w)
    want = oracle.linear_fast(x, w)
    nwords = (rg.rg_device_cu_count() + 31) // 32
    done = 0
    for mask in ([0x55555555] * nwords, [0xFFFFFFFF] * (nwords // 2) + [0] * (nwords - nwords // 2),
                 [0xFFFFFFFF, 0x1F] + [0] * (nwords - 2)):
        try:
            s = rg.rg_stream_create_cu_mask(mask)
        except rg.RgError:
            continue                                  # the runtime may refuse a mask
        try:
            ext = torch.cuda.ExternalStream(s)
            y = torch.full((M, N), 7.0, dtype=torch.float32, device=gu.dev())
            torch.cuda.synchronize()
            gu.run(xd, wd, stream=ext, out=y)
            ext.synchronize()
            gu.assert_bitwise(y.cpu().numpy(), want, f"({M},{N},{K}) mask {mask[0]:x}")
            done += 1
        finally:
            torch.cuda.synchronize()
            rg.rg_stream_destroy(s)
    assert done >= 1, "no CU mask could be exercised"


@pytest.mark.parametrize("K", [255, 270, 264])
def test_negative_zero_sums_survive_the_padding(K):
    # products that underflow to -0 from the first k on: every chain and every fold stays -0 only if the
    # staged k past K multiply as fmaf(+0, -0, -0) = -0
    import torch
    import oracle
    import paper_2609_25624_amd as rg
    M, N = 11, 50
    x = np.full((M, K), 1e-30, dtype=np.float32)
    w = np.full((N, K), 0xa000, dtype=np.uint16)     # about -1.1e-19: the product rounds to -0
    want = oracle.linear_fast(x, w)
    y = gu.run(*gu.to_dev(x, w))
    torch.cuda.synchronize()
    gu.assert_bitwise(y.cpu().numpy(), want, f"-0 sums K={K}")
