"""The layer kernel's own 64 x 64 products on a tile, element by element against FP64: in FP32, with the weights
in BF16 and with the weights in two BF16 parts."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("shift", [0.0, 30.0])
def test_tile_products(shift):
    from paper_2606_19251_amd import capi

    rng = np.random.default_rng(7)
    A = (rng.standard_normal((64, 64)) + shift).astype(np.float32)
    B = rng.standard_normal((64, 64)).astype(np.float32)
    d = [torch.full((64, 64), float("nan"), device="cuda") for _ in range(3)]
    Ad, Bd = torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda()
    st = torch.cuda.current_stream().cuda_stream
    capi.gcin_tile_gemm_check(Ad.data_ptr(), Bd.data_ptr(), d[0].data_ptr(), d[1].data_ptr(), st)
    capi.gcin_tile_gemm_check_x3(Ad.data_ptr(), Bd.data_ptr(), d[2].data_ptr(), st)
    f32, bf16, x3 = (t.cpu().numpy().astype(np.float64) for t in d)
    A64, B64 = A.astype(np.float64), B.astype(np.float64)
    Bh = torch.from_numpy(B).to(torch.bfloat16).to(torch.float64).numpy()
    size = np.abs(A64) @ np.abs(B64)  # bounds of the rounding errors, per element
    # 64 products summed in FP32
    assert (np.abs(f32 - A64 @ B64) <= 64 * 2.0 ** -24 * size).all()
    # a number in two BF16 parts is off by at most 2^-17 of itself (8 bits each, rounded to nearest); with both
    # operands in parts the product of the two lo parts (2^-9 2^-9) is left out as well
    assert (np.abs(bf16 - A64 @ Bh) <= (2.0 ** -17 + 128 * 2.0 ** -24) * (np.abs(A64) @ np.abs(Bh))).all()
    assert (np.abs(x3 - A64 @ B64) <= (2 * 2.0 ** -17 + 2.0 ** -18 + 192 * 2.0 ** -24) * size).all()
    # and no element is another's: the products differ by far more than the bounds
    assert np.abs(A64 @ Bh - A64 @ B64).max() > 2.0 ** -12 * size.max() / 64
