"""Dequantize where its wavefronts end: row counts around the eight (fp16) and four (fp32) rows of a
wavefront and the pairs that share a store, a strided output, malformed high-plane bits -- against a
dense numpy reconstruction from the storage layout (fp64)."""
import numpy as np
import pytest

from tests.packed_inputs import random_packed, unpack_numpy

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [1, 3, 7, 8, 9, 15, 16, 23, 41])
@pytest.mark.parametrize("K", [256, 1280])
def test_dequantize_row_edges(N, K):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2603_27914_amd import binding

    codes, scales = random_packed(N, K, "dqe", z_fraction=0.3)
    if N > 1:
        codes = codes.copy()
        codes[256 + 3] |= 0x00010004  # high-plane bits of row 1 (storage lane 1, second word): codes 4..6 there
    H = np.array([[(-1.0) ** bin(i & j).count("1") for j in range(256)] for i in range(256)])
    c, d, z = unpack_numpy(codes, scales, N, K)
    q = c.reshape(N, -1, 256) - 1.0 - z[:, :, None]
    want = (d[:, :, None] * (q @ H) / 16.0).reshape(N, K)
    cd, sd = (torch.from_numpy(a.view(np.int32)).cuda() for a in (codes, scales))
    for dtype, ulp in ((torch.float32, 2.0**-24), (torch.float16, 2.0**-11 + 2.0**-24)):
        buf = torch.full((N, K + 8), 7.0, dtype=dtype, device="cuda")
        flags = torch.zeros(1, dtype=torch.int32, device="cuda")
        binding.itq3s_dequantize(cd, sd, N, K, out=buf[:, :K], status_flags=flags)
        got = buf.double().cpu().numpy()
        assert np.all(got[:, K:] == 7.0)
        # integers up to fp32's 24 bits, one rounding of the product, one to fp16 (2^-25 below its normal range)
        assert np.all(np.abs(got[:, :K] - want) <= ulp * np.abs(want) + (2.0**-25 if dtype == torch.float16 else 0.0))
        assert int(flags.item()) == (binding.FLAG_BAD_CODE if N > 1 else 0)


@pytest.mark.parametrize("sub", [False, True])
def test_dequantize_rows_between_two_16_byte_boundaries(sub):
    """A row stride that is a multiple of four elements but not of eight: in fp16 every other row starts eight
    bytes behind a 16-byte boundary.  Against the contiguous output, and the padding columns stay."""
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2603_27914_amd import binding

    N, K = 41, 1280
    codes, scales = random_packed(N, K, "dqa", z_fraction=0.3)
    cd, sd = (torch.from_numpy(a.view(np.int32)).cuda() for a in (codes, scales))
    s = np.random.default_rng(5).uniform(0.25, 2.0, size=(codes.size // 384 * 64, 2)).astype(np.float16)
    ud = torch.from_numpy(s.view(np.int32).reshape(-1)).cuda()
    L = binding.lib()
    for dtype, code in ((torch.float32, binding.F32), (torch.float16, binding.F16)):
        want = binding.itq3s_dequantize_sub(cd, sd, ud, N, K, dtype=dtype) if sub else binding.itq3s_dequantize(cd, sd, N, K, dtype=dtype)
        buf = torch.full((N, K + 4), 7.0, dtype=dtype, device="cuda")
        if sub:
            rc = L.itq3s_dequantize_sub(cd.data_ptr(), sd.data_ptr(), ud.data_ptr(), N, K, buf.data_ptr(), code, K + 4, None, binding._stream())
            assert rc == 0
        else:
            binding.itq3s_dequantize(cd, sd, N, K, out=buf[:, :K])
        assert torch.equal(buf[:, :K], want) and bool((buf[:, K:] == 7.0).all())


@pytest.mark.parametrize("N", [16377, 16384, 16385, 16391, 16393, 16400])
@pytest.mark.parametrize("sub", [False, True])
def test_fp16_rows_per_wavefront_on_both_sides_of_the_line(N, sub):
    """Up to 1024 tiles four rows per wavefront, beyond eight: either way each value is the fp32 output's (one
    rounding of the same product) rounded to fp16."""
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2603_27914_amd import binding

    K = 256
    cd, sd = (torch.from_numpy(a.view(np.int32)).cuda() for a in random_packed(N, K, "dql", z_fraction=0.3))
    gen = torch.Generator(device="cuda").manual_seed(N)
    ud = (0.25 + 1.75 * torch.rand((cd.numel() // 384 * 64, 2), generator=gen, device="cuda")).half().view(torch.int32).reshape(-1)
    if sub:
        full, half = (binding.itq3s_dequantize_sub(cd, sd, ud, N, K, dtype=t) for t in (torch.float32, torch.float16))
    else:
        full, half = (binding.itq3s_dequantize(cd, sd, N, K, dtype=t) for t in (torch.float32, torch.float16))
    assert torch.equal(full.half(), half)
