"""The streaming kernel for 17 and more activation rows at the sizes where its division of the work
changes (padding of rows and row tiles, wavefronts without a block, several rounds of items, tensors
that share an item), and sizes just beyond it.  Every size says which kernel takes it, and that is asserted.  Checked on the
device against itq3s_dequantize (held to the oracle within 1e-6 elsewhere) and a dense fp64 product."""
import numpy as np
import pytest

from tests.block_scaled import ROWS, SHARES4, SHARES8, TILED, route, route_items_columns
from tests.packed_inputs import random_packed

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2603_27914_amd import binding

    binding.lib()
    return torch, binding


def tensor(torch, binding, N, K, *key, z_fraction=0.02):
    c, s = (torch.from_numpy(a.view(np.int32)).cuda() for a in random_packed(N, K, *key, z_fraction=z_fraction))
    return c, s, binding.itq3s_dequantize(c, s, N, K).double()


def check(Y, X, What, half):
    """Per row: 2e-3 relative L2, the bar of every matmul test.  Per element: one rounding to fp16 of the
    rotated activations (2^-11 relative each) against exact products, so at most 2^-11 ||x|| ||w_hat|| by
    Cauchy-Schwarz, half as much again for the fp32 sums, and the rounding of the result."""
    want = X.double() @ What.T
    err = (Y.double() - want).abs()
    bound = 1.5 * 2.0**-11 * X.double().norm(dim=1)[:, None] * What.norm(dim=1)[None, :] + 2.0 ** (-11 if half else -22) * want.abs() + 1e-30
    assert (err / bound).max().item() <= 1.0
    assert ((Y.double() - want).norm(dim=1) / want.norm(dim=1).clamp_min(1e-300)).max().item() <= 2e-3


SIZES = [
    # the many-row kernel
    (17, 16, 256),      # one row tile, one block: seven of eight wavefronts have nothing
    (33, 1000, 2304),   # nine blocks: one wavefront has two; a ragged last row tile
    (48, 257, 4096),
    (49, 4100, 512),    # 64 rows, 15 of them padding
    (64, 9000, 768),    # 563 row tiles: three per workgroup, the last item one short
    (65, 300, 2048),    # two groups of 48 rows
    (97, 13000, 512),   # two rounds of items of four row tiles
    (130, 1032, 1280),  # three groups
    (160, 4096, 1024),
    (257, 333, 11008),
    (1024, 2048, 512),
    (64, 16, 28928),    # the longest K at 64 rows
    (20, 16, 79872),    # ... and at 20
    # beyond
    (97, 17000, 256, TILED),
    (64, 40, 165376, SHARES8),  # many blocks a wavefront
    (20, 24, 250112, SHARES8),
    (64, 40, 196608, SHARES8),
    (20, 24, 262400, None),     # two passes of the kernel for up to 16 rows
]


@pytest.mark.parametrize("size", SIZES)
def test_many_rows(gpu, size):
    M, N, K, kernel = size if len(size) == 4 else (*size, ROWS)
    assert kernel is None or route(M, N, K) == kernel
    if (M, N, K) == (97, 13000, 512):
        assert route_items_columns(M, N, K)[1] > 256 and route_items_columns(M, N, K)[2] == 64
    torch, binding = gpu
    codes, scales, What = tensor(torch, binding, N, K, "rows", M)
    gen = torch.Generator(device="cuda").manual_seed(M + N)
    buf = torch.randn((M, K + 8), generator=gen, device="cuda").half()
    X = buf[:, :K]
    for dtype in (torch.float32, torch.float16):
        out = torch.full((M, N + 3), 7.0, dtype=dtype, device="cuda")
        flags = torch.zeros(1, dtype=torch.int32, device="cuda")
        binding.itq3s_matmul(codes, scales, N, K, X, out=out[:, :N], status_flags=flags)
        assert int(flags.item()) == 0 and bool((out[:, N:] == 7.0).all())
        check(out[:, :N], X, What, dtype == torch.float16)


@pytest.mark.parametrize("M", [24, 40, 64, 100])
def test_many_rows_grouped_equals_single_calls(gpu, M):
    """Items that span tensors (16 + 1000 + 17 + 300 rows, and 256-tile tensors with three tiles per item),
    and a group in which one tensor is large enough for a block-scaled kernel."""
    torch, binding = gpu
    groups = [(512, [16, 1000, 17, 300]), (1024, [4096, 4096, 4096])]
    if M == 100:
        groups.append((8192, [24576, 500]))
    for K, Ns in groups:
        assert [route(M, N, K) for N in Ns] == [SHARES8 if N == 24576 else ROWS for N in Ns]
        ts = [tensor(torch, binding, N, K, "rowsg", i) for i, N in enumerate(Ns)]
        X = torch.randn((M, K), generator=torch.Generator(device="cuda").manual_seed(M), device="cuda").half()
        outs = binding.itq3s_matmul_grouped([(c, s, N) for (c, s, _), N in zip(ts, Ns)], K, X, dtype=torch.float16)
        for (c, s, What), N, out in zip(ts, Ns, outs):
            assert torch.equal(out, binding.itq3s_matmul(c, s, N, K, X, dtype=torch.float16))
            check(out, X, What, True)


def test_many_rows_flags(gpu):
    torch, binding = gpu
    M, N, K = 50, 100, 1024
    codes, scales, _ = tensor(torch, binding, N, K, "rowsf")
    X = torch.randn((M, K), generator=torch.Generator(device="cuda").manual_seed(3), device="cuda").half()
    flags = torch.zeros(1, dtype=torch.int32, device="cuda")
    bad = codes.clone()
    bad[384 * 9 + 256 + 5] = 1  # a high-plane bit
    binding.itq3s_matmul(bad, scales, N, K, X, status_flags=flags)
    assert int(flags.item()) == binding.FLAG_BAD_CODE
    flags.zero_()
    X[49, 256:512] = 5000.0  # rotates to a spike of 16 x 5000 > 65504
    binding.itq3s_matmul(codes, scales, N, K, X, status_flags=flags)
    assert int(flags.item()) == binding.FLAG_ACT_RANGE


# one to four row tiles to an item of 16 rows; wavefronts without a block; the last group with one row
@pytest.mark.parametrize("M,N,K", [(17, 200, 512), (33, 100, 2304), (17, 4300, 16384), (33, 4300, 16384), (81, 520, 11008), (96, 1300, 8192), (96, 33, 20480)])
def test_groups_of_sixteen_rows(gpu, M, N, K):
    """A thin tensor alone goes in groups of 16 rows, beside a wide one in larger ones: the same bits."""
    torch, binding = gpu
    codes, scales, What = tensor(torch, binding, N, K, "sixteen", M)
    wide = tensor(torch, binding, 4096, K, "sixteen-wide", M)
    X = torch.randn((M, K), generator=torch.Generator(device="cuda").manual_seed(M), device="cuda").half()
    Y = binding.itq3s_matmul(codes, scales, N, K, X)
    check(Y, X, What, False)
    a, b = binding.itq3s_matmul_grouped([(codes, scales, N), (*wide[:2], 4096)], K, X, dtype=torch.float32)
    assert torch.equal(a, Y)
    check(b, X, wide[2], False)


@pytest.mark.parametrize("M,N,K,less", [(17, 1000, 4096, "pass"), (32, 100, 11008, "pass"), (64, 33000, 256, "slabs")])
def test_room_for_the_other_routes_is_still_enough(gpu, M, N, K, less):
    """A call whose workspace has room for the passes of 16 rows or for the activation rows as they are (sized for
    another M, or when the tiled kernel had fp16 operands) is computed in passes, or in slabs of rows: alone, in a
    group, twice on one workspace of garbage.  One byte less is refused."""
    torch, binding = gpu
    codes, scales, What = tensor(torch, binding, N, K, "room", M)
    X = torch.randn((M, K), generator=torch.Generator(device="cuda").manual_seed(M), device="cuda").half()
    if less == "pass":
        room = binding.itq3s_matmul_workspace_bytes(16, N, K)
        want = torch.cat([binding.itq3s_matmul(codes, scales, N, K, X[m : m + 16]) for m in range(0, M, 16)])
    else:  # (129 tiles of 128 x 256: the activation rows and 768 bytes)
        room = (M * K * 2 + 255) // 256 * 256 + 768
        want = None
    assert room < binding.itq3s_matmul_workspace_bytes(M, N, K)
    ws = torch.randint(0, 255, (room,), dtype=torch.uint8, device="cuda")
    first = binding.itq3s_matmul(codes, scales, N, K, X, workspace=ws).clone()
    check(first, X, What, False)
    assert want is None or torch.equal(first, want)
    assert torch.equal(first, binding.itq3s_matmul(codes, scales, N, K, X, workspace=ws))
    for out in binding.itq3s_matmul_grouped([(codes, scales, N), (codes, scales, N)], K, X, dtype=torch.float32, workspace=ws):
        assert torch.equal(first, out)
    with pytest.raises(binding.Itq3sError, match="workspace"):
        binding.itq3s_matmul(codes, scales, N, K, X, workspace=ws[: room - 1])


# rotated activations of more than 32 MB, or a product too large for the streaming kernel
@pytest.mark.parametrize("M,N,K,z,kernel", [(8200, 100, 2048, 0.02, SHARES8), (2100, 300, 8192, 0.6, SHARES8), (517, 9300, 4096, 0.02, SHARES8), (517, 3000, 4096, 0.3, SHARES4),
                                            (4200, 700, 4096, 0.0, TILED), (4201, 700, 4096, 0.6, TILED), (66000, 17, 256, 0.02, TILED)])
def test_larger_calls_ragged(gpu, M, N, K, z, kernel):
    torch, binding = gpu
    assert route(M, N, K) == kernel
    codes, scales, What = tensor(torch, binding, N, K, "tiled", M, z_fraction=z)
    X = torch.randn((M, K), generator=torch.Generator(device="cuda").manual_seed(M), device="cuda").half()
    for dtype in (torch.float32, torch.float16):
        check(binding.itq3s_matmul(codes, scales, N, K, X, dtype=dtype), X, What, dtype == torch.float16)
