"""The block-scaled kernels (fp4 codes, activations in three fp6 parts) at the sizes where their division of the work
changes: rows of every remainder modulo the tiles of 32 and 64, ragged columns, wavefronts without a block, several rounds,
each number of columns an item has, tensors of one launch.  Against itq3s_dequantize and a dense fp64 product."""
import pytest

from tests.block_scaled import ROWS, SHARES4, SHARES8, TILED, route, route_items_columns
from tests.test_gpu_rows import gpu, tensor  # noqa: F401  (gpu is a fixture)

# M, N, K, the kernel that takes it, the columns of an item and the rounds of one to a unit (K over wavefronts)
SIZES = [
    (481, 33, 3584, SHARES8, 32, 1),      # 14 blocks: two wavefronts have one, the others two
    (1301, 100, 1280, SHARES8, 64, 1),    # five blocks: three wavefronts have none
    (9000, 33, 1280, SHARES8, 64, 2),
    (1338, 822, 1280, SHARES8, 128, 2),
    (700, 1000, 2304, SHARES8, 128, 1),   # nine blocks
    (500, 1000, 4096, SHARES8, 64, 1),
    (20, 28672, 4096, SHARES8, 128, 1),   # rows: 12 of padding
    (2113, 300, 8192, SHARES8, 128, 1),
    (1233, 796, 28672, SHARES8, 64, 2),
    (512, 4096, 4096, SHARES4, 256, 1),
    (2081, 515, 1024, SHARES4, 256, 1),   # one block a wavefront, the last columns of an item beyond the tensor
    (993, 1032, 4096, SHARES4, 256, 1),
    (1067, 2300, 5120, SHARES4, 256, 2),
    (197, 33013, 3072, SHARES4, 256, 4),
    (6300, 17, 256, TILED, None, None),   # one block, one storage tile and a ragged one, an odd number of tiles of 32 rows
    (65, 65000, 512, TILED, None, None),  # one row in the second tile of 64
    (640, 4100, 2560, TILED, None, None),
    (33, 40000, 2816, TILED, None, None),
]


def test_sizes_take_the_routes_they_are_here_for():
    for M, N, K, kernel, columns, rounds in SIZES:
        got, items, got_columns = route_items_columns(M, N, K)
        assert got == kernel, (M, N, K)
        if columns is not None:
            assert (got_columns, (items + 255) // 256) == (columns, rounds), (M, N, K)
    # besides: a group's thin tensors go where its wide ones go
    for M, K, Ns, many in ((512, 4096, (512, 1024, 4096), False), (58, 23040, (264, 2112), True), (48, 4096, (512, 4096), True)):
        assert [route(M, N, K) == ROWS for N in Ns] == [many] * len(Ns), (M, K, Ns)


def activations(torch, M, K, seed):
    X = torch.randn((M, K), generator=torch.Generator(device="cuda").manual_seed(seed), device="cuda").half()
    X[:, 5::97] *= 10
    return X


def check(torch, Y, X, What, half):
    """A rotated value is carried to 2^-12 / 3.75 of the largest of its 32 (half the last part's step is 2^-12 of a unit that the
    largest exceeds 3.75 times), so per element at most 1.07 * 2^-14 sqrt(32) ||x|| ||w_hat|| by Cauchy-Schwarz over the
    groups (in fp16, 2^-11 of itself, less), the rest up to 1.5 for the fp32 sums; the intermediate of the rotation in two
    fp16 parts, the lower one no finer than fp16's 2^-24 (2^-25 an element; what follows it is orthonormal, so sqrt(K) of
    them in norm: rows of tiny values); and the rounding of the result.  Rows on the whole: 1e-4 (3.5e-5 measured)."""
    want = X.double() @ What.T
    err = (Y.double() - want).abs()
    x, w = X.double().norm(dim=1)[:, None], What.norm(dim=1)[None, :]
    bound = (1.5 * 2.0**-14 * 32**0.5 * x + 2.0**-25 * X.shape[1] ** 0.5) * w + 2.0 ** (-11 if half else -22) * want.abs()
    assert (err / bound).max().item() <= 1.0
    if not half:
        assert (err.norm() / want.norm()).item() <= 1e-4


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K", [s[:3] for s in SIZES])
def test_block_scaled(gpu, M, N, K):  # noqa: F811
    torch, binding = gpu
    codes, scales, What = tensor(torch, binding, N, K, "mx", M, z_fraction=0.02 if N < 5000 else 0.0)
    buf = activations(torch, M, K + 8, M)
    X = buf[:, :K]
    for dtype in (torch.float32, torch.float16):
        out = torch.full((M, N + 3), 7.0, dtype=dtype, device="cuda")
        flags = torch.zeros(1, dtype=torch.int32, device="cuda")
        ws = torch.full((binding.itq3s_matmul_workspace_bytes(M, N, K),), 0xFF, dtype=torch.uint8, device="cuda")
        binding.itq3s_matmul(codes, scales, N, K, X, out=out[:, :N], workspace=ws, status_flags=flags)
        assert int(flags.item()) == 0 and bool((out[:, N:] == 7.0).all())
        check(torch, out[:, :N], X, What, dtype == torch.float16)


@pytest.mark.gpu
@pytest.mark.parametrize("M,K,Ns", [(901, 1792, (4096, 1000, 40, 17)), (1301, 1280, (300, 9000, 2048))])
def test_group_and_slabs_equal_single_calls(gpu, M, K, Ns):  # noqa: F811
    """Tensors of all three kernels in one call; the same with room for part of the rows only, in several slabs."""
    torch, binding = gpu
    ts = [tensor(torch, binding, N, K, "mxg", i, z_fraction=(0.0, 0.9)[i & 1]) for i, N in enumerate(Ns)]
    X = activations(torch, M, K, 1)
    want = [binding.itq3s_matmul(c, s, N, K, X) for (c, s, _), N in zip(ts, Ns)]
    for (_, _, What), Y in zip(ts, want):
        check(torch, Y, X, What, False)
    full = max(binding.itq3s_matmul_workspace_bytes(M, N, K) for N in Ns)
    least = (M * K * 2 + 255) // 256 * 256 + 768  # the activation rows as they are (K below 2048: no shares of K on top)
    assert least < full
    for room in (full, least):
        ws = torch.full((room,), 0xFF, dtype=torch.uint8, device="cuda")
        outs = binding.itq3s_matmul_grouped([(c, s, N) for (c, s, _), N in zip(ts, Ns)], K, X, dtype=torch.float32, workspace=ws)
        for a, b in zip(outs, want):
            assert torch.equal(a, b), room


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K", [(500, 1000, 4096), (512, 4096, 4096), (640, 4100, 2560)])
def test_range_and_format_flags(gpu, M, N, K):  # noqa: F811
    torch, binding = gpu
    codes, scales, What = tensor(torch, binding, N, K, "mxf")
    flags = torch.zeros(1, dtype=torch.int32, device="cuda")
    bad = codes.clone()
    bad[-384 + 256 + 100] = -1 << 31  # a high-plane bit in the last tile
    X = activations(torch, M, K, 2)
    binding.itq3s_matmul(bad, scales, N, K, X, status_flags=flags)
    assert int(flags.item()) == binding.FLAG_BAD_CODE
    for value in (4100.0, float("inf"), float("nan")):  # rotates to 16 x 4100 > 65504; not finite
        Z = X.clone()
        Z[M - 1, 256:512] = value
        flags.zero_()
        Y = binding.itq3s_matmul(codes, scales, N, K, Z, status_flags=flags)
        assert int(flags.item()) == binding.FLAG_ACT_RANGE
        assert not bool(torch.isfinite(Y[M - 1]).any()) and bool(torch.isfinite(Y[: M - 1]).all())
        check(torch, Y[: M - 1], Z[: M - 1], What, False)


@pytest.mark.gpu
def test_scales_of_the_activations(gpu):  # noqa: F811
    """Rows of every magnitude that fp16 has, constants (one rotated value, all others zero), a single spike, zeros: a row's
    error is bound by its own norm."""
    torch, binding = gpu
    M, N, K = 500, 1000, 4096
    codes, scales, What = tensor(torch, binding, N, K, "mxs")
    X = activations(torch, M, K, 3)
    X[0] = 0
    X[1] = 3.0
    X[2] = 0
    X[2, 777] = 1000.0
    for i in range(3, 27):
        X[i] = (X[i].float() * 2.0 ** (i - 24)).half()
    Y = binding.itq3s_matmul(codes, scales, N, K, X)
    assert bool((Y[0] == 0).all())
    check(torch, Y, X, What, False)


# M <= 4 (straight-line code and not), 5 to 16, the many-row kernel, K over 8 and over 4 wavefronts, tiles
@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K", [(1, 200, 4096), (4, 200, 2816), (16, 200, 1024), (48, 500, 4096), (500, 1000, 4096), (512, 4096, 4096), (640, 4100, 2560)])
def test_code_three_counts_as_two(gpu, M, N, K):  # noqa: F811
    """A low-plane 3 is the digit +2 in every slot of a word, on every path (the header's promise), as in itq3s_dequantize."""
    torch, binding = gpu
    codes, scales, _ = tensor(torch, binding, N, K, "three", M)
    gen = torch.Generator(device="cuda").manual_seed(M)
    words = codes.view(-1, 384)[:, :256]
    shape = tuple(words.shape) + (16,)
    hit = (torch.rand(shape, generator=gen, device="cuda") < 0.03) << (2 * torch.arange(16, device="cuda"))
    hit = hit.sum(dim=-1)
    words |= (hit | hit << 1).to(torch.int32)
    What = binding.itq3s_dequantize(codes, scales, N, K).double()
    X = torch.randn((M, K), generator=gen, device="cuda").half()
    Y = binding.itq3s_matmul(codes, scales, N, K, X).double()
    want = X.double() @ What.T
    assert ((Y - want).norm() / want.norm()).item() <= 4e-4  # (2^-11 / sqrt(3) where x~ is rounded to fp16)

@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K", [(500, 1000, 4096), (512, 4096, 4096), (640, 4100, 2560)])
@pytest.mark.parametrize("half", [False, True])
def test_outputs_beside_a_spike(gpu, M, N, K, half):  # noqa: F811
    """Activations with an offset rotate to a spike at a block's channel 0 (with one of their own for every 64 channels: at 0, 64,
    128, 192).  Outputs whose digits there are 0 are as good as with x~ in fp16: 2^-11 / sqrt(3) in norm, of
    the rounding of x~ and, for fp16 results, of theirs.  Rows with an offset and without in one tile, and apart; a row's
    bits do not depend on the others."""
    torch, binding = gpu
    codes, scales, _ = tensor(torch, binding, N, K, "spike", M, z_fraction=0.0)
    # digit 0 (code 1) at channels 0, 64, 128, 192 of the even columns: word 4 (16 g + r), bits 1:0, r even
    lanes = codes.view(-1, 384)[:, :256].view(-1, 4, 16, 4)
    lanes[:, :, ::2, 0] = (lanes[:, :, ::2, 0] & ~3) | 1
    What = binding.itq3s_dequantize(codes, scales, N, K).double()
    gen = torch.Generator(device="cuda").manual_seed(M)
    noise = torch.randn((M, K), generator=gen, device="cuda")
    sign = torch.randint(0, 2, (M, K // 64), generator=gen, device="cuda").repeat_interleave(64, dim=1) * 2.0 - 1.0
    classes = (0.0, 0.5, 1.5, 4.0, 30.0, 300.0)
    for rows in (torch.arange(M, device="cuda") % 6, torch.arange(M, device="cuda") // 32 % 6):
        offset = torch.tensor(classes, device="cuda")[rows][:, None]
        for X in ((noise + offset).half(), (noise + offset * sign).half()):
            def call(x):
                return binding.itq3s_matmul(codes, scales, N, K, x, dtype=torch.float16 if half else torch.float32).double()

            Y = call(X)
            alone = rows % 2 == 0
            assert torch.equal(call(torch.where(alone[:, None], X, noise.half()))[alone], Y[alone])
            want = X.double() @ What.T
            for i, c in enumerate(classes):
                for cols in (slice(0, N, 2), slice(1, N, 2)):
                    y, w = Y[rows == i][:, cols], want[rows == i][:, cols]
                    err = ((y - w).norm() / w.norm()).item()
                    assert err <= (2.0**0.5 if half else 1.0) * 2.0**-11 / 3**0.5, (c, cols.start, err)


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K,rows", [(64, 40, 140032, 64), (2048, 4096, 16640, 33), (700, 1000, 2304, 1), (6300, 17, 256, 6300), (1338, 822, 1280, 700), (1067, 2300, 5120, 500)])
def test_fp16_groups_of_many_blocks(gpu, M, N, K, rows):  # noqa: F811
    """Blocks with groups of fp16 between blocks without, one step of a block and several; many blocks a wavefront; in some
    tiles of rows only, in one row, in all; one block; items of a second round."""
    torch, binding = gpu
    codes, scales, What = tensor(torch, binding, N, K, "steps", M, z_fraction=0.02 if N < 5000 else 0.0)
    gen = torch.Generator(device="cuda").manual_seed(M)
    X = torch.randn((M, K), generator=gen, device="cuda")
    at = torch.arange(K, device="cuda")
    X[M - rows :, (at // 256) % 2 == 0] += 40.0
    X[M - rows :, (at // 256) % 5 == 3] += 25.0 * (1 - 2 * (at[(at // 256) % 5 == 3] // 64 % 2))
    X = X.half()
    Y = binding.itq3s_matmul(codes, scales, N, K, X).double()
    want = X.double() @ What.T
    assert ((Y - want).norm(dim=1) / want.norm(dim=1)).max().item() <= 2.0**-11 / 3**0.5 * 1.5  # (a row at a time: 17 outputs at the least)
