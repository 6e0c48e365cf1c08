"""The block-scaled kernels, the tiled one above all: several tensors in one launch, tensors of several kernels in a call, and
what they keep in the workspace (the rotated activations) under reuse, graph replay, threads and the static scratch.
Every test asserts which kernel takes each of its tensors, by the rule that the library is built with, and that the workspace
holds the operand of the block-scaled kernels behind the call.  Results against itq3s_dequantize (held to the
oracle within 1e-6 elsewhere) and a dense fp64 product."""
import threading

import numpy as np
import pytest

from tests.block_scaled import ROWS, SHARES4, SHARES8, TILED, holds_operand, route
from tests.test_gpu_rows import check, gpu, tensor  # noqa: F401  (gpu is a fixture)

pytestmark = pytest.mark.gpu


def activations(torch, M, K, seed):
    return torch.randn((M, K), generator=torch.Generator(device="cuda").manual_seed(seed), device="cuda").half()


def workspace(torch, binding, calls, fill=0xA5):
    return torch.full((max(binding.itq3s_matmul_workspace_bytes(*c) for c in calls),), fill, dtype=torch.uint8, device="cuda")


# (M, K, N...): tiled tensors, three and four to a launch, ragged, so that a chiplet's run of items and a workgroup's
# neighbours cross from one tensor to the next
TOGETHER = [(517, 512, (9300, 8200, 12001)), (1030, 256, (4100, 4352, 5000, 3800)), (600, 1024, (7000, 11008))]
# ... next to tensors of the other kernels (N: its kernel)
MIXED = [(512, 2048, (7000, 9000, 300, 12001)), (513, 2304, (6650, 8300, 6700)), (512, 4096, (7936, 4096, 1000))]
OTHERS = {300: ROWS, 4096: SHARES4, 1000: SHARES8}


def kernels(M, K, Ns):
    got = [route(M, N, K) for N in Ns]
    assert got == [OTHERS.get(N, TILED) if (M, K, Ns) in MIXED else TILED for N in Ns], got


@pytest.mark.parametrize("M,K,Ns", TOGETHER + MIXED)
def test_grouped_equals_single_calls(gpu, M, K, Ns):
    torch, binding = gpu
    kernels(M, K, Ns)
    ts = [tensor(torch, binding, N, K, "tg", i, z_fraction=(0.0, 0.02, 0.7, 0.02)[i]) for i, N in enumerate(Ns)]
    buf = activations(torch, M, K + 8, M)
    X = buf[:, :K]
    ws = workspace(torch, binding, [(M, N, K) for N in Ns])
    for dtype in (torch.float16, torch.float32):
        outs = [torch.full((M, N + 5), 7.0, dtype=dtype, device="cuda") for N in Ns]
        flags = torch.zeros(1, dtype=torch.int32, device="cuda")
        binding.itq3s_matmul_grouped([(c, s, N) for (c, s, _), N in zip(ts, Ns)], K, X, outs=[o[:, :N] for o, N in zip(outs, Ns)],
                                     workspace=ws, status_flags=flags)
        assert int(flags.item()) == 0 and holds_operand(torch, ws, X)
        for (c, s, What), N, out in zip(ts, Ns, outs):
            assert bool((out[:, N:] == 7.0).all())
            assert torch.equal(out[:, :N], binding.itq3s_matmul(c, s, N, K, X, dtype=dtype))
            check(out[:, :N], X, What, dtype == torch.float16)


@pytest.mark.parametrize("M,K,Ns", [TOGETHER[0], MIXED[1]])
def test_format_check_covers_the_last_tensor_of_a_group(gpu, M, K, Ns):
    torch, binding = gpu
    kernels(M, K, Ns)
    ts = [tensor(torch, binding, N, K, "tb", i) for i, N in enumerate(Ns)]
    bad = ts[-1][0].clone()
    bad[-384 + 256 + 9] = 1 << 7  # a high-plane bit in the last tile
    X = activations(torch, M, K, 1)
    for last, expect in ((ts[-1][0], 0), (bad, binding.FLAG_BAD_CODE)):
        flags = torch.zeros(1, dtype=torch.int32, device="cuda")
        ws = workspace(torch, binding, [(M, N, K) for N in Ns])
        group = [(c, s, N) for (c, s, _), N in zip(ts[:-1], Ns)] + [(last, ts[-1][1], Ns[-1])]
        binding.itq3s_matmul_grouped(group, K, X, workspace=ws, status_flags=flags)
        assert holds_operand(torch, ws, X) and int(flags.item()) == expect


@pytest.mark.parametrize("M,N,K,kernel", [(2051, 40, 8192, SHARES8), (517, 3000, 4096, SHARES4), (517, 7000, 2048, TILED)])
def test_activation_range_flag(gpu, M, N, K, kernel):
    """At the edge of the stated domain the flag stays clear; beyond it (the intermediate, the rotated value,
    an infinity, in the first and the last row) it is set, and other rows are not touched."""
    torch, binding = gpu
    assert route(M, N, K) == kernel
    codes, scales, What = tensor(torch, binding, N, K, "tr")
    base = activations(torch, M, K, 2)
    ws = workspace(torch, binding, [(M, N, K)])

    def run(X):
        flags = torch.zeros(1, dtype=torch.int32, device="cuda")
        return binding.itq3s_matmul(codes, scales, N, K, X, workspace=ws, status_flags=flags), int(flags.item())

    X = base.clone()
    X[0, 288:304] = 16376.0
    X[M - 1, K - 256 :] = 4094.0
    Y, f = run(X)
    assert f == 0
    check(Y, X, What, False)
    for row, cols, value in ((M - 1, slice(16, 32), 16400.0), (0, slice(512, 768), 4100.0), (M - 1, slice(K - 1, K), float("inf"))):
        X = base.clone()
        X[row, cols] = value
        Y, f = run(X)
        assert f == binding.FLAG_ACT_RANGE
        keep = torch.arange(M, device="cuda") != row
        check(Y[keep], X[keep], What, False)


@pytest.mark.parametrize("M,N,K,kernel", [(512, 7000, 2048, TILED), (2100, 300, 8192, SHARES8), (517, 9300, 512, TILED), (517, 3000, 4096, SHARES4)])
def test_fp16_output_with_zero_points_in_most_blocks(gpu, M, N, K, kernel):
    """The zero-point terms are applied before the output is rounded (bars as for the smaller calls of the same kind)."""
    torch, binding = gpu
    assert route(M, N, K) == kernel
    codes, scales, What = tensor(torch, binding, N, K, "tz", z_fraction=0.9)
    X = activations(torch, M, K, 3)
    want = X.double() @ What.T
    ws = workspace(torch, binding, [(M, N, K)])
    for dtype, bar in ((torch.float16, 1e-3), (torch.float32, 6e-4)):
        got = binding.itq3s_matmul(codes, scales, N, K, X, dtype=dtype, workspace=ws).double()
        assert holds_operand(torch, ws, X)
        assert ((got - want).norm(dim=1) / want.norm(dim=1)).max().item() <= bar


# one workspace for the calls of all kernels
STATE = [(512, 7000, 2048), (517, 9300, 512), (2100, 300, 8192), (48, 500, 2048), (513, 6700, 2304), (517, 3000, 4096), (600, 7000, 1024)]


def test_state_calls_are_of_all_kernels():
    assert [route(*s) for s in STATE] == [TILED, TILED, SHARES8, ROWS, TILED, SHARES4, TILED]


def state_calls(torch, binding, key):
    calls = []
    for i, (M, N, K) in enumerate(STATE):
        c, s, What = tensor(torch, binding, N, K, key, i, z_fraction=(0.02, 0.0)[i & 1])
        calls.append((c, s, N, K, activations(torch, M, K, 10 + i), What))
    return calls


def test_calls_share_a_workspace_of_garbage(gpu):
    """In changing order, without synchronisation in between: every result equals the one computed alone."""
    torch, binding = gpu
    calls = state_calls(torch, binding, "ts")
    alone = [binding.itq3s_matmul(c, s, N, K, X) for c, s, N, K, X, _ in calls]
    for (c, s, N, K, X, What), Y in zip(calls, alone):
        check(Y, X, What, False)
    ws = workspace(torch, binding, STATE, fill=0xFF)
    for step in (1, 2, 3, 4):  # (seven calls: every order has all of them)
        order = [(step * i) % len(calls) for i in range(len(calls))]
        outs = [binding.itq3s_matmul(*calls[i][:5], workspace=ws) for i in order]
        torch.cuda.synchronize()
        for i, out in zip(order, outs):
            assert torch.equal(alone[i], out), (step, i)


def test_captured_calls_replay_like_eager(gpu):
    """Single calls and a mixed group in one HIP graph; before every replay the workspace and the outputs are
    overwritten, eager work runs in between, and every replay reproduces the eager bits."""
    torch, binding = gpu
    calls = state_calls(torch, binding, "tc")
    M, K, Ns = MIXED[0]
    group = [tensor(torch, binding, N, K, "tcg", i)[:2] + (N,) for i, N in enumerate(Ns)]
    Xg = activations(torch, M, K, 20)
    ws = workspace(torch, binding, STATE + [(M, N, K) for N in Ns])
    outs = [torch.empty((X.shape[0], N), device="cuda") for _, _, N, _, X, _ in calls]
    gouts = [torch.empty((M, N), dtype=torch.float16, device="cuda") for N in Ns]
    flags = torch.zeros(1, dtype=torch.int32, device="cuda")

    def enqueue():
        for (c, s, N, Kc, X, _), out in zip(calls, outs):
            binding.itq3s_matmul(c, s, N, Kc, X, out=out, workspace=ws, status_flags=flags)
        binding.itq3s_matmul_grouped(group, K, Xg, outs=gouts, workspace=ws, status_flags=flags)

    enqueue()
    torch.cuda.synchronize()
    eager = [t.clone() for t in outs + gouts]
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        enqueue()
    for rep in range(3):
        for t in outs + gouts:
            t.fill_(float("nan"))
        ws.fill_(0x5A + rep)
        torch.cuda.synchronize()
        g.replay()
        binding.itq3s_matmul(*calls[0][:5])  # eager work of the program between the replays
        torch.cuda.synchronize()
        assert holds_operand(torch, ws, Xg) and int(flags.item()) == 0
        for a, b in zip(eager, outs + gouts):
            assert torch.equal(a, b), rep


def test_two_host_threads(gpu):
    torch, binding = gpu
    calls = state_calls(torch, binding, "tt")
    alone = [binding.itq3s_matmul(c, s, N, K, X) for c, s, N, K, X, _ in calls]
    torch.cuda.synchronize()
    errors = []

    def worker(timed):
        try:
            torch.cuda.set_device(0)
            ws = workspace(torch, binding, STATE)
            call = binding.itq3s_matmul_timed if timed else binding.itq3s_matmul
            for _ in range(4):
                outs = [call(*c[:5], workspace=ws) for c in calls]
                torch.cuda.synchronize()
                for a, b in zip(alone, outs):
                    assert torch.equal(a, b[0] if timed else b)
        except BaseException as e:  # reported by the main thread
            errors.append(repr(e))

    threads = [threading.Thread(target=worker, args=(t,)) for t in (False, True)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors


def test_static_scratch(gpu):
    """Calls of all kernels one after another in the static array, twice."""
    torch, binding = gpu
    for c, s, N, K, X, _ in state_calls(torch, binding, "tn") * 2:
        want = binding.itq3s_matmul(c, s, N, K, X)
        out = torch.full_like(want, float("nan"))
        assert torch.equal(binding.itq3s_matmul_static(c, s, N, K, X, out), want), (X.shape[0], N, K)


@pytest.mark.parametrize("seed", [1, 2])
def test_random_shapes(gpu, seed):
    """Seeded shapes beyond the many-row kernel's (more than 3.4 million outputs), with and without zero-points; all but
    a few the tiled kernel's."""
    torch, binding = gpu
    rng = np.random.default_rng(seed)
    taken = [0] * 4
    for i in range(24):
        K = 256 * int(rng.choice([1, 2, 3, 5, 8, 9, 11, 16, 20]))
        M = int(rng.integers(200, 2500))
        N = int(rng.integers(3_450_000 // M + 1, 3 * 3_450_000 // M))
        codes, scales, What = tensor(torch, binding, N, K, "trs", seed, i, z_fraction=float(rng.choice([0.0, 0.001, 0.05, 0.8])))
        X = activations(torch, M, K, 100 * seed + i)
        if rng.random() < 0.3:
            X[:, ::97] *= 10
        ws = workspace(torch, binding, [(M, N, K)])
        taken[route(M, N, K)] += 1
        for dtype in (torch.float32, torch.float16):
            got = binding.itq3s_matmul(codes, scales, N, K, X, dtype=dtype, workspace=ws)
            assert holds_operand(torch, ws, X), (M, N, K)
            check(got, X, What, dtype == torch.float16)
    assert taken[ROWS] == 0 and taken[TILED] >= 20, taken
