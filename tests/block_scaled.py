"""For the tests of the calls with more than 16 rows: which kernel takes a size (the host rule, compiled from its header), and
the operand that the block-scaled kernels read, decoded from a workspace."""
import atexit
import functools
import os
import shutil
import subprocess
import tempfile

ROWS, SHARES8, SHARES4, TILED = range(4)  # many-row kernel; K over 8 and over 4 wavefronts; tiles

MAIN = r"""
#include "itq3s_mx_rule.h"
#include <cstdio>
int main() {
    long long M, N, K;
    while (std::scanf("%lld %lld %lld", &M, &N, &K) == 3) {
        const itq3s::Route r = itq3s::many_row_route(M, N, K);
        const int64_t n = N;
        // of a call with this tensor alone, for 256 units: items, and the columns of one
        long long items = 0, cols = 256;
        if (r == itq3s::Route::rows) {
            const itq3s::RowsSplit s = itq3s::rows_split((N + 15) / 16, M, K, 256);
            items = s.items;
            cols = 16 * s.rt;
        } else {
            if (r == itq3s::Route::shares8) cols = 32 * itq3s::shares8_columns(&n, 1, M, K, 256);
            items = (M + (r == itq3s::Route::tiled ? 63 : 31)) / (r == itq3s::Route::tiled ? 64 : 32) * ((N + cols - 1) / cols);
        }
        std::printf("%d %lld %lld\n", (int)r, items, cols);
    }
}
"""


@functools.lru_cache(maxsize=None)
def _rule():
    from paper_2603_27914_amd import build

    folder = tempfile.mkdtemp(prefix="itq3s_rule_")
    atexit.register(shutil.rmtree, folder, ignore_errors=True)
    source, exe = os.path.join(folder, "rule.cpp"), os.path.join(folder, "rule")
    with open(source, "w") as f:
        f.write(MAIN)
    subprocess.run(["g++", "-std=c++17", "-I", build.CSRC, source, "-o", exe], check=True)
    return exe


@functools.lru_cache(maxsize=None)
def route_items_columns(M, N, K):
    out = subprocess.run([_rule()], input="%d %d %d\n" % (M, N, K), check=True, stdout=subprocess.PIPE, text=True).stdout.split()
    return tuple(int(v) for v in out)


def route(M, N, K):
    return route_items_columns(M, N, K)[0]


def holds_operand(torch, ws, X):
    """Whether the workspace starts with the rotated activations as the block-scaled kernels read them: per 32 rows and block
    four steps of 64 channels, three parts of fp6 (e2m3) under one power of two per 32 channels and row (the first two
    tiles of rows; ordinary activations, which need no fp16 step)."""
    M, K = X.shape
    rows = min(M, 64)
    tiles, KB = (rows + 31) // 32, K // 256
    i = torch.arange(256, device="cuda")
    bits = i[:, None] & i[None, :]
    parity = sum((bits >> b) & 1 for b in range(8)) & 1
    H = (1 - 2 * parity).double() / 16.0
    want = (X[:rows].double().reshape(-1, 256) @ H).reshape(rows, KB, 256)
    raw = ws[: tiles * KB * 18944].view(tiles, KB, 18944)
    steps = raw[:, :, : 4 * 4608].reshape(tiles, KB, 4, 3, 1536)
    # lane 32 kg + row of a step: 16 bytes, and 8 behind the lanes' 16
    lane = torch.cat([steps[..., :1024].reshape(tiles, KB, 4, 3, 64, 16), steps[..., 1024:].reshape(tiles, KB, 4, 3, 64, 8)], dim=-1).long()
    j = torch.arange(32, device="cuda") * 6
    pair = lane | torch.cat([lane[..., 1:], torch.zeros_like(lane[..., :1])], dim=-1) << 8
    field = (pair[..., j // 8] >> (j % 8)) & 63
    e, m = (field >> 3) & 3, (field & 7).double()
    value = torch.where(e == 0, m / 8, (1 + m / 8) * 2.0 ** (e - 1).double()) * torch.where(field >= 32, -1.0, 1.0)
    value = value[..., 0, :, :] + value[..., 1, :, :] / 16 + value[..., 2, :, :] / 512  # tile, block, step, lane, place
    scale = raw[:, :, 4 * 4608 : 4 * 4608 + 256].reshape(tiles, KB, 64, 4).long()  # byte q of a lane: step q
    value = value * 2.0 ** (scale.permute(0, 1, 3, 2).double() - 127)[..., None]
    # step 2 h + odd, lane 32 kg + row, place 8 i + s / 2: element 64 (2 h + kg) + 16 i + s, s = 2 (place % 8) + odd
    got = value.view(tiles, KB, 2, 2, 2, 32, 4, 8).permute(0, 5, 1, 2, 4, 6, 7, 3).reshape(tiles * 32, KB, 256)[:rows]
    group = want.view(rows, KB, 4, 4, 8, 2).abs().amax(dim=(3, 4), keepdim=True)
    err = (got - want).view(rows, KB, 4, 4, 8, 2).abs()
    # 2^-12 / 3.75 of the largest of the 32; the rotation itself, whose intermediate has 22 bits
    return bool((err <= (2.0**-12 / 3.75 + 2.0**-18) * group).all())  # (false for NaN)
