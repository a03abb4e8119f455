"""GPU parity of the exact scorers (Direct, GIP, PIP) against the oracle.

The oracle's Direct scorer (explicit fp64 gradients; pinned against GIP, PIP
and autograd) is the reference for all three methods.  Inputs are bf16,
every product is exact in fp32 and the target-mean gradient enters PIP as a
bf16 hi + lo pair (relative rounding ~2^-17), so each layer's score vector
must match to a relative error of 1e-4 (tighter than the 2e-3 allowed for
bf16 sketches).
"""

import numpy as np
import pytest
import torch

import oracle
from paper_2605_07063_amd import api
from gpu_helpers import host64, rel

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
TOL_SCORE = 1e-4
METHODS = ["direct", "gip", "pip"]


def make(specs, N, T, lens, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(777 + seed)
    mask = torch.arange(T, device=DEV)[None, :] >= lens[:, None]
    out = []
    for di, do in specs:
        x = torch.randn(N, T, di, generator=g, device=DEV).to(torch.bfloat16)
        dy = torch.randn(N, T, do, generator=g, device=DEV).to(torch.bfloat16)
        x[mask] = float("nan")
        dy[mask] = float("nan")
        out.append(dict(x=x, dy=dy))
    return out


def reference(layers, n, m, lens):
    lh = lens.cpu().numpy()
    refs = []
    for L in layers:
        x, dy = host64(L["x"]), host64(L["dy"])
        refs.append(oracle.score_direct(x[:n], dy[:n], lh[:n], x[n:n + m], dy[n:n + m], lh[n:n + m]))
    return refs


@pytest.mark.parametrize("method", METHODS)
def test_ragged_lengths_and_dimension_tails(method):
    n, m, T = 7, 3, 150
    lens = torch.tensor([150, 0, 1, 127, 128, 129, 60, 150, 0, 77], dtype=torch.int32, device=DEV)
    layers = make([(136, 264), (64, 200)], n + m, T, lens, seed=1)
    s = api.score_exact(layers, n, m, lens, method=method)
    torch.cuda.synchronize()
    for l, ref in enumerate(reference(layers, n, m, lens)):
        got = host64(s[l])
        assert np.isfinite(got).all()
        assert got[1] == 0.0                              # an empty example scores exactly 0
        assert rel(got, ref) <= TOL_SCORE, f"{method} layer {l}: {rel(got, ref):.2e}"


def test_methods_agree_at_full_layer_width():
    """One 2048 x 2048 layer of the small-block workload's shape, 16 general
    and 4 target examples of up to 512 tokens."""
    n, m, T = 16, 4, 512
    lens = torch.randint(128, T + 1, (n + m,), generator=torch.Generator().manual_seed(2),
                         dtype=torch.int32).to(DEV)
    layers = make([(2048, 2048)], n + m, T, lens, seed=2)
    (ref,) = reference(layers, n, m, lens)
    outs = {}
    for method in METHODS:
        s = api.score_exact(layers, n, m, lens, method=method)
        torch.cuda.synchronize()
        outs[method] = host64(s[0])
        assert rel(outs[method], ref) <= TOL_SCORE, f"{method}: {rel(outs[method], ref):.2e}"
    # the orderings agree with each other (top-4 sets too)
    for method in METHODS:
        assert set(np.argsort(-outs[method])[:4]) == set(np.argsort(-ref)[:4])


def test_null_lengths_and_no_general_examples():
    n, m, T = 4, 2, 40
    full = torch.full((n + m,), T, dtype=torch.int32, device=DEV)
    layers = make([(64, 64)], n + m, T, full, seed=3)
    for method in METHODS:
        a = api.score_exact(layers, n, m, None, method=method)
        b = api.score_exact(layers, n, m, full, method=method)
        torch.cuda.synchronize()
        assert torch.equal(a, b)
        s = torch.empty(1, 0, device=DEV)
        api.dr_score_exact(layers, 0, m, T, None, method, s)


def check_all(layers, n, m, lens, methods):
    refs = reference(layers, n, m, lens)
    for method in methods:
        s = api.score_exact(layers, n, m, lens, method=method)
        torch.cuda.synchronize()
        for l, ref in enumerate(refs):
            got = host64(s[l])
            assert np.isfinite(got).all()
            assert (got[lens[:n].cpu().numpy() == 0] == 0.0).all()
            assert rel(got, ref) <= TOL_SCORE, f"{method} layer {l}: {rel(got, ref):.2e}"


def test_packed_tiles_of_many_short_examples():
    """Tiles that hold many examples, with a run of more empty examples than
    a tile has rows inside one tile, and output blocks past 256 columns."""
    n, m, T = 700, 40, 5
    g = torch.Generator().manual_seed(4)
    lens = torch.randint(0, T + 1, (n + m,), generator=g, dtype=torch.int32)
    lens[30:330] = 0
    lens[n + 3:n + 9] = 0
    lens = lens.to(DEV)
    check_all(make([(72, 520), (136, 8)], n + m, T, lens, seed=4), n, m, lens, ["gip", "pip"])


@pytest.mark.parametrize("length", [255, 256, 257])
def test_packed_tile_edges(length):
    n, m, T = 3, 2, 257
    lens = torch.tensor([length, 1, length, length, 128], dtype=torch.int32, device=DEV)
    check_all(make([(64, 264)], n + m, T, lens, seed=5), n, m, lens, ["gip", "pip"])


def test_rows_further_apart_than_a_tile_can_address():
    """Row strides for which the examples of one tile would span 4 GiB: a
    tile then holds rows of one example only."""
    n, m, T, ld = 5, 2, 300, 1_500_000
    lens = torch.tensor([300, 0, 257, 128, 1, 300, 129], dtype=torch.int32, device=DEV)
    layers = make([(72, 136)], n + m, T, lens, seed=6)
    wide = torch.empty((n + m) * T * ld, dtype=torch.bfloat16, device=DEV).view(n + m, T, ld)
    wide[:, :, :72] = layers[0]["x"]
    layers[0]["x"] = wide[:, :, :72]
    check_all(layers, n, m, lens, ["gip", "pip"])


def test_empty_examples_between_the_rows_of_a_tile():
    """Runs of empty examples inside one tile (general rows, and targets) over which the examples lie more than 4 GiB
    apart, although as many examples as a tile has rows do not.  What 32-bit offsets would wrap to is padding (NaN)."""
    n, m, T, ld = 700, 600, 8, 524288      # 8 MiB an example: 512 of them reach 4 GiB
    lens = torch.zeros(n + m, dtype=torch.int32)
    for i, L in ((0, 8), (2, 3), (514, 5), (600, 8), (601, 1), (699, 7), (n, 8), (n + 1, 2), (n + 520, 8), (n + 599, 4)):
        lens[i] = L
    lens[603:640] = 8                      # a second tile of 128 rows
    lens = lens.to(DEV)
    layers = make([(72, 136)], n + m, T, lens, seed=8)
    wide = torch.empty((n + m) * T * ld, dtype=torch.bfloat16, device=DEV).view(n + m, T, ld)
    wide[:, :, :72] = layers[0]["x"]
    layers[0]["x"] = wide[:, :, :72]
    check_all(layers, n, m, lens, ["gip", "pip"])


def test_more_tiles_than_one_grid_dimension_takes():
    """2^24 tiles of 256 threads (by T, not by the lengths): a launch takes fewer than 2^32 threads per dimension."""
    n, m, T, count = 512, 32, 1024, 16
    assert (n * T // 128) * (m * T // 128) * count * 256 >= 1 << 32
    g = torch.Generator().manual_seed(9)
    lens = torch.randint(0, 4, (n + m,), generator=g, dtype=torch.int32)
    lens[n - 1], lens[n + m - 1] = 300, 200
    lens = lens.to(DEV)
    layers = make([(8, 16)], n + m, T, lens, seed=9)
    (ref,) = reference(layers, n, m, lens)
    s = api.score_exact(layers * count, n, m, lens, method="gip")
    torch.cuda.synchronize()
    for l in range(count):
        assert rel(host64(s[l]), ref) <= TOL_SCORE


def test_layer_groups():
    """More layers than one group holds, of different widths."""
    n, m, T = 3, 2, 20
    lens = torch.tensor([20, 7, 16, 20, 3], dtype=torch.int32, device=DEV)
    specs = [(64 + 8 * (l % 5), 40 + 72 * (l % 4)) for l in range(18)]
    check_all(make(specs, n + m, T, lens, seed=7), n, m, lens, METHODS)


# Calls of up to 256 tiles of 128 x 128 (at T tokens an example) take rows of one example to a tile; larger ones pack
# the tokens.

@pytest.mark.parametrize("length", [255, 256, 257])
def test_packed_tile_edges_of_larger_calls(length):
    n, m, T = 3, 2, 257
    lens = torch.tensor([length, 1, length, length, 128], dtype=torch.int32, device=DEV)
    check_all(make([(64, 3720)], n + m, T, lens, seed=5), n, m, lens, ["pip"])
    check_all(make([(64, 264)] * 10, n + m, T, lens, seed=5), n, m, lens, ["gip"])


def test_rows_further_apart_in_a_larger_call():
    n, m, T, ld = 5, 2, 300, 1_500_000
    lens = torch.tensor([300, 0, 257, 128, 1, 300, 129], dtype=torch.int32, device=DEV)
    layers = make([(72, 2200)], n + m, T, lens, seed=6)
    wide = torch.empty((n + m) * T * ld, dtype=torch.bfloat16, device=DEV).view(n + m, T, ld)
    wide[:, :, :72] = layers[0]["x"]
    layers[0]["x"] = wide[:, :, :72]
    check_all(layers, n, m, lens, ["pip"])


def test_layer_groups_of_packed_tiles():
    n, m, T = 30, 10, 20
    g = torch.Generator().manual_seed(10)
    lens = torch.randint(0, T + 1, (n + m,), generator=g, dtype=torch.int32).to(DEV)
    specs = [(64 + 8 * (l % 5), 40 + 72 * (l % 4)) for l in range(18)]
    check_all(make(specs, n + m, T, lens, seed=7), n, m, lens, METHODS)


@pytest.mark.parametrize("d_in,d_out", [(8, 8), (64, 128), (72, 136), (200, 1000)])
@pytest.mark.parametrize("T", [1, 127, 128, 129])
def test_small_calls_at_the_edges_of_a_tile(T, d_in, d_out):
    n, m = 5, 2
    lens = torch.tensor([T, 0, 1, max(1, T - 1), T, T, 1], dtype=torch.int32, device=DEV)
    check_all(make([(d_in, d_out)], n + m, T, lens, seed=11), n, m, lens, ["gip", "pip"])
