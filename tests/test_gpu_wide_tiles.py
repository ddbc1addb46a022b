"""The two-group kernel's 256 x 256 and 128 x 128 tiles at their edges: remainders of M, N and K, widths
off the 8-column group, several tiles per block, conv taps at image borders, residuals, activations and
float32 results -- against the oracle (bf16 tolerance of the parity tests) and, sub-sliced, bit for bit
against the unsplit launch.  Each case first asserts the tile that the dispatch rule takes for it."""
import pytest
import torch

import oracle
import synth
from tests.helpers import TOL, conv_halo_ok, pp_tile_size, rel_err
from tests.test_gpu_parity import P, _np, conv_model, run_gpu, seq_ids, seq_input_model

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,k,n,act,res,ksub,tile", [
    (8961, 264, 1000, "gelu", False, 3, 256),     # 36 x 4 tiles: one row, 232 columns and 8 of k in the last ones
    (8961, 320, 1001, "relu", True, 4, 256),      # rows at odd addresses, a last group of one column, residual
    (8960, 256, 1022, "none", False, 2, 256),     # a last group of six columns
    (20001, 256, 1000, "none", True, 8, 256),     # 79 x 4 tiles: two per block, residual
    (4481, 264, 500, "gelu", False, 3, 128),      # 128-wide tiles, 36 x 4: one row, 116 columns, 8 of k in the last ones
    (4480, 576, 513, "relu", True, 4, 128),       # 35 x 5, the last with one column; rows at odd addresses, residual
    (12801, 256, 512, "none", True, 8, 128),      # 101 x 4 in two rounds, residual
    (20001, 296, 1004, "gelu", True, 1, 256),     # the same off the group, a last group of four columns
])
def test_linear_edges(m, k, n, act, res, ksub, tile):
    assert pp_tile_size(m, n, k) == tile
    bld, x = seq_input_model("bf16", 1, m, k)
    r = bld.linear(x, n, "none", "r", "rand") if res else None
    y = bld.linear(x, n, act, "lin", "rand", res=r, rd=True)
    mod = bld.finish(y, 1)
    ids = seq_ids(1, m)
    y1, _, _ = run_gpu(mod, ids, P.make_plan(1, [0], [1]))
    assert rel_err(_np(y1), oracle.forward(mod, ids)) <= TOL["bf16"]
    yk, _, _ = run_gpu(mod, ids, P.make_plan(1, [0], [ksub]))
    assert torch.equal(yk, y1)


@pytest.mark.parametrize("n,c,hw,cout,k,stride,pad,residual,tile", [
    (9, 64, 63, 200, 3, 1, 1, False, 256),        # 140 tiles, 200 of 256 columns, borders on every side
    (10, 128, 61, 201, 3, 1, 1, True, 256),       # odd width with a residual
    (9, 64, 126, 192, 3, 2, 1, False, 256),       # strided
    (9, 64, 63, 192, 5, 1, 2, False, 256),        # 25 taps, two pixels of padding
    (5, 128, 61, 128, 3, 1, 1, True, 128),        # 128-wide tiles: 146, residual
    (5, 64, 123, 100, 3, 2, 1, False, 128),       # 149, strided, 100 of 128 columns
    (19, 256, 31, 132, 1, 2, 0, False, 0),      # a strided 1x1 conv, 38 x 2 tiles stay on the general path
])
def test_conv_edges(n, c, hw, cout, k, stride, pad, residual, tile):
    ho = (hw + 2 * pad - k) // stride + 1
    assert not conv_halo_ok(k, k, stride, pad, c, cout, ho, ho, n * ho * ho)
    assert pp_tile_size(n * ho * ho, cout, k * k * c) == tile
    mod = conv_model("bf16", n, c, hw, cout, k, stride, pad, residual=residual, pre=True)
    x = synth.random_tensor((n, c, hw, hw), "f32", seed=11)
    y1, _, _ = run_gpu(mod, x, P.make_plan(1, [0], [1]))
    assert rel_err(_np(y1), oracle.forward(mod, x)) <= TOL["bf16"]
    yk, _, _ = run_gpu(mod, x, P.make_plan(1, [0], [3]))
    assert torch.equal(yk, y1)


@pytest.mark.parametrize("m,k,n,act,ksub,tile", [
    (1, 256, 18000, "none", 8, 128),      # few rows on the 128-wide tiles: 141 of them, 127 rows empty
    (16, 320, 18001, "gelu", 3, 128),     # off the 8-column group
    (65, 264, 18008, "relu", 4, 128),
    (33, 264, 34000, "none", 8, 128),     # two rounds: 266 tiles
    (100, 264, 36000, "none", 8, 0),    # too few rows for a 256-wide tile: gemm_kernel's
    (300, 256, 18000, "none", 8, 128),    # 423 tiles, 1.65 rounds of a short K
    (300, 584, 18000, "none", 8, 0),
])
def test_linear_few_rows(m, k, n, act, ksub, tile):
    assert pp_tile_size(m, n, k) == tile
    bld, x = seq_input_model("bf16", 1, m, k)
    mod = bld.finish(bld.linear(x, n, act, "lin", "rand", rd=True), 1)
    ids = seq_ids(1, m)
    y1, _, _ = run_gpu(mod, ids, P.make_plan(1, [0], [1]))
    assert rel_err(_np(y1), oracle.forward(mod, ids)) <= TOL["bf16"]
    yk, _, _ = run_gpu(mod, ids, P.make_plan(1, [0], [ksub]))
    assert torch.equal(yk, y1)


@pytest.mark.parametrize("b,t,e,h,tile", [
    (897, 5, 264, 136, 128),     # 36 x 5 tiles: five rows, 32 of 544 columns and 8 of k in the last ones
    (6667, 3, 256, 248, 256),    # 79 x 4, two per block: 33 rows, 224 of 992 columns
    (2988, 3, 264, 256, 256),    # 36 x 4, whole columns, 8 of k
])
def test_lstm_input_projection_edges(b, t, e, h, tile):
    assert pp_tile_size(b * t, 4 * h, e) == tile
    bld, x = seq_input_model("bf16", b, t, e)
    mod = bld.finish(bld.lstm(x, h, "lstm", -0.1, 0.1), 1)
    ids = seq_ids(b, t)
    y, _, _ = run_gpu(mod, ids, P.make_plan(1, [0], [1]))
    assert rel_err(_np(y), oracle.forward(mod, ids)) <= TOL["bf16"]
