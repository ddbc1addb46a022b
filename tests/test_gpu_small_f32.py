"""float32 attention on the matrix cores, the first-layer conv with and without its pool, and the
small-tile GEMM choices, at the sizes where their tiles, masks and remainders meet."""
import numpy as np
import pytest
import torch

import oracle
import synth
from tests.helpers import TOL, rel_err
from tests.test_gpu_parity import P, _np, run_gpu, seq_ids, seq_input_model

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("b,s,heads", [(1, 1, 1), (2, 16, 3), (1, 17, 2), (3, 64, 1), (2, 65, 4), (1, 127, 2), (2, 128, 5)])
def test_attention_f32(b, s, heads):
    bld, x = seq_input_model("f32", b, s, 3 * 64 * heads, scale=1.5)
    m = bld.finish(bld.attention(x, heads, "att"), 1)
    ids = seq_ids(b, s)
    y, _, _ = run_gpu(m, ids, P.make_plan(1, [0], [1]))
    assert rel_err(_np(y), oracle.forward(m, ids)) <= 5e-6   # softmax over at most 128 float32 products of 64


def stem_model(n, c, hw, cout, pad, act, pool):
    b = synth._Builder("stem", "bf16", n, 17)
    x = b.tensor((n, c, hw[0], hw[1]), "f32")
    b.new_layer("L0")
    y = b.conv(x, cout, 7, 2, pad, act, "c", bn_fold=True)
    if pool:
        y = b.maxpool(y, 3, 2, 1, "p")
    return b.finish(y, 1)


@pytest.mark.parametrize("n,c,hw,cout,pad,act", [
    (2, 3, (97, 61), 64, 3, "relu"),     # odd, not square: conv 49 x 31, pool 25 x 16, partial tiles both ways
    (1, 3, (64, 224), 64, 3, "none"),    # whole tiles; negative results
    (1, 4, (33, 35), 72, 0, "relu"),     # four channels, no padding, a second group of 8 output channels
    (2, 1, (15, 9), 8, 2, "relu"),       # smaller than a tile
])
def test_first_layer_conv_and_pool(n, c, hw, cout, pad, act):
    x = synth.random_tensor((n, c, *hw), "f32", seed=21)
    m = stem_model(n, c, hw, cout, pad, act, True)
    plan = P.make_plan(1, [0], [1])
    y, _, _ = run_gpu(m, x, plan)
    assert rel_err(_np(y), oracle.forward(m, x)) <= TOL["bf16"]
    # while ops are timed: the same bits, and a time for both ops
    sm = P.SlicedModel(m)
    sm.set_timing(True)
    out = sm.forward(plan, torch.from_numpy(np.ascontiguousarray(x)).cuda(), sm.alloc_output(), ws=sm.alloc_workspace(plan))
    torch.cuda.synchronize()
    assert torch.equal(out, y) and min(sm.op_times()[0]) > 0
    mc = stem_model(n, c, hw, cout, pad, act, False)
    yc, _, _ = run_gpu(mc, x, plan)
    assert rel_err(_np(yc), oracle.forward(mc, x)) <= TOL["bf16"]


@pytest.mark.parametrize("bad", [np.inf, np.nan])
def test_first_layer_conv_keeps_a_non_finite_pixel_to_its_windows(bad):
    x = synth.random_tensor((1, 3, 40, 40), "f32", seed=23)
    x[0, 1, 17, 20] = bad                # one column right of the 7 taps of output column 8
    m = stem_model(1, 3, (40, 40), 16, 3, "none", False)
    y, _, _ = run_gpu(m, x, P.make_plan(1, [0], [1]))
    got, ref = _np(y), oracle.forward(m, x)
    assert 0 < (~np.isfinite(ref)).sum() < ref.size // 8
    assert np.array_equal(np.isfinite(got), np.isfinite(ref))
    ok = np.isfinite(ref)
    assert rel_err(got[ok], ref[ok]) <= TOL["bf16"]


def test_pool_of_a_tensor_read_twice_stays_its_own_pass():
    n, hw = 1, (40, 40)
    b = synth._Builder("stem2", "bf16", n, 18)
    x = b.tensor((n, 3, *hw), "f32")
    b.new_layer("L0")
    y = b.conv(x, 16, 7, 2, 3, "relu", "c", bn_fold=True)
    z = b.maxpool(y, 3, 2, 1, "p")
    w = b.conv(y, 16, 3, 2, 1, "relu", "q", res=z, bn_fold=True)
    m = b.finish(w, 1)
    xi = synth.random_tensor((n, 3, *hw), "f32", seed=22)
    o, _, _ = run_gpu(m, xi, P.make_plan(1, [0], [1]))
    assert rel_err(_np(o), oracle.forward(m, xi)) <= TOL["bf16"]


@pytest.mark.parametrize("dt,m,k,n,ksub", [
    ("f32", 65, 1028, 68, 3),      # few tiles: K split over the waves, a K tail, blocks of 64 summed
    ("f32", 256, 96, 128, 2),
    ("f32", 308, 780, 768, 4),     # 64-row tiles, no split-K
    ("f32", 300, 1100, 200, 3),    # split-K with blocked sums
    ("bf16", 33, 520, 130, 4),     # 32 x 16 tiles, ragged
    ("bf16", 64, 72, 1024, 1),
    ("f32", 33, 100, 9220, 8),     # 32 x 16 tiles, 145 blocks of 64 x 64 unsplit, 152 in sub-slices
    ("f32", 64, 36, 12300, 4),     # 193 blocks: 64 x 64 tiles
    ("f32", 17, 36, 16400, 5),     # up to 32 rows always 32 x 16
    ("f32", 77, 780, 768, 3),      # 24 tiles: four splits of a ragged K
    ("f32", 16, 2056, 700, 4),     # 16 x 64 tiles, sixteen splits
    ("f32", 3, 1028, 72, 2),       # 32 x 16 tiles, eight splits
    ("f32", 1000, 128, 16, 3),     # 64 x 16 tiles, one block sum
    ("f32", 65, 36, 10, 2),
    ("f32", 1040, 144, 16, 3),     # 17 tiles: 64 x 16, the second block sum of 16
    ("f32", 40, 3076, 3200, 3),    # four splits of 64 x 64 tiles
])
def test_small_products(dt, m, k, n, ksub):
    bld, x = seq_input_model(dt, 1, m, k)
    y = bld.linear(x, n, "gelu", "lin", "rand", rd=True)
    mod = bld.finish(y, 1)
    ids = seq_ids(1, m)
    y1, _, _ = run_gpu(mod, ids, P.make_plan(1, [0], [1]))
    assert rel_err(_np(y1), oracle.forward(mod, ids)) <= TOL[dt]
    yk, _, _ = run_gpu(mod, ids, P.make_plan(1, [0], [ksub]))
    assert torch.equal(yk, y1)


def two_node_stem(n=2, hw=(50, 62)):
    b = synth._Builder("stem3", "bf16", n, 19)
    x = b.tensor((n, 3, *hw), "f32")
    b.new_layer("conv")
    y = b.conv(x, 24, 7, 2, 3, "relu", "c", bn_fold=True)
    b.new_layer("pool")
    return b.finish(b.maxpool(y, 3, 2, 1, "p"), 1), synth.random_tensor((n, 3, *hw), "f32", seed=24)


def test_first_layer_conv_and_pool_of_two_nodes():
    """One kernel where both nodes sit in a slice, two where a cut parts them: the same bits."""
    m, x = two_node_stem()
    y1, _, _ = run_gpu(m, x, P.make_plan(2, [1], [1, 1]))
    y2, _, _ = run_gpu(m, x, P.make_plan(2, [0, 1], [1, 1]), "raw")
    assert rel_err(_np(y1), oracle.forward(m, x)) <= TOL["bf16"]
    assert torch.equal(y1, y2)


def test_timing_runs_the_kernels_of_an_untimed_forward():
    m, x = two_node_stem()
    sm, plan = P.SlicedModel(m), P.make_plan(2, [1], [1, 1])
    xin = torch.from_numpy(np.ascontiguousarray(x)).cuda()
    ws, outs, left = sm.alloc_workspace(plan), [], []
    for timing in (False, True):
        sm.set_timing(timing)
        ws.fill_(0x5A)
        outs.append(sm.forward(plan, xin, sm.alloc_output(), ws=ws))
        torch.cuda.synchronize()
        left.append(ws.clone())
    assert torch.equal(outs[0], outs[1])
    # the conv's own result, which the one kernel keeps to itself, goes to the workspace in neither
    assert torch.equal(left[0], left[1]) and bool((left[1] == 0x5A).all())
    conv, pool = sm.op_times()[0]
    prof = [t for _, t, _, _ in sm.profile()]
    assert conv > 0 and pool > 0 and abs(pool / conv - prof[1] / prof[0]) < 1e-3 * pool / conv
    tp = sm.measure(xin, k_max=1, reps=3, ws=ws)
    assert tp[0][0] > 0 and tp[1][0] > 0


def test_pipeline_runs_the_kernels_of_a_forward():
    m, x = two_node_stem()
    sm, plan = P.SlicedModel(m), P.make_plan(2, [1], [1, 1])
    xin = torch.from_numpy(np.ascontiguousarray(x)).cuda()
    ref = sm.forward(plan, xin, sm.alloc_output(), ws=sm.alloc_workspace(plan))
    pipe = sm.pipeline(plan, "raw", None, depth=1, replicas=1)
    pipe.ws.fill_(0x5A)
    out = pipe.submit(xin, sm.alloc_output())
    pipe.synchronize()
    torch.cuda.synchronize()
    assert torch.equal(out, ref) and bool((pipe.ws == 0x5A).all())   # the conv's own result is stored in neither
