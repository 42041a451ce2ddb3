"""Batches of a few tokens and large ones, which run kernels of their own:
captured in a graph, on a side stream, by every path, with values that are not
finite in one token, and where the two projections run different kernels.  That
the kernels named here are the ones that run is checked without a GPU."""
import numpy as np
import pytest
import torch

from paper_2607_00466_amd import binding as B
from paper_2607_00466_amd import synth
from tests import gpu_util as G
from tests import test_gpu_ffn_wide as W
from tests import test_gpu_mxfp4 as MX
from tests import test_gpu_parity as P

pytestmark = pytest.mark.gpu

# (format, E, K, H, I, T): the one-wave kernel, the wide kernel behind several
# bucket workgroups and the gate by token tiles, and in between.
SLIM = [("bf16", 40, 5, 544, 288, 3), ("mxfp4", 40, 5, 576, 320, 3)]
WIDE = [("bf16", 248, 4, 352, 288, 2080), ("mxfp4", 248, 4, 320, 192, 2080)]
# up by the small-batch kernel with down by the wide one, then both by the wide one
MIXED = [("bf16", 64, 4, 1280, 640, 256), ("bf16", 64, 4, 1280, 640, 400)]


def _layer(fmt, E, K, H, I, T):
    sh = synth.LayerShape(f"choice_{fmt}", E=E, K=K, H=H, I=I)
    return (G.Layer if fmt == "bf16" else MX.MxLayer)(sh, T, seed=T)


def _call(layer, x, d, buf, routing, path):
    if isinstance(layer, G.Layer):
        B.moe_layer(x, layer.wg, layer.p13, layer.p2, d, buf, routing=routing, path=path)
    else:
        B.moe_layer_mxfp4(x, layer.wg, layer.up, layer.down, d, buf, routing=routing, path=path)


@pytest.mark.parametrize("case", SLIM + WIDE)
@pytest.mark.parametrize("path", ["routed", "split"])
def test_graph_replays_and_side_stream(case, path):
    fmt, E, K, H, I, T = case
    G.say(f"case: graph and side stream, {path}, {case}, gate-routed")
    layer = _layer(*case)
    d, buf = layer.d, B.LayerBuffers.allocate(layer.d)
    outputs = ("logits", "topk_ids", "topk_w", "pair_pos", "y_perm", "out")
    _call(layer, layer.x, d, buf, None, path)
    torch.cuda.synchronize()
    eager = {n: getattr(buf, n).clone() for n in outputs}
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        buf.out.fill_(float("nan"))
        _call(layer, layer.x, d, buf, None, path)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    assert torch.equal(buf.out, eager["out"]), "side stream"
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        _call(layer, layer.x, d, buf, None, path)
    for rep in range(4):
        for n in outputs:
            getattr(buf, n).fill_(-7)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        for n in outputs:
            assert torch.equal(getattr(buf, n), eager[n]), f"replay {rep}: {n}"
        _call(layer, layer.x, d, buf, None, path)  # eager work of its own between the replays
        torch.cuda.synchronize()


@pytest.mark.parametrize("case", SLIM + WIDE + MIXED)
def test_every_path_leaves_the_same_buffers(case):
    fmt, E, K, H, I, T = case
    G.say(f"case: paths, {case}")
    layer = _layer(*case)
    ids, w, _ = synth.controlled_routing(T, E, K, U=min(E, T * K), seed=T)
    runs = {p: W._run(layer, T, ids, w, p) for p in ("routed", "split", "fused")}
    for p in ("split", "fused"):
        for n in ("counts", "offsets", "perm_token", "pair_pos", "union_ids", "union_size", "y_slots", "out"):
            assert np.array_equal(runs["routed"][n], runs[p][n]), f"{p}: {n}"
    if fmt == "bf16":
        P._full_check(layer, runs["routed"], False, routing=(ids.astype(np.int64), w))
    else:
        MX._check_layer(layer, runs["routed"], (ids, w))


@pytest.mark.parametrize("case", SLIM + WIDE + MIXED[1:])
@pytest.mark.parametrize("value", [float("inf"), float("nan")])
def test_a_token_that_is_not_finite_stays_alone(case, value):
    fmt, E, K, H, I, T = case
    G.say(f"case: one token holds {value}, {case}")
    layer = _layer(*case)
    ids, w, _ = synth.controlled_routing(T, E, K, U=min(E, 2 * K), seed=T)  # buckets shared by many tokens
    clean = W._run(layer, T, ids, w)["out"]
    bad = T // 2
    layer.x[bad, H // 3] = value
    got = W._run(layer, T, ids, w)["out"]
    assert not np.isfinite(got[bad]).any()
    rest = np.arange(T) != bad
    assert np.array_equal(got[rest], clean[rest]), "another token's output changed"
