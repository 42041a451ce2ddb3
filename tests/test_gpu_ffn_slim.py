"""The expert FFN's kernel for batches of at most 4 tokens: every bucket size
(1 .. 4 tokens), reductions of one step, one ring, one staged chunk and one
step more than each (chunks hold 64, 32 or 16 steps), bands of a short last
workgroup band, against the oracle and, bit for bit, against the same tokens
in a batch that the four-wave kernel runs; and its routing, valid or not."""
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


@pytest.mark.parametrize("fmt,H,I", [("bf16", 32, 288), ("bf16", 544, 32), ("bf16", 2080, 96), ("bf16", 1056, 2048),
                                     ("mxfp4", 64, 576), ("mxfp4", 2112, 64), ("mxfp4", 576, 1088)])
def test_bucket_sizes_and_reductions(fmt, H, I):
    E, K = 40, 5
    sh = synth.LayerShape(f"slim_{fmt}", E=E, K=K, H=H, I=I)
    layer = G.Layer(sh, 8, seed=H + I) if fmt == "bf16" else MX.MxLayer(sh, 8, seed=H + I)
    # experts 3, 20 and 39 in 4, 3 and 2 of the first 4 tokens' picks, the others once or twice
    ids, w = G.fixed_bucket_routing(8, E, K, [(3, 4), (20, 3), (39, 2)], seed=I)
    full = {path: W._run(layer, 8, ids, w, path) for path in ("routed", "split")}
    for T in (1, 2, 3, 4):
        G.say(f"case: {fmt} E={E} top-{K} H={H} I={I} T={T}")
        for path in ("routed", "split"):
            g = W._run(layer, T, ids, w, path)
            assert np.array_equal(g["out"], full[path]["out"][:T]), f"T={T} {path}: not the bits of the batch of 8"
            G.compare_buckets(g, ids[:T].astype(np.int64), E)
            assert np.array_equal(g["y_slots"], W._run(layer, T, ids, w, "routed")["y_slots"])
    if fmt == "bf16":
        P._full_check(layer, full["routed"], False, routing=(ids.astype(np.int64), w))
    else:
        MX._check_layer(layer, full["routed"], (ids, w))


@pytest.mark.parametrize("E,K,T", [(256, 16, 4), (16, 16, 3), (1, 1, 4), (256, 1, 1)])
def test_routing_limits(E, K, T):
    G.say(f"case: E={E} top-{K} T={T}, H=64 I=32")
    layer = G.Layer(synth.LayerShape("slim_route", E=E, K=K, H=64, I=32), T, seed=E + K)
    ids, w, _ = synth.controlled_routing(T, E, K, U=E, seed=T)
    P._full_check(layer, W._run(layer, T, ids, w), False, routing=(ids.astype(np.int64), w))


@pytest.mark.parametrize("kind", ["repeated", "too large", "negative"])
def test_invalid_routing_does_nothing(kind):
    layer = G.Layer(synth.LayerShape("slim_bad", E=16, K=4, H=64, I=32), 4, seed=1)
    ids, w, _ = synth.controlled_routing(4, 16, 4, U=16, seed=2)
    ids[2, 1] = {"repeated": ids[2, 0], "too large": 16, "negative": -1}[kind]
    buf = layer.buf
    buf.y_perm.fill_(123.0)
    r = (torch.from_numpy(ids).cuda(), torch.from_numpy(w).cuda())
    buf.pair_pos.fill_(-1)
    B.moe_layer(layer.x, layer.wg, layer.p13, layer.p2, layer.d, buf, routing=r)
    torch.cuda.synchronize()
    assert int(buf.union_size.item()) == -1
    assert bool((buf.y_perm == 123.0).all())
