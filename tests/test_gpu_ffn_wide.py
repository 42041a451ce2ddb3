"""The expert FFN's large-bucket kernel at the edges of its tiles.

The batches are ones that kernel takes (248 experts, so enough items, and
buckets that average over 32 tokens), with buckets set on both sides of
every pass shape (16, 32, 64 and 128 tokens), of the guarded last tiles (65,
80, 96, 97 tokens) and of the cut into equal token groups (129, 144, 257,
400).  Shapes: rows that fill half an item, an odd number of 32-row slots, a
last item of a single wave, and reductions of 1 to 18 steps, most of them no
multiple of a chunk of 2, 4 or 8.
"""
import numpy as np
import pytest
import torch

from paper_2607_00466_amd import binding as B
from paper_2607_00466_amd import synth
from tests import gpu_util as G
from tests import test_gpu_mxfp4 as MX
from tests import test_gpu_parity as P

pytestmark = pytest.mark.gpu

COUNTS = [400, 257, 144, 129, 128, 113, 97, 96, 81, 80, 65, 64, 49, 48, 33, 32, 31, 17, 16, 15, 1]


def _run(layer, T, ids, w, path="routed"):
    d = B.dims(T, layer.shape.H, layer.shape.E, layer.shape.K, layer.shape.I)
    buf = B.LayerBuffers.allocate(d)
    buf.y_perm.fill_(float("nan"))
    r = (torch.from_numpy(np.ascontiguousarray(ids[:T], np.int32)).cuda(),
         torch.from_numpy(np.ascontiguousarray(w[:T], np.float32)).cuda())
    x = layer.x[:T].contiguous()
    if isinstance(layer, G.Layer):
        B.moe_layer(x, layer.wg, layer.p13, layer.p2, d, buf, routing=r, path=path)
    else:
        B.moe_layer_mxfp4(x, layer.wg, layer.up, layer.down, d, buf, routing=r, path=path)
    torch.cuda.synchronize()
    return G.fetch(buf, d)


@pytest.mark.parametrize("fmt,H,I", [("bf16", 352, 288), ("bf16", 288, 32), ("bf16", 64, 416),
                                     ("mxfp4", 320, 192), ("mxfp4", 64, 448), ("mxfp4", 576, 64)])
def test_bucket_sizes_around_every_tile(fmt, H, I):
    E, K, T = 248, 4, 2080  # 33.5 tokens an expert, 313 items a row band
    G.say(f"case: {fmt} E={E} top-{K} H={H} I={I} T={T}, buckets {COUNTS}")
    rng = np.random.default_rng(H + I)
    # one pick of most tokens fills the listed buckets in turn, the others spread over the rest
    heavy = np.repeat(np.arange(len(COUNTS)), COUNTS)
    ids = np.stack([len(COUNTS) + rng.choice(E - len(COUNTS), K, replace=False) for _ in range(T)]).astype(np.int32)
    ids[:heavy.size, 0] = heavy
    ids = np.take_along_axis(ids, rng.permuted(np.tile(np.arange(K), (T, 1)), axis=1), 1)
    w = rng.dirichlet(np.ones(K), size=T).astype(np.float32)
    sh = synth.LayerShape(f"wide_{fmt}", E=E, K=K, H=H, I=I)
    layer = G.Layer(sh, T, seed=I) if fmt == "bf16" else MX.MxLayer(sh, T, seed=I)
    g = _run(layer, T, ids, w)
    assert g["counts"][:len(COUNTS)].tolist() == COUNTS
    if fmt == "bf16":
        P._full_check(layer, g, False, routing=(ids.astype(np.int64), w))
    else:
        MX._check_layer(layer, g, (ids, w))
    # the same bits as in a batch that the small-batch kernel runs
    for n in (40, 64):
        part = _run(layer, n, ids, w)
        assert np.array_equal(g["out"][:n], part["out"]), f"first {n} tokens differ"


@pytest.mark.parametrize("fmt,H,I", [("bf16", 352, 288), ("bf16", 288, 32), ("mxfp4", 320, 192)])
def test_few_active_experts_take_smaller_groups(fmt, H, I):
    # 4 experts hold every token: 17 groups of 128 tokens each make 204 items of
    # 3 row bands (cut to 64 tokens), or 68 of one (cut to 32), for 256 CUs.
    E, K, T = 248, 4, 2080
    G.say(f"case: {fmt} E={E} top-{K} H={H} I={I} T={T}, 4 experts active")
    sh = synth.LayerShape(f"few_{fmt}", E=E, K=K, H=H, I=I)
    layer = G.Layer(sh, T, seed=I) if fmt == "bf16" else MX.MxLayer(sh, T, seed=I)
    ids, w, _ = synth.controlled_routing(T, E, K, U=4, seed=I)
    g = _run(layer, T, ids, w)
    if fmt == "bf16":
        P._full_check(layer, g, False, routing=(ids.astype(np.int64), w))
    else:
        MX._check_layer(layer, g, (ids, w))
