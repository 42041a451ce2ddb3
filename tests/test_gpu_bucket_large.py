"""moe_bucket at the edges of its launch rules: one or several workgroups
(2048 pairs each, up to 16), one or several threads an expert (256 tokens and
3072 pairs; 64 and 128 experts), bitmaps above and below 64 KiB of either, a
partial last bitmap word, and invalid routing that another
workgroup's stretch of the pairs holds."""
import numpy as np
import pytest
import torch

from paper_2607_00466_amd import binding as B
from tests import gpu_util as G

pytestmark = pytest.mark.gpu


def _bucket(ids, E, in_place=False):
    T, K = ids.shape
    d = B.dims(T, 64, E, K, 32)
    buf = B.LayerBuffers.allocate(d)
    for t in (buf.counts, buf.offsets, buf.perm_token, buf.pair_pos, buf.union_ids, buf.union_size):
        t.fill_(-7)
    dev = torch.from_numpy(np.ascontiguousarray(ids, np.int32)).cuda()
    if in_place:
        buf.pair_pos = dev.view(-1)
    B.moe_bucket(dev, d, buf.counts, buf.offsets,
                 buf.perm_token, buf.pair_pos, buf.union_ids, buf.union_size)
    torch.cuda.synchronize()
    return G.fetch(buf, d)


@pytest.mark.parametrize("T,E,K", [(256, 9, 8), (257, 9, 8), (257, 16, 1), (2049, 64, 1), (1000, 65, 5),
                                   (1025, 129, 16), (4095, 128, 8), (4096, 37, 16), (300, 1, 1),
                                   (384, 128, 8), (385, 128, 8), (768, 256, 4), (3072, 170, 1), (3073, 168, 1)])
def test_bucket_launch_rules(T, E, K):
    G.say(f"case: bucket only, T={T} E={E} K={K}")
    rng = np.random.default_rng(T + E + K)
    # half the tokens from a few experts, so that bitmap words are full and empty
    few = min(E, K + 2)
    ids = np.stack([rng.choice(few if t % 2 else E, K, replace=False) for t in range(T)]).astype(np.int32)
    G.compare_buckets(_bucket(ids, E), ids.astype(np.int64), E)


@pytest.mark.parametrize("T,E,K", [(64, 16, 4), (256, 9, 8), (300, 40, 8), (4096, 37, 16)])
def test_bucket_in_place(T, E, K):
    # pair_pos written over topk_ids, in batches of one workgroup's pairs and of more
    G.say(f"case: bucket only, in place, T={T} E={E} K={K}")
    ids = np.stack([np.random.default_rng(t).choice(E, K, replace=False) for t in range(T)]).astype(np.int32)
    G.compare_buckets(_bucket(ids, E, in_place=True), ids.astype(np.int64), E)


@pytest.mark.parametrize("where", [0, 1, -1])
@pytest.mark.parametrize("kind", ["repeated", "too large", "negative"])
def test_bucket_invalid_in_any_stretch(where, kind):
    T, E, K = 1500, 40, 8  # 12000 pairs: 6 workgroups
    G.say(f"case: bucket only, T={T} E={E} K={K}, {kind} pick in token {where}")
    ids = np.stack([np.random.default_rng(t).choice(E, K, replace=False) for t in range(T)]).astype(np.int32)
    ids[where, 3] = {"repeated": ids[where, 2], "too large": E, "negative": -1}[kind]
    assert _bucket(ids, E)["union_size"] == -1
