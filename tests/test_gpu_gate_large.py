"""Gate scores of batches on both sides of the tile switches (128 and 256
tokens; gate rows of more than 4 MiB), with partial expert and token tiles,
reductions of less than one position a lane and of several, and a last XCD
round with few token tiles: against the oracle, and the same bits as in batches of 4 x 4 tiles."""
import numpy as np
import pytest
import torch

from paper_2607_00466_amd import synth
from tests import gpu_util as G
from tests.test_gpu_parity import _gate

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,E,K,H", [(129, 13, 4, 1056), (256, 9, 2, 32), (257, 13, 4, 2880), (263, 256, 16, 96),
                                     (321, 1, 1, 4160), (1025, 60, 3, 544),
                                     (258, 256, 8, 4128), (265, 129, 5, 8192)])
def test_gate_tiles_and_reductions(T, E, K, H):
    G.say(f"case: gate only, T={T} E={E} top-{K} H={H}")
    sh = synth.LayerShape("gate", E=E, K=K, H=H, I=32)
    x = synth.hidden_states(T, H, seed=T)
    wg_np = synth.gate_weights(sh, seed=E)
    wg = torch.from_numpy(wg_np).cuda()
    logits, ids, w = _gate(x, wg, sh)
    G.check_gate({"logits": logits, "ids": ids, "weights": w}, x, wg_np, K)
    for t0 in range(0, T, 128):
        part = _gate(x[t0:t0 + 128], wg, sh)
        assert np.array_equal(logits[t0:t0 + 128], part[0]), f"logits of tokens {t0} .."
        assert np.array_equal(ids[t0:t0 + 128], part[1]) and np.array_equal(w[t0:t0 + 128], part[2])
