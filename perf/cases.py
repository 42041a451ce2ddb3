"""The workloads by which this framework's speed is measured.

A case is one of two kinds:

* ``"layer"``: a stack of MoE layers of one shape, each run by ``moe_layer`` or
  ``moe_layer_mxfp4`` on its own weights: a decode step, or a prefill chunk.
  A decode step (up to 256 tokens) holds several layers and is replayed from a
  HIP graph, as a serving loop holds it, so that a layer's weights come from
  HBM and not from a cache; a prefill chunk is one layer called eagerly.
* ``"signature"``: the expert-signature cache of a prefill forward: the blocks
  handed to new requests are zeroed, the forward's picks are added, and the
  requests' counts are read back.

The batch is routed by the gate, by a fixed random subset of U experts
(``"controlled"``), or by domain-clustered picks (``"domain"``: every token of
a run of consecutive ones prefers its domain's experts, by Zipf popularity).
"""
from __future__ import annotations

import dataclasses
import math

import numpy as np
import torch

from paper_2607_00466_amd import binding as B
from paper_2607_00466_amd import synth

QWEN = dict(shape="qwen3_30b_a3b", E=128, K=8, H=2048, I=768)
GPT_OSS = dict(shape="gpt_oss_120b", E=128, K=4, H=2880, I=2880)
TINY = dict(shape="tiny", E=16, K=2, H=256, I=128)

REPLAY_TOKENS = 256  # the largest batch whose step is replayed from a graph
SIG_BLOCK = 16       # tokens a KV block holds
MAX_FLOPS = 2048 * 4 * 6 * 2880 * 2880  # the largest listed case's expert products


def _layer(name, shape, T, fmt="bf16", routing="gate", U=0, run=1, layers=1, replay=True, path="routed"):
    return dict(name=name, kind="layer", **shape, T=T, fmt=fmt, routing=routing, U=U, run=run,
                layers=layers, replay=replay, path=path)


def listed():
    return [
        # the smallest shape, called eagerly with a ragged batch: launches and host work only
        _layer("tiny T=13 eager", TINY, 13, replay=False),
        # one user's decode step: the latency of a single token
        _layer("qwen3 decode T=1", QWEN, 1, layers=4),
        # a lightly loaded decode worker
        _layer("qwen3 decode T=12", QWEN, 12, layers=4),
        # the headline layer: a full decode batch, all experts but one or two active
        _layer("qwen3 decode T=64", QWEN, 64, layers=4),
        # a decode batch that locality routing has confined to 32 experts
        _layer("qwen3 decode T=64 U=32", QWEN, 64, routing="controlled", U=32, layers=4),
        # a large same-domain decode batch: skewed buckets
        _layer("qwen3 decode T=200 domain", QWEN, 200, routing="domain", run=200, layers=4),
        # a prefill chunk of mixed prompts
        _layer("qwen3 prefill T=1000", QWEN, 1000, replay=False),
        # the largest batch: a long prefill of a few prompts, each of one domain
        _layer("qwen3 prefill T=4096", QWEN, 4096, routing="domain", run=1024, replay=False),
        # MXFP4 experts: a decode batch, a large one, and a prefill chunk
        _layer("gpt-oss mxfp4 decode T=32", GPT_OSS, 32, fmt="mxfp4", layers=2),
        _layer("gpt-oss mxfp4 decode T=256", GPT_OSS, 256, fmt="mxfp4", layers=2),
        _layer("gpt-oss mxfp4 prefill T=2048", GPT_OSS, 2048, fmt="mxfp4", replay=False),
        # the signature cache over one prefill forward of 2048 tokens
        dict(name="signature T=2048", kind="signature", E=128, K=8, L=48, T=2048, requests=8),
    ]


def _log_int(rng, lo, hi):
    return min(hi, int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))


def draw(rng):
    if rng.random() < 0.08:
        return dict(kind="signature", E=4 * rng.randint(4, 64), K=rng.randint(1, 8), L=rng.randint(4, 64),
                    T=_log_int(rng, 16, 2048), requests=rng.randint(1, 8))
    pick = rng.random()
    if pick < 0.40:
        shape, fmt = dict(QWEN), "bf16"
    elif pick < 0.65:
        shape, fmt = dict(GPT_OSS), "mxfp4"
    elif pick < 0.72:
        shape, fmt = dict(GPT_OSS), "bf16"
    elif pick < 0.80:
        shape, fmt = dict(TINY), rng.choice(["bf16", "mxfp4"])
    else:  # a generic shape, ragged against every tile
        fmt = rng.choice(["bf16", "mxfp4"])
        step = 32 if fmt == "bf16" else 64
        E = rng.randint(8, 256)
        shape = dict(shape="generic", E=E, K=rng.randint(1, 8), H=step * _log_int(rng, 256 // step, 4096 // step),
                     I=step * _log_int(rng, 128 // step, 3072 // step))
        while E * shape["H"] * shape["I"] > 128 * 2880 * 2880:
            shape["I"] = max(step, shape["I"] // (2 * step) * step)
    E, K = shape["E"], shape["K"]
    expert = 3 * shape["H"] * shape["I"] * (2.0 if fmt == "bf16" else 17 / 32)
    # the largest batch that the buckets take and that costs no more than the largest listed case
    top = min(4096, 32 * (16384 // E), int(MAX_FLOPS // (6 * K * shape["H"] * shape["I"])))
    T = _log_int(rng, 1, top)
    routing = rng.choice(["gate", "gate", "domain", "controlled"])
    U = rng.randint(K, E) if routing == "controlled" else 0
    run = 1
    if routing == "domain":
        run = rng.choice([1, T]) if T <= REPLAY_TOKENS else rng.choice([256, 1024])
    replay = T <= REPLAY_TOKENS and rng.random() < 0.85
    layers = max(1, min(16, int(4.5e9 // (E * expert)))) if replay else 1
    path = rng.choice(["routed", "routed", "routed", "routed", "split", "fused"])
    case = _layer("", shape, T, fmt, routing, U, run, layers, replay, path)
    case.pop("name")
    return case


# ----------------------------------------------------------------------------- inputs

def _shape(case):
    return synth.LayerShape(case["shape"], E=case["E"], K=case["K"], H=case["H"], I=case["I"])


def _domains(case):
    return synth.DomainModel(E=case["E"], K=case["K"], subset_size=max(case["K"], min(32, case["E"] // 4)))


def _routing(case, seed, layer):
    """The layer's (ids, weights) on the host, or None where the gate routes."""
    T, E, K = case["T"], case["E"], case["K"]
    if case["routing"] == "gate":
        return None
    if case["routing"] == "controlled":
        ids, w, _ = synth.controlled_routing(T, E, K, case["U"], seed, layer)
        return ids, w
    model = _domains(case)
    subsets = synth.domain_subsets(model, 1, seed + layer)
    run = min(case["run"], T)
    n = -(-T // run)
    rng = np.random.default_rng([seed, layer])
    ids = synth.domain_requests(model, subsets, np.arange(n) % model.n_domains if n > 1 else
                                rng.integers(0, model.n_domains, 1), run, seed + layer)[0]
    return np.ascontiguousarray(ids.reshape(n * run, K)[:T]), synth.dirichlet_weights(T, K, rng)


def _inputs(case, seed, layer):
    """x, gate weights, routing and unpacked expert weights of one layer, on the GPU."""
    s = _shape(case)
    x = torch.from_numpy(synth.hidden_states(case["T"], s.H, seed, layer)).cuda()
    wg = torch.from_numpy(synth.gate_weights(s, seed, layer)).cuda()
    routing = _routing(case, seed, layer)
    if routing is not None:
        routing = tuple(torch.from_numpy(a).cuda() for a in routing)
    if case["fmt"] == "mxfp4":
        w = synth.mxfp4_expert_weights(s, seed, layer, device="cuda")
        w = (w["w1"], w["w3"], w["w2"])
    else:
        w = synth.expert_weights(s, seed, layer, device="cuda")
    return x, wg, routing, w


def _signature_inputs(case, seed):
    """Picks of a forward, the block of each token, and the requests' block tables."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    L, T, K, E, R = (case[k] for k in ("L", "T", "K", "E", "requests"))
    heat = -1.2 * torch.log(1 + torch.argsort(torch.rand((L, 1, E), generator=gen, device="cuda"), -1).float())
    keys = heat - torch.log(-torch.log(torch.rand((L, T, E), generator=gen, device="cuda").clamp(1e-7, 1 - 1e-7)))
    ids = torch.topk(keys, K, dim=-1).indices.to(torch.int32).contiguous()
    # each request's new tokens fill blocks of its own, after a prefix of blocks cached before
    per = [T // R + (r < T % R) for r in range(R)]
    new = [-(-n // SIG_BLOCK) for n in per]
    prefix = [max(1, n // 2) for n in new]
    total = sum(new) + sum(prefix)
    order = torch.randperm(total, generator=gen, device="cuda").to(torch.int32).cpu().numpy()
    sig = torch.randint(0, 4, (total, L, E), generator=gen, device="cuda", dtype=torch.int8)
    table = np.full((R, max(a + b for a, b in zip(new, prefix))), -1, np.int32)
    token_block, fresh, at = [], [], 0
    for r in range(R):
        own = order[at:at + prefix[r] + new[r]]
        at += len(own)
        table[r, :len(own)] = own
        fresh.append(own[prefix[r]:])
        token_block.append(own[prefix[r] + np.arange(per[r]) // SIG_BLOCK])
    put = lambda a: torch.from_numpy(np.ascontiguousarray(a, np.int32)).cuda()  # noqa: E731
    return dict(ids=ids, sig=sig, token_block=put(np.concatenate(token_block)), fresh=put(np.concatenate(fresh)),
                table=put(table), n_blocks=put(np.add(new, prefix)))


# ----------------------------------------------------------------------------- the passes

def _layers(state):
    for x, wg, w, routing, buf in state["layers"]:
        state["call"](x, wg, *w, state["d"], buf, routing=routing, path=state["path"])


def prepare(case, seed):
    if case["kind"] == "signature":
        state = _signature_inputs(case, seed)
        state["counts"] = torch.empty((case["requests"], case["L"], case["E"]), dtype=torch.int32, device="cuda")
        state["kind"] = "signature"
        return state
    d = B.dims(case["T"], case["H"], case["E"], case["K"], case["I"])
    mx = case["fmt"] == "mxfp4"
    shared = B.LayerBuffers.allocate(d)  # one set of scratch buffers for the stack, results of each layer apart
    state = dict(kind="layer", d=d, path=case["path"], call=B.moe_layer_mxfp4 if mx else B.moe_layer, layers=[],
                 outputs=[], graph=None)
    for layer in range(case["layers"]):
        x, wg, routing, w = _inputs(case, seed, layer)
        w = B.pack_mxfp4_expert_weights(*w) if mx else B.pack_expert_weights(*w)
        buf = dataclasses.replace(shared, out=torch.empty_like(shared.out), topk_ids=torch.empty_like(shared.topk_ids),
                                  topk_w=torch.empty_like(shared.topk_w))
        state["layers"].append((x, wg, w, routing, buf))
        out = dict(out=buf.out)
        if routing is None:
            out.update(ids=buf.topk_ids, weights=buf.topk_w)
        state["outputs"].append(out)
    if case["replay"]:
        _layers(state)
        torch.cuda.synchronize()
        state["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(state["graph"]):
            _layers(state)
    return state


def run(state):
    if state["kind"] == "signature":
        L, E = state["sig"].shape[1:]
        B.moe_sig_reset(state["fresh"], state["sig"])
        B.moe_sig_capture(state["ids"], state["token_block"], 0, L, E, state["sig"])
        B.moe_sig_request_counts(state["sig"], state["table"], state["n_blocks"], out=state["counts"])
        return dict(sig=state["sig"], counts=state["counts"])
    if state["graph"] is not None:
        state["graph"].replay()
    else:
        _layers(state)
    return state["outputs"]


# ----------------------------------------------------------------------------- what a pass needs

def _union(case):
    """Expected distinct experts of one layer's batch."""
    T, E, K = case["T"], case["E"], case["K"]
    if case["routing"] == "controlled":
        return case["U"] * (1 - (1 - K / case["U"]) ** T)
    if case["routing"] == "gate":
        return E * (1 - (1 - K / E) ** T)
    model = _domains(case)
    subsets = synth.domain_subsets(model, 1, 0)
    run = min(case["run"], T)
    miss = np.ones(E)
    for r in range(-(-T // run)):
        miss *= (1 - synth.domain_pick_probs(model, subsets, r % model.n_domains, 0)) ** (K * min(run, T - r * run))
    return float(E - miss.sum())


def work(case):
    T, E, K = case["T"], case["E"], case["K"]
    if case["kind"] == "signature":
        row = case["L"] * E
        blocks = -(-T // SIG_BLOCK)
        # picks in; new rows written; prefix and new rows read; counts out
        return dict(bytes=4 * case["L"] * T * K + blocks * row + 1.5 * blocks * row + 4 * case["requests"] * row,
                    flops=0)
    H, I = case["H"], case["I"]
    expert = 3 * H * I * (2.0 if case["fmt"] == "bf16" else 17 / 32)
    gate = case["routing"] == "gate"
    bytes_ = _union(case) * expert + 2 * 4 * T * H + 8 * T * K + (4 * E * H if gate else 0)
    flops = 6 * T * K * H * I + (2 * T * E * H if gate else 0) + 2 * T * K * H
    return dict(bytes=case["layers"] * bytes_, flops=case["layers"] * flops)


def tolerance(case):
    if case["kind"] == "signature":
        return "exact"
    # Activations enter the products with about 16 significant bits and the
    # sums are 32-bit: up to 5e-6 was seen against 64 bits.  A token whose
    # last pick is a near tie may take the other expert.
    return dict(rel=2e-5, max=1e-3, differ=1e-3)


# ----------------------------------------------------------------------------- the same in 64 bits

_E2M1 = (0.0, 0.5, 1.0, 1.5, 2.0, 3.0, 4.0, 6.0)


def _dense(w, e):
    """Expert e's matrix in 64 bits (bf16, or MXFP4 codes and scales)."""
    if isinstance(w, torch.Tensor):
        return w[e].double()
    codes, scales = w[0][e].long(), w[1][e]
    nib = torch.stack((codes & 15, codes >> 4), -1).flatten(1)
    mag = torch.tensor(_E2M1, dtype=torch.float64, device=codes.device)[nib & 7]
    scale = torch.exp2(scales.double() - 127).repeat_interleave(32, 1)
    return torch.where(nib >= 8, -mag, mag) * scale


def exact(case, seed):
    if case["kind"] == "signature":
        s = _signature_inputs(case, seed)
        L, T, K = s["ids"].shape
        sig = s["sig"].long()
        sig[s["fresh"].long()] = 0
        layer = torch.arange(L, device="cuda")[:, None, None].expand(L, T, K)
        block = s["token_block"].long()[None, :, None].expand(L, T, K)
        sig.index_put_((block, layer, s["ids"].long()), torch.ones((), dtype=torch.int64, device="cuda"), accumulate=True)
        rows = [s["table"][r, :n].long() for r, n in enumerate(s["n_blocks"].tolist())]
        return dict(sig=sig.to(torch.int8), counts=torch.stack([sig[r].sum(0) for r in rows]).to(torch.int32))
    outputs = []
    for l in range(case["layers"]):
        x, wg, routing, (w1, w3, w2) = _inputs(case, seed, l)
        x = x.double()
        got = {}
        if routing is None:
            logits, ids = torch.sort(x @ wg.double().T, dim=-1, descending=True, stable=True)
            ids, w = ids[:, :case["K"]], torch.softmax(logits[:, :case["K"]], -1)
            got = dict(ids=ids.to(torch.int32), weights=w)
        else:
            ids, w = routing[0].long(), routing[1].double()
        out = torch.zeros_like(x)
        for e in torch.unique(ids).tolist():
            t, j = torch.nonzero(ids == e, as_tuple=True)
            a, b = x[t] @ _dense(w1, e).T, x[t] @ _dense(w3, e).T
            out[t] += ((a * torch.sigmoid(a) * b) @ _dense(w2, e).T) * w[t, j, None]
        got["out"] = out
        outputs.append(got)
    return outputs
