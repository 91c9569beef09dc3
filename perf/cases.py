"""The work this library is used for, as cases that can be timed and checked.

A pass is one MoE layer as a serving or training program issues it: lay out the routing, send the
token rows to their experts' receive rows, and (given the experts' output rows) gather them back
into token order. The listed cases run from a toy layer and a few decoding tokens, where launches
count, over decode batches of the model shapes that the paper evaluates, to prefill. ``draw`` gives
more cases of the same ranges.

Fields of a case:

* ``path``     ``layer`` (layout, dispatch, combine), ``scheduled`` (the hierarchical schedule and the
               dispatch in its order, then combine), ``decomposed`` (layout and dispatch in one launch,
               then combine) or ``one_launch`` (the whole layer, identity experts, in one launch);
* ``calls``    how ``layer`` is issued: ``prepared`` (a serving loop that checked its arguments once),
               ``fused`` (layout_dispatch, combine) or ``separate`` (layout, dispatch, combine);
* ``sync``     what synchronises the combine of ``one_launch``: ``sentinel``, ``flag`` or ``checksum``;
* ``workers``  workers per source rank of ``scheduled``;
* ``R, E, k, Tr, H``  ranks, experts, choices per token, tokens per rank, hidden size;
* ``payload``  format of the dispatched rows, ``bf16`` or ``fp8``;
* ``routing``  ``uniform``, ``zipf_group`` (skewed popularity, group-limited) or ``hot_group``;
* ``pad``      tokens at the end of each rank's batch that are padding (expert id -1).
"""
from __future__ import annotations

import math

import torch

from paper_2607_06202_amd import epl
from paper_2607_06202_amd import workloads as W


def _case(name, path, R, E, k, Tr, H, payload="bf16", routing="uniform", pad=0, calls="fused", sync="", workers=0):
    c = dict(path=path, calls=calls, sync=sync, workers=workers, R=R, E=E, k=k, Tr=Tr, H=H, payload=payload,
             routing=routing, pad=pad)
    return dict(c, name=name) if name else c


def _named(name, w, path="layer", **more):
    w = W.WORKLOADS[w]
    return _case(name, path, w.R, w.E, w.k, w.Tr, w.H, w.payload, w.routing, **more)


def listed():
    return [
        # The smallest layer of the tests and the smoke run: launches and latency are all of it.
        _named("tiny", "tiny", calls="prepared"),
        # A few sequences decoding on the Qwen3-30B shape: 8 tokens on each of 16 ranks.
        _case("qwen3_decode_bs8", "layer", 16, 128, 8, 8, 2048, calls="prepared"),
        # A small GLM-4.7 batch of odd size whose last rows are padding (a captured batch not full).
        _case("glm47_ragged_padded", "layer", 32, 160, 8, 37, 5120, pad=5),
        # The Qwen3-30B shape at its decode batch.
        _named("qwen3_30b_ep16", "qwen3_30b_ep16", calls="prepared"),
        # The same shape as one launch, the combine polling the rows (Sentinel Polling).
        _named("qwen3_30b_sentinel", "qwen3_30b_ep16", path="one_launch", sync="sentinel"),
        # The headline: DeepSeek decode on 64 ranks.
        _named("decode_ep64", "decode_ep64", calls="prepared"),
        # The same layer with layout and dispatch in one launch (Kernel Decomposition).
        _named("decode_ep64_decomposed", "decode_ep64", path="decomposed"),
        # The paper's default ablation setting, dispatched in the hierarchical schedule's order.
        _named("deepseek_ep128_scheduled", "deepseek_ep128_bs64", path="scheduled", workers=64),
        # One expert per rank on 256 ranks with a hot group of experts.
        _named("large_ep256", "large_ep256"),
        # Skewed routing, rows quantised to fp8 as they are sent.
        _named("skewed_fp8_ep64", "skewed_fp8_ep64"),
        # An fp8 prefill on few ranks with a ragged number of tokens, as three separate calls.
        _case("prefill_fp8_ep8_ragged", "layer", 8, 256, 8, 2039, 7168, "fp8", calls="separate"),
        # Prefill on 32 ranks: the largest layer.
        _named("prefill_ep32", "prefill_ep32"),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    path = rng.choice(["layer"] * 7 + ["scheduled", "decomposed", "one_launch"])
    R = rng.choice([4, 8, 16, 32, 64, 128, 256])
    El = rng.choice([n for n in (1, 2, 3, 4, 5, 8, 16, 32) if 16 <= n * R <= 256] or [4])
    E = R * El
    k = rng.choice([1, 2, 4, 6, 8, 8, 8, 10, 16])
    k = min(k, E)
    payload = rng.choice(["bf16", "bf16", "fp8"]) if path in ("layer", "scheduled") else "bf16"
    step = 128 if payload == "fp8" else rng.choice([8, 64, 128])
    H = max(step, _log_uniform(rng, 256, 7168) // step * step)
    most = 1 << 20 if path == "layer" else 1 << 16  # pairs
    tokens = min(most // k, (7168 << 20) // (k * H))
    if path != "layer":
        tokens = min(tokens, 256 * (256 // k))  # what the one-launch calls take
    Tr = _log_uniform(rng, 1, max(1, min(4096, tokens // R)))
    routing = rng.choice(["uniform", "zipf_group", "hot_group"])
    groups = 16 if routing == "hot_group" else 8
    if (R if routing == "zipf_group" else E) % groups or (E // groups if routing == "hot_group" else E // 2) < k:
        routing = "uniform"
    pad = rng.randrange(Tr) // 4 if rng.random() < 0.3 else 0
    return _case("", path, R, E, k, Tr, H, payload, routing, pad,
                 calls=rng.choice(["prepared", "fused", "separate"]) if path == "layer" else "fused",
                 sync=rng.choice(["sentinel", "flag", "checksum"]) if path == "one_launch" else "",
                 workers=rng.choice([16, 32, 48, 64, 128]) if path == "scheduled" else 0)


# ------------------------------------------------------------------------------------ inputs
def _gumbel(shape, g, dev):
    u = torch.rand(shape, generator=g, device=dev, dtype=torch.float32).clamp_(1e-12, 1 - 1e-7)
    return -torch.log(-torch.log(u))


def _routing(c, g, dev):
    """[T, k] int32 expert ids, distinct per token; the last ``pad`` tokens of each rank get -1."""
    R, E, k, Tr = c["R"], c["E"], c["k"], c["Tr"]
    T = R * Tr
    ids = torch.empty(T, k, dtype=torch.int32, device=dev)
    logp = torch.zeros(E, device=dev)
    if c["routing"] == "zipf_group":  # popularity (rank + 1)^-1.2; each token draws 4 of 8 rank groups
        order = torch.randperm(E, generator=g, device=dev)
        logp = -1.2 * torch.log(order.float() + 1)
        group = (torch.arange(E, device=dev) // (E // R)) // (R // 8)
        mass = torch.log(torch.zeros(8, device=dev).index_add_(0, group, logp.exp()))
    elif c["routing"] == "hot_group":  # a fifth of the tokens go to one sixteenth of the experts
        per = E // 16
        hot = torch.randint(16, (1,), generator=g, device=dev)
        in_hot = torch.arange(E, device=dev) // per == hot
    for t0 in range(0, T, 1 << 15):
        n = min(T, t0 + (1 << 15)) - t0
        key = _gumbel((n, E), g, dev) + logp
        if c["routing"] == "zipf_group":
            top = (mass + _gumbel((n, 8), g, dev)).topk(4, dim=1).indices
            allowed = torch.zeros(n, 8, dtype=torch.bool, device=dev).scatter_(1, top, True)
            key = torch.where(allowed[:, group], key, key - 1e6)
        elif c["routing"] == "hot_group":
            is_hot = torch.rand(n, 1, generator=g, device=dev) < 0.2
            key = torch.where(is_hot & ~in_hot, key - 1e6, key)
        ids[t0:t0 + n] = key.topk(k, dim=1).indices.to(torch.int32)
    if c["pad"]:
        ids.view(R, Tr, k)[:, Tr - c["pad"]:] = -1
    return ids


def _normal(shape, g, dev):
    return torch.randn(shape, generator=g, device=dev, dtype=torch.bfloat16)


def _inputs(c, seed):
    dev = torch.device("cuda", torch.cuda.current_device())
    g = torch.Generator(device=dev)
    g.manual_seed(int(seed))
    cfg = epl.config(c["R"], c["E"], c["k"], c["H"], c["Tr"], c["payload"],
                     row_pitch=epl.tuned_pitch(c["H"], c["payload"]))
    T = cfg.T
    idx = _routing(c, g, dev)
    # Activations: N(0, 1) with one channel in 64 sixteen times as large, as hidden states have.
    x = _normal((T, c["H"]), g, dev)
    x[:, ::64] *= 16
    topk_w = torch.softmax(torch.randn(T, c["k"], generator=g, device=dev), dim=1)
    y = None
    if c["path"] != "one_launch":  # the experts' output rows, at the receive layout's pitch
        y = _normal((max(T * c["k"], 1), cfg.pitch), g, dev)[:, :c["H"]]
    return dev, cfg, idx, x, topk_w, y


def prepare(case, seed):
    c = case
    dev, cfg, idx, x, topk_w, y = _inputs(c, seed)
    L = epl.alloc_layout(cfg, dev)
    L.recv_src.fill_(-1)  # rows past the valid pairs are never written
    L.recv_j.fill_(-1)
    recv, scale = epl.alloc_recv(cfg, dev)
    out = torch.empty(cfg.T, c["H"], dtype=torch.bfloat16, device=dev)
    s = dict(case=c, cfg=cfg, idx=idx, x=x, w=topk_w, y=y, L=L, recv=recv, scale=scale, out=out)
    if c["path"] == "one_launch":
        epl.sentinel_fill(recv)
        s["status"] = torch.empty(1, dtype=torch.int32, device=dev)
        s["marks"] = epl.alloc_marks(cfg, dev) if c["sync"] != "sentinel" else None
        s["epoch"] = 0
    else:
        recv.zero_()
        if scale is not None:
            scale.zero_()
    if c["path"] == "decomposed":
        s["status"] = torch.empty(1, dtype=torch.int32, device=dev)
    if c["path"] == "scheduled":
        s["hop"] = torch.from_numpy(W.node_hop_classes(c["R"])).to(dev)
    if c["path"] == "layer" and c["calls"] == "prepared":
        s["layer"] = epl.PreparedLayer(cfg, idx, [x], topk_w, L, recv, scale, y=y, out=out)
    return s


# ------------------------------------------------------------------------------------ one pass
_LAYOUT = ("send_cnt", "rank_cnt", "expert_off", "rank_off", "seg_off", "tok_nranks", "pair_row", "pair_rslot",
           "recv_src", "recv_j", "num_invalid")


def run(state):
    s = state
    c, cfg, L = s["case"], s["cfg"], s["L"]
    more = {}
    if c["path"] == "one_launch":
        if c["sync"] == "sentinel":
            epl.layer_sentinel(cfg, s["idx"], s["x"], s["w"], s["recv"], out=s["out"], layout_out=L,
                               status=s["status"])
        else:
            s["epoch"] += 1
            variant = epl.DAF_TOKEN_FLAG_FUSION if c["sync"] == "flag" else epl.DAF_DATA_CHECKSUM
            epl.layer_data_as_flag(cfg, s["idx"], s["x"], s["w"], s["recv"], s["marks"], variant, s["epoch"],
                                   out=s["out"], layout_out=L, status=s["status"])
        more["status"] = s["status"]
    elif c["path"] == "decomposed":
        epl.layout_dispatch_decomposed(cfg, s["idx"], s["x"], out=L, recv=s["recv"], status=s["status"])
        epl.combine(cfg, s["y"], s["w"], L, out=s["out"])
        more["status"] = s["status"]
    elif c["path"] == "scheduled":
        epl.layout(cfg, s["idx"], out=L)
        more["schedule"] = epl.hop_schedule(cfg, L.send_cnt, s["hop"], c["workers"], 2)
        epl.dispatch_scheduled(cfg, s["x"], L, c["workers"], recv=s["recv"], recv_scale=s["scale"])
        epl.combine(cfg, s["y"], s["w"], L, out=s["out"])
    elif c["calls"] == "prepared":
        s["layer"].run()
    elif c["calls"] == "fused":
        epl.layout_dispatch(cfg, s["idx"], s["x"], out=L, recv=s["recv"], recv_scale=s["scale"])
        epl.combine(cfg, s["y"], s["w"], L, out=s["out"])
    else:
        epl.layout(cfg, s["idx"], out=L)
        epl.dispatch(cfg, s["x"], L, s["recv"], s["scale"])
        epl.combine(cfg, s["y"], s["w"], L, out=s["out"])
    if c["path"] != "one_launch":  # whose receive rows are scratch
        more["recv"], more["scale"] = s["recv"], s["scale"]
    return dict(more, layout={n: getattr(L, n) for n in _LAYOUT}, out=s["out"])


# ------------------------------------------------------------------------------------ what it needs
def work(case):
    """Bytes: the ids, token rows, weights and expert rows read once; the layout, the receive rows
    (with their scales) and the output rows written once. Flops: the combine's multiply-adds."""
    c = case
    R, E, k, H = c["R"], c["E"], c["k"], c["H"]
    T = R * c["Tr"]
    P = R * (c["Tr"] - c["pad"]) * k
    row = 2 * H if c["payload"] == "bf16" else H + H // 128 * 4
    ids, weights, x, out = 4 * T * k, 4 * T * k, 2 * T * H, 2 * T * H
    layout = 4 * (2 * R * E + R * R + E + R + 3 + T + 2 * T * k + 2 * P)
    received = P * (2 * H if c["path"] == "one_launch" else row)
    return {"bytes": ids + weights + x + layout + received + 2 * P * H + out, "flops": 2 * P * H}


def tolerance(case):
    """The interface fixes every value bit by bit: rows are copies, a block's fp8 scale and quotients
    are single IEEE operations, and the combine is an fp32 fmaf chain in choice order rounded once."""
    return "exact"


def exact(case, seed):
    """The combined rows (and fp8 scales) in 64 bits; the other outputs are copies and whole numbers."""
    c = case
    dev, cfg, idx, x, topk_w, y = _inputs(c, seed)
    T, k, H = cfg.T, c["k"], c["H"]
    flat = idx.reshape(-1).long()
    valid = (flat >= 0) & (flat < c["E"])
    order = torch.sort(torch.where(valid, flat, c["E"]), stable=True).indices  # packed rows: by expert, then pair
    row = torch.empty_like(order)
    row[order] = torch.arange(T * k, device=dev)
    out = torch.empty(T, H, dtype=torch.float64, device=dev)
    for t0 in range(0, T, 4096):
        t1 = min(T, t0 + 4096)
        acc = torch.zeros(t1 - t0, H, dtype=torch.float64, device=dev)
        for j in range(k):
            p = torch.arange(t0, t1, device=dev) * k + j
            v = x[t0:t1] if y is None else y[row[p]]
            wj = torch.where(valid[p], topk_w[t0:t1, j].double(), 0.0)
            acc += wj[:, None] * v.double()
        out[t0:t1] = acc
    scale = None
    if c["payload"] == "fp8":
        block = x.view(T, H // 128, 128).abs().amax(dim=2).double() / 448
        scale = torch.zeros(T * k, H // 128, dtype=torch.float64, device=dev)
        n = int(valid.sum())
        scale[:n] = block[order[:n] // k]
    more = {}
    if c["path"] in ("one_launch", "decomposed"):
        more["status"] = None
    if c["path"] == "scheduled":
        more["schedule"] = None
    if c["path"] != "one_launch":
        more["recv"], more["scale"] = None, scale
    return dict(more, layout=None, out=out)
