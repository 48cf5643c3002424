"""Workloads whose speed is tracked: what a program that serves, profiles or
verifies an expert-parallel MoE layer asks of this library, from a handful of
decode tokens to a prefill of 16384.

Five kinds of call, all through the public entry points:

  layer    `MoELayer.forward`: gate -> dispatch -> expert FFN -> combine on one
           GPU's share of the experts (optionally followed by the routing
           history update between the previous layer and this one)
  receive  the receiving side of the first all-to-all: the segment table from
           the ranks' gathered counts, then the expert FFN over the segments
  router   the linear router with its top-k selection
  profile  one batch of a profiling run over two neighbouring layers: gates,
           per-expert counts, transition counts, and the two placement
           objectives of the maps in use

Shapes are those of `paper_2502_06643_amd.synth.config` (a Mixtral-8x7B-shaped
layer, a fine-grained 64-expert layer, a tiny fp32 layer) or generic.  Router
logits are N(0,1) plus a Zipf log-bias, the routing skew of those configurations.
"""
import math

import numpy as np
import torch

from paper_2502_06643_amd import binding as B
from paper_2502_06643_amd import synth
from paper_2502_06643_amd.layer import MoELayer

MIXTRAL = dict(d=4096, f=14336, E=8, k=2, zipf=1.0, dtype="bf16")
FINE = dict(d=2048, f=1408, E=64, k=6, zipf=1.2, dtype="bf16")


def _layer(T, shape, G=1, local_gpu=-1, history=False):
    return dict(kind="layer", T=T, G=G, local_gpu=local_gpu, history=history, **shape)


def listed():
    return [
        # a unit-test-sized fp32 layer, one of four expert-parallel ranks: next to no work, so launches and host time
        dict(name="layer_f32_256", **_layer(256, dict(d=128, f=256, E=8, k=2, zipf=1.2, dtype="f32"), G=4, local_gpu=0)),
        # an fp32 layer of a small model, all experts on the GPU: verification runs, training-time evaluation
        dict(name="layer_f32_1000", **_layer(1000, dict(d=1024, f=2816, E=8, k=2, zipf=1.0, dtype="f32"))),
        # decode with almost nobody in the batch: the touched experts' weights are all there is
        dict(name="decode_5", **_layer(5, MIXTRAL)),
        # an ordinary decode step
        dict(name="decode_64", **_layer(64, MIXTRAL)),
        # a chunk of a prefill mixed with decode tokens, ragged: neither weight-bound nor compute-bound
        dict(name="chunk_777", **_layer(777, MIXTRAL)),
        # prefill, the benchmark's workload and step (layer plus routing history)
        dict(name="prefill_4096", **_layer(4096, MIXTRAL, history=True)),
        # a long prefill batch, the largest configuration
        dict(name="prefill_16384", **_layer(16384, MIXTRAL)),
        # many small experts, 8 of 64 on this GPU: routing and data movement weigh as much as the FFN
        dict(name="fine_grained_8192", **_layer(8192, FINE, G=8, local_gpu=0)),
        # the receiving side of a 4-way expert-parallel layer, 1000 tokens on every rank
        dict(name="receive_ep4_1000", kind="receive", T=1000, G=4, local_gpu=1, **MIXTRAL),
        # the router in front of a layer, ragged batch, logits kept
        dict(name="router_10007", kind="router", T=10007, d=4096, E=8, k=2, dtype="bf16"),
        # a profiling batch of a million tokens over two 8-expert layers on 4 GPUs
        dict(name="profile_1m", kind="profile", T=1 << 20, E=8, k=2, G=4, zipf=1.0),
        # the same for the many-expert layer on 8 GPUs, ragged
        dict(name="profile_e64_100003", kind="profile", T=100003, E=64, k=6, G=8, zipf=1.2),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["mixtral", "mixtral", "generic", "f32", "receive", "router", "profile"])
    if kind == "mixtral":
        # the benchmark shape at any batch size, whole or a tensor-parallel share of it, all experts or one rank's
        G, local = rng.choice([(1, -1), (1, -1), (4, 0), (4, 1), (2, 1)])
        return _layer(_log_int(rng, 1, 16384), dict(MIXTRAL, f=rng.choice([14336, 14336, 7168, 3584])), G, local, rng.random() < 0.5)
    if kind == "generic":
        E = rng.choice([8, 16, 32, 64])
        k = rng.choice([1, 2, 4, 6])
        G = rng.choice([1, 2, 4, 8])
        return _layer(_log_int(rng, 1, 8192), dict(d=64 * _log_int(rng, 8, 64), f=64 * _log_int(rng, 8, 64), E=E, k=k, zipf=rng.choice([0.0, 0.6, 1.2]),
                                                   dtype="bf16"), G, -1 if G == 1 else rng.randrange(G), False)
    if kind == "f32":
        G = rng.choice([1, 4])
        return _layer(_log_int(rng, 1, 2048), dict(d=4 * _log_int(rng, 32, 256), f=4 * _log_int(rng, 32, 704), E=rng.choice([4, 8, 16]), k=rng.choice([1, 2]),
                                                   zipf=rng.choice([0.0, 1.0]), dtype="f32"), G, -1 if G == 1 else rng.randrange(G), False)
    if kind == "receive":
        G = rng.choice([2, 4, 8])
        shape = rng.choice([MIXTRAL, FINE])
        return dict(kind="receive", T=_log_int(rng, 8, 4096), G=G, local_gpu=rng.randrange(G), **shape)
    if kind == "router":
        E = rng.choice([8, 16, 64, 128])
        return dict(kind="router", T=_log_int(rng, 1, 65536), d=64 * _log_int(rng, 16, 64), E=E, k=rng.choice([1, 2, 4, 6]), dtype="bf16")
    E, k, G = rng.choice([(8, 2, 4), (16, 4, 4), (64, 6, 8), (128, 8, 16)])
    return dict(kind="profile", T=_log_int(rng, 1000, (1 << 22) // E), E=E, k=k, G=G, zipf=rng.choice([0.6, 1.0, 1.2]))


# ---- inputs -------------------------------------------------------------------
def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _normal(g, shape, sigma, dtype):
    t = torch.randn(shape, generator=g, device="cuda", dtype=torch.bfloat16 if dtype == "bf16" else torch.float32)
    return t.mul_(sigma) if sigma != 1.0 else t


def _logits(g, T, E, zipf):
    bias = torch.from_numpy(synth.zipf_log_bias(E, zipf).astype(np.float32)).cuda()
    return torch.randn((T, E), generator=g, device="cuda") + bias


def _placement(case):
    """One map per case: contiguous, or shuffled for the many-expert layers (as the configurations have it)."""
    if case["E"] >= 32:
        return synth.placement_balanced_random(case["E"], case["G"], 4000)
    return synth.placement_contiguous(case["E"], case["G"])


def _weights(g, case):
    E, d, f, dt = case["E"], case["d"], case["f"], case["dtype"]
    return _normal(g, (E, d, f), d ** -0.5, dt), _normal(g, (E, d, f), d ** -0.5, dt), _normal(g, (E, f, d), f ** -0.5, dt)


def _i32(*shape):
    return torch.empty(shape, dtype=torch.int32, device="cuda")


def prepare(case, seed):
    g = _gen(seed)
    T, E, k = case["T"], case["E"], case["k"]
    kind = case["kind"]
    if kind == "layer":
        L = MoELayer(T, case["d"], case["f"], E, k, case["G"], case["local_gpu"], case["dtype"])
        L.set_placement(_placement(case))
        L.set_weights(*_weights(g, case))
        s = dict(case=case, L=L, x=_normal(g, (T, case["d"]), 1.0, case["dtype"]), logits=_logits(g, T, E, case["zipf"]))
        if case["history"]:
            s["prev"] = _logits(g, T, E, 0.0).topk(k, dim=1).indices.to(torch.int32).contiguous()
            s["R"] = torch.zeros((E, E), dtype=torch.int64, device="cuda")
        return s
    if kind == "receive":
        # every rank's routing of its own tokens; this rank receives the rows of its experts, sorted per source
        G, dest, d, f = case["G"], case["local_gpu"], case["d"], case["f"]
        pl = _placement(case)
        counts = torch.stack([torch.bincount(_logits(g, T, E, case["zipf"]).topk(k, dim=1).indices.reshape(-1), minlength=E)
                              for _ in range(G)]).to(torch.int32).contiguous()
        mine = torch.from_numpy((pl == dest).astype(np.int32)).cuda()
        n = int((counts * mine).sum())
        cap = G * T * min(k, int((pl == dest).sum()))          # the buffers hold whatever the ranks may send
        dt = B.MOE_BF16
        packed = torch.empty(B.moe_packed_weights_bytes(E, d, f, dt), dtype=torch.uint8, device="cuda")
        w = _weights(g, case)
        B.moe_pack_weights(*w, E, d, f, dt, packed)
        n_seg = G * int((pl == dest).sum())
        return dict(case=case, n=n, n_seg=n_seg, counts=counts, pl=torch.from_numpy(pl).cuda(), packed=packed,
                    recv=_normal(g, (cap, d), 1.0, "bf16"), out=torch.zeros((cap, d), dtype=torch.bfloat16, device="cuda"),
                    seg=(_i32(n_seg), _i32(n_seg), _i32(n_seg)), src_offset=_i32(G + 1), n_seg_dev=_i32(1),
                    ws=torch.empty(B.moe_ffn_workspace_bytes(cap, d, f, E, dt), dtype=torch.uint8, device="cuda"))
    if kind == "router":
        d = case["d"]
        w_g = _normal(g, (d, E), d ** -0.5, "bf16")
        packed = torch.empty(B.moe_router_packed_bytes(d, E, B.MOE_BF16), dtype=torch.uint8, device="cuda")
        B.moe_pack_router(w_g, d, E, B.MOE_BF16, packed)
        return dict(case=case, x=_normal(g, (T, d), 1.0, "bf16"), packed=packed,
                    bias=torch.from_numpy(synth.zipf_log_bias(E, 1.0).astype(np.float32)).cuda(),
                    logits=torch.empty((T, E), device="cuda"), idx=_i32(T, k), w=torch.empty((T, k), device="cuda"))
    # profile: the second layer favours two successors of the first layer's top-1 expert (routing affinity)
    G = case["G"]
    lg0, lg1 = _logits(g, T, E, case["zipf"]), _logits(g, T, E, case["zipf"])
    succ = torch.from_numpy(synth.successors(1000, E).astype(np.int64)).cuda()
    lg1.scatter_add_(1, succ[lg0.argmax(dim=1)], torch.full((T, 2), 3.0, device="cuda"))
    i64 = dict(dtype=torch.int64, device="cuda")
    return dict(case=case, logits=(lg0, lg1), idx=(_i32(T, k), _i32(T, k)), w=(torch.empty((T, k), device="cuda"), torch.empty((T, k), device="cuda")),
                pl=(torch.from_numpy(synth.placement_contiguous(E, G)).cuda(), torch.from_numpy(synth.placement_balanced_random(E, G, 4000)).cuda()),
                perm=(_i32(T * k), _i32(T * k)), inv=(_i32(T * k), _i32(T * k)), cnt=(_i32(E), _i32(E)), start=_i32(E), gcnt=_i32(G), goff=_i32(G + 1),
                ws=torch.empty(max(256, B.moe_dispatch_workspace_bytes(T, E, k)), dtype=torch.uint8, device="cuda"),
                P=(torch.zeros(E, **i64), torch.zeros(E, **i64)), R=torch.zeros((E, E), **i64), loads=(torch.zeros(G, **i64), torch.zeros(G, **i64)),
                imb=(torch.zeros(1, dtype=torch.float64, device="cuda"), torch.zeros(1, dtype=torch.float64, device="cuda")),
                C=torch.zeros((G, G), **i64), cost=torch.zeros(1, dtype=torch.float64, device="cuda"),
                bw=(1.0 + torch.rand((G, G), generator=g, device="cuda")).double())


# ---- one pass -------------------------------------------------------------------
def run(s):
    c = s["case"]
    T, E, k = c["T"], c["E"], c["k"]
    if c["kind"] == "layer":
        L = s["L"]
        out = dict(y=L.forward(s["x"], s["logits"]), topk_idx=L.topk_idx, topk_w=L.topk_w, send_buf=L.send_buf, perm=L.perm, inv_perm=L.inv_perm,
                   expert_counts=L.expert_counts, expert_start=L.expert_start, gpu_counts=L.gpu_counts, gpu_offsets=L.gpu_offsets)
        if c["history"]:
            B.moe_transition_counts(s["prev"], L.topk_idx, T, k, k, E, E, s["R"])
            out["R"] = s["R"]
        return out
    if c["kind"] == "receive":
        B.moe_receive_segments(s["counts"], s["pl"], E, c["G"], c["local_gpu"], s["n_seg"], *s["seg"], s["src_offset"], s["n_seg_dev"])
        B.moe_expert_ffn_segments(s["recv"], B.MOE_BF16, s["n"], c["d"], c["f"], E, s["packed"], s["n_seg"], *s["seg"], s["out"], s["ws"])
        return dict(out=s["out"], seg=s["seg"], src_offset=s["src_offset"], n_seg=s["n_seg_dev"])
    if c["kind"] == "router":
        B.moe_router_gate(s["x"], B.MOE_BF16, s["packed"], s["bias"], T, c["d"], E, k, s["logits"], s["idx"], s["w"])
        return dict(logits=s["logits"], topk_idx=s["idx"], topk_w=s["w"])
    G = c["G"]
    for l in (0, 1):
        B.moe_topk_gate(s["logits"][l], T, E, k, s["idx"][l], s["w"][l])
        B.moe_dispatch(None, B.MOE_BF16, s["idx"][l], T, 0, E, k, s["pl"][l], G, None, s["perm"][l], s["inv"][l], s["cnt"][l], s["start"], s["gcnt"],
                       s["goff"], s["ws"])
        B.moe_accumulate_counts(s["cnt"][l], E, s["P"][l])
        B.moe_placement_loads(s["P"][l], s["pl"][l], E, G, s["loads"][l], s["imb"][l])
    B.moe_transition_counts(s["idx"][0], s["idx"][1], T, k, k, E, E, s["R"])
    B.moe_placement_traffic(s["R"], s["pl"][0], s["pl"][1], E, E, G, s["C"], s["bw"], s["cost"])
    return dict(idx=s["idx"], w=s["w"], perm=s["perm"], inv=s["inv"], cnt=s["cnt"], P=s["P"], R=s["R"], loads=s["loads"], imb=s["imb"], C=s["C"],
                cost=s["cost"])


# ---- what a pass cannot do without ---------------------------------------------------
def _routing(case, tokens):
    """(rows that reach this GPU's experts, those experts that get any) for `tokens` tokens: expectation over seeded draws."""
    E, k = case["E"], case["k"]
    mine = np.ones(E, dtype=bool) if case["local_gpu"] < 0 else _placement(case) == case["local_gpu"]
    rng = np.random.RandomState(0)
    reps = max(1, min(64, 20000 // tokens))
    n = min(tokens, 20000)
    rows, touched = [], []
    for _ in range(reps):
        lg = rng.standard_normal((n, E)) + synth.zipf_log_bias(E, case["zipf"])
        cnt = np.bincount(np.argpartition(-lg, k - 1, axis=1)[:, :k].reshape(-1), minlength=E)
        rows.append(cnt[mine].sum() * (tokens / n))
        touched.append((cnt[mine] > 0).sum())
    return float(np.mean(rows)), float(np.mean(touched))


def work(case):
    T, E, k = case["T"], case["E"], case["k"]
    N = T * k
    if case["kind"] == "router":
        d = case["d"]
        return dict(bytes=T * d * 2 + d * E * 2 + 4 * T * E + 8 * N, flops=2.0 * T * d * E)
    if case["kind"] == "profile":
        # two layers' logits, indices and weights (the indices read again by sort and history), the sorted order, the tables
        return dict(bytes=2 * (4 * T * E + 8 * N + 4 * N + 8 * N) + 8 * N + 16 * E * E, flops=0.0)
    d, f, elt = case["d"], case["f"], 2 if case["dtype"] == "bf16" else 4
    if case["kind"] == "receive":
        rows, touched = _routing(case, T * case["G"])
        return dict(bytes=touched * 3.0 * d * f * elt + 2 * rows * d * elt, flops=6.0 * d * f * rows)
    # layer: x, logits, the touched experts' weights in; gate outputs, sorted order, send buffer and y out
    rows, touched = _routing(case, T)
    b = 2 * T * d * elt + N * d * elt + 4 * T * E + 16 * N + touched * 3.0 * d * f * elt
    return dict(bytes=b + (4 * N if case["history"] else 0), flops=6.0 * d * f * rows)


def tolerance(case):
    """Four times what was measured against the same formulas in fp64 on the same inputs; indices and counts are exact.

    bf16 layer and receive (H and the expert outputs are rounded to bf16): 2-norm 2.9e-3, largest element 1.7e-2.
    fp32 layer: 2-norm 1.3e-6, largest element 8.0e-6.  Router: 1.2e-7 and 6.2e-7; two logits closer than that rounding
    may change places, one token in ten thousand.  Gate weights: 6.0e-8 and 2.3e-7."""
    if case["kind"] == "profile":
        return {"rel": 2.4e-7, "max": 1e-6}
    if case["kind"] == "router":
        return {"rel": 5e-7, "max": 2.5e-6, "differ": 2e-4}
    if case["dtype"] == "f32":
        return {"rel": 5.2e-6, "max": 3.2e-5}
    return {"rel": 1.15e-2, "max": 7e-2}
