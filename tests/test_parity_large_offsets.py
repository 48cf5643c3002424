"""GPU parity at sizes whose buffers pass 4 GiB and 2^31 elements.

The configurations' own buffers stay below 2^31 bytes, so an element or byte
offset kept in 32 bits anywhere in the row copy, the combine or the grouped
GEMM would pass every other test.  Here the send buffer of moe_dispatch is
4.9 GB (2.46e9 bf16 elements), the intermediate H of the expert FFN 4.6 GB
(2.29e9 elements), the gate's logits and the transition counts' index array
sit at their documented limits, and the router reads 4.9 GB of activations;
the rows checked include the last ones, which lie at the highest offsets.
Integer outputs and row copies are compared in full where the oracle can
afford it, float outputs on sampled rows that the oracle computes one by one.
"""
import numpy as np
import pytest
import torch

from oracle import moe_oracle as O
from paper_2502_06643_amd import synth
from paper_2502_06643_amd.layer import MoELayer, to_device, to_host
from util import TOL_BF16, TOL_F32, as_f64, rel_err

pytestmark = pytest.mark.gpu


def ends_and_random(rng, n, n_ends, n_random):
    """first and last n_ends of range(n) plus n_random others, sorted, distinct"""
    pick = set(range(min(n_ends, n))) | set(range(max(0, n - n_ends), n))
    pick |= set(rng.integers(0, n, size=n_random).tolist())
    return np.array(sorted(pick), dtype=np.int64)


def test_dispatch_rows_and_combine_past_4_GiB(lib):
    T, d, E, k, G = 300_000, 4096, 8, 2, 4
    assert T * k * d > 2 ** 31 and T * k * d * 2 > 2 ** 32
    x = synth.normal(71, 0, (T, d), 1.0, "bf16")
    idx = synth.random_topk_idx(71, T, E, k)
    pl = synth.placement_contiguous(E, G)
    rng = np.random.default_rng(71)
    w = rng.random((T, k)).astype(np.float32)
    ref = O.dispatch(x, idx, pl, G)

    L = MoELayer(T, d, 64, E, k, G, -1, "bf16")
    L.set_placement(pl)
    L.topk_idx.copy_(torch.from_numpy(idx))
    L.topk_w.copy_(torch.from_numpy(w))
    L.send_buf.fill_(3.0)
    L.dispatch(to_device(x))
    torch.cuda.synchronize()
    for n in ("expert_counts", "expert_start", "gpu_counts", "gpu_offsets", "perm", "inv_perm"):
        np.testing.assert_array_equal(getattr(L, n).cpu().numpy(), ref[n], err_msg=n)
    step = 50_000
    for r0 in range(0, T * k, step):                       # bit copies, compared in pieces to bound the temporaries
        got = to_host(L.send_buf[r0:r0 + step])
        assert np.array_equal(got, ref["send_buf"][r0:r0 + step]), f"send_buf rows {r0}..{r0 + step}"

    # combine on the oracle's own buffers: the expert outputs are the oracle's send buffer (an identity expert)
    L.ffn_out.copy_(to_device(ref["send_buf"]))
    L.inv_perm.copy_(torch.from_numpy(ref["inv_perm"]))
    tokens = ends_and_random(rng, T, 32, 400)
    o_sub = ref["send_buf"][ref["inv_perm"].reshape(T, k)[tokens].reshape(-1)]
    inv_sub = np.arange(len(tokens) * k, dtype=np.int32)
    for local in (-1, G - 1):                              # all resident; the last GPU, whose buckets lie at the highest offsets
        L.local_gpu = local
        L.y.fill_(5.0)
        L.combine()
        torch.cuda.synchronize()
        got = as_f64(to_host(L.y[torch.from_numpy(tokens).cuda()]))
        want = O.combine(o_sub, inv_sub, idx[tokens], w[tokens], pl, local)
        assert rel_err(got, want) <= 4e-3, local           # one bf16 rounding of a fp32 sum of k terms
        if local >= 0:
            none_local = ~(pl[idx[tokens]] == local).any(axis=1)
            assert none_local.any() and not got[none_local].any()


def test_expert_ffn_with_an_intermediate_past_2_to_31_elements(lib):
    cfg = synth.config("c2").with_(T=80_000, name="c2@T=80000")
    N = cfg.T * cfg.k
    assert N * cfg.f > 2 ** 31
    x = synth.make_x(cfg)
    idx = synth.random_topk_idx(72, cfg.T, cfg.E, cfg.k)
    pl = synth.make_placement(cfg)
    weights = synth.make_expert_weights(cfg)
    dsp = O.dispatch(x, idx, pl, cfg.G)

    L = MoELayer(cfg.T, cfg.d, cfg.f, cfg.E, cfg.k, cfg.G, -1, "bf16")
    L.set_placement(pl)
    L.set_weights(*weights)
    L.send_buf.copy_(to_device(dsp["send_buf"]))
    L.expert_counts.copy_(torch.from_numpy(dsp["expert_counts"]))
    L.expert_start.copy_(torch.from_numpy(dsp["expert_start"]))
    L.ffn()
    torch.cuda.synchronize()

    rng = np.random.default_rng(72)
    rows = []
    for e in range(cfg.E):                                 # per bucket: its ends (first and last row tiles) and random rows
        c, s = int(dsp["expert_counts"][e]), int(dsp["expert_start"][e])
        rows.append(s + ends_and_random(rng, c, 3, 6))
    rows = np.concatenate(rows)
    assert rows.max() == N - 1
    want = O.expert_ffn_grouped(dsp["send_buf"], *weights, dsp["expert_counts"], dsp["expert_start"], pl, -1, positions=rows)[rows]
    got = as_f64(to_host(L.ffn_out[torch.from_numpy(rows).cuda()]))
    err = rel_err(got, want)
    print(f"\nffn_out on {len(rows)} sampled rows of {N}: rel_err {err:.3e}")
    assert err <= TOL_BF16


def test_gate_at_the_size_limit_of_its_logits(lib):
    """T * E just under 2^31 (the call's documented limit): the last tokens' logits lie 8.5 GB into the array."""
    T, E, k = 8_300_000, 256, 8
    assert T * E < 2 ** 31 and T * E * 4 > 2 ** 32
    lg = synth.normal(73, 1, (T, E), 2.0, "f32")
    dl = torch.from_numpy(lg).cuda()
    idx = torch.full((T, k), -7, dtype=torch.int32, device="cuda")
    w = torch.full((T, k), -1.0, dtype=torch.float32, device="cuda")
    lib.moe_topk_gate(dl, T, E, k, idx, w)
    torch.cuda.synchronize()
    tokens = ends_and_random(np.random.default_rng(73), T, 256, 4000)
    sel = torch.from_numpy(tokens).cuda()
    gi, gw = idx[sel].cpu().numpy(), w[sel].cpu().numpy()
    oi, ow = O.topk_gate(lg[tokens], k)
    np.testing.assert_array_equal(gi, oi)
    assert float(np.max(np.abs(gw.astype(np.float64) - ow) / np.maximum(ow, 1e-30))) <= 1e-4
    # every token got its k distinct experts: nothing left at the fill value anywhere
    assert int((idx < 0).sum()) == 0 and int((w < 0).sum()) == 0


def test_transition_counts_at_the_size_limit_of_an_index_array(lib):
    """T * k just under 2^31 entries (the documented limit) in layer l's array: 8.6 GB of indices.  Layer l lists all
    16 experts per token (a rotation of 0..15 by a seeded offset: cheap to make at this size), layer l+1 one expert,
    so every row of R is the histogram of layer l+1's choices and the top-1 pairs are (offset, choice)."""
    T, E, k = 134_000_000, 16, 16
    assert T * k < 2 ** 31 and T * k * 4 > 2 ** 32
    rng = np.random.default_rng(74)
    ra = rng.integers(0, E, size=T, dtype=np.int32)
    rb = rng.integers(0, E, size=T, dtype=np.int32)
    base = torch.arange(E, dtype=torch.int32, device="cuda")
    a = ((torch.from_numpy(ra).cuda()[:, None] + base[None, :]) % E).contiguous()
    b = torch.from_numpy(rb).cuda().reshape(T, 1)
    R = torch.zeros((E, E), dtype=torch.int64, device="cuda")
    lib.moe_transition_counts(a, b, T, k, 1, E, E, R)
    Rp = torch.zeros((E, E), dtype=torch.int64, device="cuda")
    lib.moe_transition_counts_pairs(a, b, T, k, 1, E, E, lib.MOE_PAIRS_TOP1, Rp)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(R.cpu().numpy(), np.tile(np.bincount(rb, minlength=E), (E, 1)))
    want = np.zeros((E, E), dtype=np.int64)
    np.add.at(want, (ra, rb), 1)
    np.testing.assert_array_equal(Rp.cpu().numpy(), want)


def test_router_gate_with_activations_past_4_GiB(lib):
    """The fused router reads 4.9 GB of activations; logits and selection of sampled tokens (the last ones included)
    against the fp64 router, with the margin rule for near ties that the router tests use."""
    T, d, E, k = 600_000, 4096, 8, 2
    assert T * d > 2 ** 31
    x = synth.normal(75, 0, (T, d), 1.0, "bf16")
    w_g = synth.normal(75, 1, (d, E), 1.0 / np.sqrt(d), "bf16")
    bias = np.random.default_rng(75).standard_normal(E).astype(np.float32)
    packed = torch.empty(lib.moe_router_packed_bytes(d, E, lib.MOE_BF16), dtype=torch.uint8, device="cuda")
    lib.moe_pack_router(to_device(w_g), d, E, lib.MOE_BF16, packed)
    logits = torch.full((T, E), 7.0, dtype=torch.float32, device="cuda")
    idx = torch.full((T, k), -1, dtype=torch.int32, device="cuda")
    w = torch.full((T, k), -1.0, dtype=torch.float32, device="cuda")
    lib.moe_router_gate(to_device(x), lib.MOE_BF16, packed, torch.from_numpy(bias).cuda(), T, d, E, k, logits, idx, w)
    torch.cuda.synchronize()
    assert int((idx < 0).sum()) == 0
    tokens = ends_and_random(np.random.default_rng(75), T, 64, 2000)
    sel = torch.from_numpy(tokens).cuda()
    lg, gi = logits[sel].cpu().numpy(), idx[sel].cpu().numpy()
    lg_ref, idx_ref, _ = O.router_gate(x[tokens], w_g, bias, k)
    scale = np.sqrt(np.mean(lg_ref ** 2, axis=1, keepdims=True)) + 1e-30
    assert np.max(np.abs(lg - lg_ref) / np.maximum(np.abs(lg_ref), scale)) <= 1e-5
    srt = -np.sort(-lg_ref, axis=1)
    clear = np.all(srt[:, :k] - srt[:, 1:k + 1] > 2e-5 * scale, axis=1)
    assert clear.mean() > 0.9
    np.testing.assert_array_equal(gi[clear], idx_ref[clear])


def test_router_weights_past_4_GiB(lib):
    """One token past the smallest batches, and a reduction so long that a panel of 32 experts' weights has 4.3 GB: the
    logits are whole numbers that the first, the middle and the last weights of the reduction make."""
    T, d, E, k = 513, 1 << 26, 8, 2
    if torch.cuda.mem_get_info()[0] < 90 << 30:
        pytest.skip("needs 75 GB")
    x = torch.ones((T, d), dtype=torch.bfloat16, device="cuda")
    t = torch.arange(T, device="cuda") % 100
    x[:, d - 1] = t.to(torch.bfloat16)
    w = torch.zeros((d, E), dtype=torch.bfloat16, device="cuda")
    e = torch.arange(E, device="cuda")
    w[0], w[d // 2 + 5], w[d - 1] = (e % 3).to(torch.bfloat16), (e % 2).to(torch.bfloat16), e.to(torch.bfloat16)
    packed = torch.empty(lib.moe_router_packed_bytes(d, E, lib.MOE_BF16), dtype=torch.uint8, device="cuda")
    lib.moe_pack_router(w, d, E, lib.MOE_BF16, packed)
    logits, idx = torch.empty((T, E), device="cuda"), torch.empty((T, k), dtype=torch.int32, device="cuda")
    lib.moe_router_gate(x, lib.MOE_BF16, packed, None, T, d, E, k, logits, idx, torch.empty((T, k), device="cuda"))
    torch.cuda.synchronize()
    want = (e % 3 + e % 2)[None, :] + t[:, None] * e[None, :]
    assert torch.equal(logits, want.float())
    del x, w, packed
    torch.cuda.empty_cache()


@pytest.mark.parametrize("dtype,E", [("f32", 98), ("bf16", 196)])
def test_packed_weights_of_more_than_2_to_32_units(lib, dtype, E):
    """64.3 GiB of packed weights, more units of 16 bytes than HIP launches threads: the first, a middle and the last expert
    against the oracle.  W1 and W3 are the same array, and W2 is another view of it."""
    d, f, k = 4096, 14336, 1
    assert E * 3 * d * f * (4 if dtype == "f32" else 2) > 16 << 32
    if torch.cuda.mem_get_info()[0] < 100 << 30:
        pytest.skip("needs 92 GB")
    g = torch.Generator(device="cuda").manual_seed(76)
    w = torch.empty((E, d, f), dtype=torch.float32 if dtype == "f32" else torch.bfloat16, device="cuda")
    for e in range(E):
        w[e].normal_(0.0, d ** -0.5, generator=g)
    dt = lib.MOE_F32 if dtype == "f32" else lib.MOE_BF16
    packed = torch.empty(lib.moe_packed_weights_bytes(E, d, f, dt), dtype=torch.uint8, device="cuda")
    lib.moe_pack_weights(w, w, w.view(E, f, d), E, d, f, dt, packed)
    experts = [0, E // 2, E - 1]
    x = synth.normal(76, 0, (9, d), 1.0, dtype)
    counts, start = np.zeros(E, dtype=np.int32), np.zeros(E, dtype=np.int32)
    counts[experts] = 3
    start[1:] = np.cumsum(counts)[:-1]
    pl = np.zeros(E, dtype=np.int32)
    out = torch.zeros((9, d), dtype=w.dtype, device="cuda")
    ws = torch.empty(lib.moe_ffn_workspace_bytes(9, d, f, E, dt), dtype=torch.uint8, device="cuda")
    lib.moe_expert_ffn_grouped(to_device(x), dt, 9, d, f, E, packed, *[torch.from_numpy(a).cuda() for a in (counts, start, pl)], -1, out, ws)
    torch.cuda.synchronize()
    some = [to_host(w[e]) for e in experts]
    del w, packed
    torch.cuda.empty_cache()
    w1, w2 = np.stack(some), np.stack([a.reshape(f, d) for a in some])
    ref = O.expert_ffn_grouped(x, w1, w1, w2, np.full(3, 3, dtype=np.int32), np.array([0, 3, 6], dtype=np.int32), np.zeros(3, dtype=np.int32), -1)
    assert rel_err(as_f64(to_host(out)), ref) <= (TOL_F32 if dtype == "f32" else TOL_BF16)


def test_packed_matrix_of_more_than_2_to_30_units(lib):
    """One expert whose matrices have 16 GiB each, so that a thread packs several units; against the same formula in fp64, a piece of
    the reduction at a time."""
    d, f, N = 65536, 65600, 3
    assert d * f > 4 << 30
    if torch.cuda.mem_get_info()[0] < 80 << 30:
        pytest.skip("needs 70 GB")
    g = torch.Generator(device="cuda").manual_seed(77)
    w = torch.empty((d, f), device="cuda")
    for i in range(0, d, 4096):
        w[i:i + 4096].normal_(0.0, d ** -0.5, generator=g)
    packed = torch.empty(lib.moe_packed_weights_bytes(1, d, f, lib.MOE_F32), dtype=torch.uint8, device="cuda")
    lib.moe_pack_weights(w, w, w.view(f, d), 1, d, f, lib.MOE_F32, packed)
    x = torch.randn((N, d), generator=g, device="cuda")
    i32 = lambda v: torch.tensor([v], dtype=torch.int32, device="cuda")
    out = torch.zeros((N, d), device="cuda")
    ws = torch.empty(lib.moe_ffn_workspace_bytes(N, d, f, 1, lib.MOE_F32), dtype=torch.uint8, device="cuda")
    lib.moe_expert_ffn_grouped(x, lib.MOE_F32, N, d, f, 1, packed, i32(N), i32(0), i32(0), -1, out, ws)

    def product(a, b):
        return sum(a[:, i:i + 2048].double() @ b[i:i + 2048].double() for i in range(0, len(b), 2048))

    up = product(x, w)
    ref = product(up * torch.sigmoid(up) * up, w.view(f, d)).cpu().numpy()
    got = out.cpu().numpy()
    del w, packed
    torch.cuda.empty_cache()
    assert rel_err(got.astype(np.float64), ref) <= TOL_F32
