"""GPU parity: the receiving side of the expert-parallel layer (Section 2.2 / Fig. 2b) emulated on one
GPU: G virtual ranks dispatch, the buckets are copied as the all-to-all would move them, every rank runs
moe_expert_ffn_segments over the (source, expert) segments it received, results return, ranks combine.
Receive layout and segment tables bit exact against oracle.exchange_to; floats to the usual tolerances;
every rank's y must equal the single-GPU, all-experts-resident layer on that rank's tokens."""
import numpy as np
import pytest
import torch

from oracle import moe_oracle as O
from paper_2502_06643_amd import binding as B
from paper_2502_06643_amd import synth
from paper_2502_06643_amd.ep_emulation import ExpertParallelGroup
from paper_2502_06643_amd.layer import to_device, to_host
from util import TOL_BF16, TOL_F32, as_f64, fro_err, rel_err

pytestmark = pytest.mark.gpu


def make_group(seed, G, T_rank, d, f, E, k, dtype, placement):
    w1 = synth.normal(seed, 2, (E, d, f), 1 / np.sqrt(d), dtype)
    w3 = synth.normal(seed, 3, (E, d, f), 1 / np.sqrt(d), dtype)
    w2 = synth.normal(seed, 4, (E, f, d), 1 / np.sqrt(f), dtype)
    xs = [synth.normal(seed, 10 + r, (T_rank, d), 1.0, dtype) for r in range(G)]
    rng = np.random.default_rng(seed)
    lgs = [(rng.standard_normal((T_rank, E)) * 2 - np.log(np.arange(1, E + 1))[None, :]).astype(np.float32) for _ in range(G)]
    grp = ExpertParallelGroup(G, T_rank, d, f, E, k, placement, dtype, w1, w3, w2)
    return grp, (w1, w3, w2), xs, lgs


@pytest.mark.parametrize("dtype,G,T_rank,d,f,E,k,placement", [
    ("f32", 4, 64, 64, 128, 8, 2, [0, 0, 1, 1, 2, 2, 3, 3]),
    ("f32", 4, 50, 36, 100, 8, 2, [3, 1, 0, 2, 1, 3, 2, 0]),          # non-contiguous map
    ("f32", 3, 40, 32, 64, 7, 3, [0, 0, 0, 0, 2, 2, 2]),               # uneven: rank 1 owns no expert
    ("bf16", 4, 512, 256, 512, 8, 2, [0, 0, 1, 1, 2, 2, 3, 3]),
    ("bf16", 2, 700, 128, 320, 16, 4, [1, 0] * 8),
    ("bf16", 8, 96, 128, 192, 64, 6, list(np.arange(64) % 8)),        # 8 segments of each of 8 experts per receiver
])
def test_expert_parallel_group_matches_oracle(lib, dtype, G, T_rank, d, f, E, k, placement):
    pl = np.array(placement, dtype=np.int32)
    grp, weights, xs, lgs = make_group(T_rank + d, G, T_rank, d, f, E, k, dtype, pl)
    ys = grp.forward([to_device(x) for x in xs], [torch.from_numpy(l).cuda() for l in lgs])
    torch.cuda.synchronize()
    tol = TOL_BF16 if dtype == "bf16" else TOL_F32
    gates = [O.topk_gate(l, k) for l in lgs]
    dsps = [O.dispatch(xs[r], gates[r][0], pl, G) for r in range(G)]
    for dest in range(G):
        ex = O.exchange_to(dsps, pl, dest)
        got = grp.received[dest]
        np.testing.assert_array_equal(to_host(got["recv_buf"]).reshape(ex["recv_buf"].shape), ex["recv_buf"])
        # the segment table was built on the device (moe_receive_segments): bit exact against the oracle's exchange
        np.testing.assert_array_equal(got["seg_expert"].cpu().numpy(), ex["seg_expert"])
        np.testing.assert_array_equal(got["seg_counts"].cpu().numpy(), ex["seg_counts"])
        np.testing.assert_array_equal(got["seg_start"].cpu().numpy(), ex["seg_start"])
        if got["n_seg"]:
            assert int(got["n_seg_dev"].cpu()[0]) == len(ex["seg_expert"])
            np.testing.assert_array_equal(got["src_offset"].cpu().numpy(), ex["src_offset"])
        if len(ex["recv_buf"]) == 0:
            continue
        ref = O.expert_ffn_segments(ex["recv_buf"], *weights, ex["seg_expert"], ex["seg_counts"], ex["seg_start"])
        out = as_f64(to_host(got["out"]))
        assert rel_err(out, ref) <= tol
        assert fro_err(out, ref) <= tol
    for r in range(G):
        single = O.moe_layer(xs[r], lgs[r], k, *weights, pl, G, -1)            # all experts resident on one GPU
        y = as_f64(to_host(ys[r]))
        assert fro_err(y, single["y"]) <= tol
        e2e = rel_err(y, single["y"])
        print(f"receive side {dtype} G={G} rank {r}: y end to end rel_err = {e2e:.3e}")
        assert e2e <= tol


@pytest.mark.parametrize("dtype,d,f,E,segs", [
    # (expert, rows): segments of one expert apart from each other, empty ones, an expert with one segment only
    ("bf16", 64, 128, 4, [(2, 3), (0, 1), (2, 0), (1, 5), (2, 40), (0, 2)]),                       # streaming kernels
    ("bf16", 128, 192, 3, [(1, 9), (0, 7)] * 10),                                                  # ... 160 rows, ten segments a bucket
    ("bf16", 128, 192, 3, [(1, 9), (0, 7)] * 10 + [(2, 1)]),                                       # the first batch on tiles
    ("bf16", 128, 1088, 3, [(0, 130), (2, 126), (0, 127), (2, 1), (1, 256), (0, 3)]),              # tiles across segments; 17 k tiles
    ("bf16", 2048, 2048, 2, [(0, 300), (1, 20), (0, 201), (1, 90), (0, 12)]),                      # one round, cut along k
    ("bf16", 64, 64, 2, [(0, 600), (1, 520), (0, 544), (1, 560)]),                                 # large segments stay buckets (tall tiles)
    ("bf16", 64, 64, 256, [(e, 1 + e % 3) for e in range(255, -1, -1)]),                           # 256 buckets, nothing to merge
    ("bf16", 64, 64, 2, [(i % 2, 1 + i % 5) for i in range(256)]),                                 # 128 segments a bucket
    ("f32", 36, 100, 3, [(2, 3), (0, 31), (2, 33), (0, 1), (2, 0), (1, 64), (2, 30)]),
    ("f32", 1028, 1500, 2, [(0, 300), (1, 20), (0, 401), (1, 590), (0, 350)]),                     # large enough for the three-piece kernels
])
def test_segments_of_one_expert_in_any_order(lib, dtype, d, f, E, segs):
    """moe_expert_ffn_segments over a buffer whose segments lie in an order of their own, with rows between them that
    belong to none: those stay untouched, the others match the oracle."""
    rng = np.random.default_rng(d + f + len(segs))
    w = [synth.normal(d, i, s, s[1] ** -0.5, dtype) for i, s in ((2, (E, d, f)), (3, (E, d, f)), (4, (E, f, d)))]
    se, sc = np.array(segs, dtype=np.int32).T.copy()
    starts, at = np.zeros(len(segs), dtype=np.int32), 0
    gaps = 2 if sc.sum() > 160 or sc.sum() < 100 else 0
    for j in rng.permutation(len(segs)):
        starts[j] = at
        at += int(sc[j]) + (gaps if j % 2 else 0)
    N = max(at, 1)
    x = synth.normal(d + 1, 0, (N, d), 1.0, dtype)
    dt = B.MOE_BF16 if dtype == "bf16" else B.MOE_F32
    packed = torch.empty(B.moe_packed_weights_bytes(E, d, f, dt), dtype=torch.uint8, device="cuda")
    B.moe_pack_weights(*[to_device(a) for a in w], E, d, f, dt, packed)
    ws = torch.empty(B.moe_ffn_workspace_bytes(N, d, f, E, dt), dtype=torch.uint8, device="cuda").fill_(0xAA)
    out = torch.full((N, d), 7.0, dtype=torch.bfloat16 if dtype == "bf16" else torch.float32, device="cuda")
    dev = lambda a: torch.from_numpy(a).cuda()
    B.moe_expert_ffn_segments(to_device(x), dt, N, d, f, E, packed, len(segs), dev(se), dev(sc), dev(starts), out, ws)
    torch.cuda.synchronize()
    ref = O.expert_ffn_segments(x, *w, se, sc, starts)
    mine = np.zeros(N, dtype=bool)
    for s, c in zip(starts, sc):
        mine[s:s + c] = True
    got, tol = as_f64(to_host(out)), TOL_BF16 if dtype == "bf16" else TOL_F32
    assert rel_err(got[mine], np.asarray(ref)[mine]) <= tol
    assert np.all(got[~mine] == 7.0)


def test_f32_segments_with_infinite_and_tiny_rows(lib):
    """Merged buckets of the three-piece kernels: rows that are computed again are found where their segments lie."""
    d, f, E = 1028, 1500, 2
    se, sc = np.array([(0, 300), (1, 20), (0, 401), (1, 590), (0, 350)], dtype=np.int32).T.copy()
    ss = np.zeros(5, dtype=np.int32)
    at = 0
    for j in (3, 0, 4, 1, 2):                                          # in an order of their own
        ss[j] = at
        at += int(sc[j])
    w = [synth.normal(d, i, s, s[1] ** -0.5, "f32") for i, s in ((2, (E, d, f)), (3, (E, d, f)), (4, (E, f, d)))]
    x = synth.normal(d + 1, 0, (at, d), 1.0, "f32")
    bad, tiny = np.zeros(at, dtype=bool), np.zeros(at, dtype=bool)
    for s, c in zip(ss, sc):
        bad[s + c // 2] = tiny[[s, s + c - 1]] = True                  # the first and the last row of every segment
    x[tiny] *= np.float32(2e-18)
    dev = lambda a: torch.from_numpy(a).cuda()
    packed = torch.empty(B.moe_packed_weights_bytes(E, d, f, B.MOE_F32), dtype=torch.uint8, device="cuda")
    B.moe_pack_weights(*[to_device(a) for a in w], E, d, f, B.MOE_F32, packed)
    ws = torch.empty(B.moe_ffn_workspace_bytes(at, d, f, E, B.MOE_F32), dtype=torch.uint8, device="cuda")
    ref = np.asarray(O.expert_ffn_segments(x, *w, se, sc, ss))
    x[bad, 5] = np.inf
    out = torch.full((at, d), 7.0, device="cuda")
    B.moe_expert_ffn_segments(to_device(x), B.MOE_F32, at, d, f, E, packed, 5, dev(se), dev(sc), dev(ss), out, ws)
    torch.cuda.synchronize()
    assert int(ws[28:32].view(torch.int32)) == 1                       # the plan's header: merged
    got = to_host(out)
    assert not np.isfinite(got[bad]).any()
    for rows in (tiny, ~tiny & ~bad):
        assert fro_err(got[rows], ref[rows]) <= 1e-6
        assert rel_err(got[rows], ref[rows]) <= TOL_F32


@pytest.mark.parametrize("d,f,E,segs,merged", [
    # whether the plan merges the segments of an expert, on both sides of its rule (256 compute units), and what it computes then
    (64, 1408, 6, [(0, 6)] * 9 + [(0, 5)] + [(e, 3) for e in (1, 2, 3, 4, 5)], 0),                 # streaming, a bucket of 59 rows: apart
    (64, 1408, 6, [(0, 4)] * 10 + [(e, 3) for e in (1, 2, 3, 4, 5)], 1),                           # ... of 40 rows
    (64, 14336, 3, [(0, 4), (1, 2), (0, 2), (2, 1)], 0),                                           # four segments, three experts
    (128, 1408, 3, [(i % 3, 20) for i in range(17)], 0),                                           # tiles: one round either way
    (128, 2112, 3, [(i % 3, 1 + 7 * i % 60) for i in range(48)], 1),                               # ... more than two rounds
    (64, 320, 2, [(i % 2, 1 + i % 5) for i in range(256)], 1),                                     # ... 128 segments a bucket
    (64, 64, 2, [(0, 1000), (1, 600), (0, 544), (1, 560)], 0),                                     # enough rows a segment for tall tiles
])
def test_segments_merge_where_it_pays(lib, d, f, E, segs, merged):
    w = [synth.normal(d, i, s, s[1] ** -0.5, "bf16") for i, s in ((2, (E, d, f)), (3, (E, d, f)), (4, (E, f, d)))]
    se, sc = np.array(segs, dtype=np.int32).T.copy()
    ss = np.concatenate([[0], np.cumsum(sc)[:-1]]).astype(np.int32)
    N = int(sc.sum())
    x = synth.normal(d + 1, 0, (N, d), 1.0, "bf16")
    packed = torch.empty(B.moe_packed_weights_bytes(E, d, f, B.MOE_BF16), dtype=torch.uint8, device="cuda")
    B.moe_pack_weights(*[to_device(a) for a in w], E, d, f, B.MOE_BF16, packed)
    ws = torch.empty(B.moe_ffn_workspace_bytes(N, d, f, E, B.MOE_BF16), dtype=torch.uint8, device="cuda").fill_(0xAA)
    out = torch.full((N, d), 7.0, dtype=torch.bfloat16, device="cuda")
    dev = lambda a: torch.from_numpy(a).cuda()
    B.moe_expert_ffn_segments(to_device(x), B.MOE_BF16, N, d, f, E, packed, len(segs), dev(se), dev(sc), dev(ss), out, ws)
    torch.cuda.synchronize()
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        assert int(ws[28:32].view(torch.int32)) == merged              # the plan's header
    assert rel_err(as_f64(to_host(out)), O.expert_ffn_segments(x, *w, se, sc, ss)) <= TOL_BF16


def test_receive_segments_table_edge_cases(lib):
    """moe_receive_segments against a host loop: uneven map, a destination without experts, negative counts, a table
    that is larger than needed (padded with empty segments at the end) and one that is too small (n_seg says so)."""
    G, E = 5, 12
    rng = np.random.default_rng(9)
    pl = np.array([0, 3, 3, 1, 0, 3, 4, 4, 3, 0, 1, 3], dtype=np.int32)          # GPU 2 owns nothing
    counts = rng.integers(0, 50, (G, E)).astype(np.int32)
    counts[2, 5] = -7                                                            # treated as 0
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    for dest in range(G):
        experts = [e for e in range(E) if pl[e] == dest]
        want_e = np.array(experts * G, dtype=np.int32)
        want_c = np.array([max(0, counts[s, e]) for s in range(G) for e in experts], dtype=np.int32)
        want_s = np.concatenate([[0], np.cumsum(want_c)[:-1]]).astype(np.int32) if len(want_c) else want_c
        total = int(want_c.sum())
        for max_seg in (max(1, len(want_e)), len(want_e) + 3, max(1, len(want_e) - 2)):
            i32 = dict(dtype=torch.int32, device="cuda")
            se, sc, ss = (torch.full((max_seg,), -1, **i32) for _ in range(3))
            off, n = torch.full((G + 1,), -1, **i32), torch.full((1,), -1, **i32)
            B.moe_receive_segments(dev(counts), dev(pl), E, G, dest, max_seg, se, sc, ss, off, n)
            torch.cuda.synchronize()
            assert int(n.cpu()[0]) == len(want_e)
            m = min(max_seg, len(want_e))
            np.testing.assert_array_equal(se.cpu().numpy()[:m], want_e[:m])
            np.testing.assert_array_equal(sc.cpu().numpy()[:m], want_c[:m])
            np.testing.assert_array_equal(ss.cpu().numpy()[:m], want_s[:m])
            if max_seg >= len(want_e):
                assert np.all(sc.cpu().numpy()[m:] == 0) and np.all(ss.cpu().numpy()[m:] == total)
                per_src = want_c.reshape(G, -1).sum(axis=1) if len(want_c) else np.zeros(G, dtype=np.int64)
                np.testing.assert_array_equal(off.cpu().numpy(), np.concatenate([[0], np.cumsum(per_src)]))
    with pytest.raises(B.MoeError):
        B.moe_receive_segments(dev(counts), dev(pl), E, G, G, 8, se, sc, ss, off, n)          # dest outside [0,G)
    with pytest.raises(B.MoeError):
        B.moe_receive_segments(dev(counts), dev(pl), E, G, 0, 257, se, sc, ss, off, n)        # more than the segment FFN takes


@pytest.mark.parametrize("E,G,dest,own,cuts", [
    # the experts of dest; table sizes beside one that is just large enough
    (256, 1, 0, range(256), (255, 193, 65, 1)),                                 # 256 segments of one source
    (256, 4, 2, range(2, 256, 4), (255, 129, 128, 100)),                        # 16 experts in each of the four groups of 64
    (256, 3, 1, [0, 63, 64, 65, 127, 128, 191, 192, 254, 255], (31, 25, 20)),   # at the ends of the groups, 30 segments
    (200, 5, 4, range(150, 200), (249, 130, 64)),                               # none in the first group
    (130, 13, 0, [5, 66, 67, 128, 129], (66, 63)),                              # 65 segments
    (256, 100, 99, [70, 250], (256, 199, 129, 3)),                              # more sources than a wavefront has lanes
    (80, 256, 7, [79], (255, 200)),                                             # one segment a source
    (256, 256, 7, [3, 200], (256,)),                                            # 512 segments, more than any table holds
    (256, 70, 5, [], (1, 256)),                                                 # no expert here
])
def test_receive_segments_across_wavefronts(lib, E, G, dest, own, cuts):
    """More than 64 experts, segments or sources: ranks, starts and totals that are carried from one wavefront to the next.  A table that
    is too small holds the first segments; a source whose first segment fits begins there, the others at the table's total."""
    rng = np.random.default_rng(E + G)
    own = list(own)
    pl = np.full(E, (dest + 1) % G, dtype=np.int32)
    pl[own] = dest
    counts = rng.integers(0, 50, (G, E)).astype(np.int32)
    counts[rng.random((G, E)) < 0.2] = 0
    want_e, want_c = np.array(own * G, dtype=np.int32), counts[:, own].reshape(-1)
    ends = np.concatenate([[0], np.cumsum(want_c)])
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    for max_seg in (min(256, max(1, len(want_e))), *cuts):
        se, sc, ss, off, n = (torch.full((m,), -1, dtype=torch.int32, device="cuda") for m in (max_seg, max_seg, max_seg, G + 1, 1))
        lib.moe_receive_segments(dev(counts), dev(pl), E, G, dest, max_seg, se, sc, ss, off, n)
        torch.cuda.synchronize()
        m = min(max_seg, len(want_e))
        assert int(n.cpu()[0]) == len(want_e)
        np.testing.assert_array_equal(se.cpu().numpy()[:m], want_e[:m])
        np.testing.assert_array_equal(sc.cpu().numpy(), np.concatenate([want_c[:m], np.zeros(max_seg - m, dtype=np.int32)]))
        np.testing.assert_array_equal(ss.cpu().numpy(), np.concatenate([ends[:m], np.full(max_seg - m, ends[m])]))
        np.testing.assert_array_equal(off.cpu().numpy(), ends[np.minimum(np.arange(G + 1) * len(own), m)])


def test_segments_entry_point_edge_cases(lib):
    d, f, E = 64, 128, 4
    w1 = synth.normal(1, 2, (E, d, f), 1 / np.sqrt(d), "f32")
    w3 = synth.normal(1, 3, (E, d, f), 1 / np.sqrt(d), "f32")
    w2 = synth.normal(1, 4, (E, f, d), 1 / np.sqrt(f), "f32")
    packed = torch.empty(B.moe_packed_weights_bytes(E, d, f, B.MOE_F32), dtype=torch.uint8, device="cuda")
    B.moe_pack_weights(to_device(w1), to_device(w3), to_device(w2), E, d, f, B.MOE_F32, packed)
    N = 300
    a = synth.normal(1, 0, (N, d), 1.0, "f32")
    ws = torch.empty(B.moe_ffn_workspace_bytes(N, d, f, E, B.MOE_F32), dtype=torch.uint8, device="cuda")

    def run(se, sc, ss):
        out = torch.full((N, d), 7.0, device="cuda")
        B.moe_expert_ffn_segments(to_device(a), B.MOE_F32, N, d, f, E, packed, len(se), to_device(np.array(se, dtype=np.int32)),
                                  to_device(np.array(sc, dtype=np.int32)), to_device(np.array(ss, dtype=np.int32)), out, ws)
        torch.cuda.synchronize()
        return out.cpu().numpy().astype(np.float64)

    # the same expert in several segments, an empty segment, rows that belong to no segment (left untouched)
    se, sc, ss = [2, 0, 2, 1, 3], [100, 0, 37, 1, 50], [0, 100, 100, 137, 200]
    got = run(se, sc, ss)
    ref = O.expert_ffn_segments(a, w1, w3, w2, se, sc, ss)
    covered = np.zeros(N, dtype=bool)
    for c, s in zip(sc, ss):
        covered[s:s + c] = True
    assert rel_err(got[covered], ref[covered]) <= TOL_F32
    assert np.all(got[~covered] == 7.0)
    # segments that leave the buffer or name a missing expert are skipped, the others still run
    got = run([1, 9, 0, 2], [50, 50, 400, 20], [0, 50, 100, 280])
    ref = O.expert_ffn_segments(a, w1, w3, w2, [1, 2], [50, 20], [0, 280])
    assert rel_err(got[:50], ref[:50]) <= TOL_F32 and rel_err(got[280:], ref[280:]) <= TOL_F32
    assert np.all(got[50:280] == 7.0)
    # no segment at all: nothing happens
    out = torch.full((N, d), 7.0, device="cuda")
    B.moe_expert_ffn_segments(to_device(a), B.MOE_F32, N, d, f, E, packed, 0, packed, packed, packed, out, ws)
    torch.cuda.synchronize()
    assert torch.all(out == 7.0)
    with pytest.raises(B.MoeError):
        B.moe_expert_ffn_segments(to_device(a), B.MOE_F32, N, d, f, E, packed, 257, packed, packed, packed, out, ws)


def test_mixtral_shape_receiver_sampled(lib):
    """4 ranks x 1024 tokens of the Mixtral-8x7B shape, EP=4 contiguous map: receiver 0's buffer and segment table
    bit for bit against the oracle's exchange, and its segment FFN on sampled rows (first, last and random rows of
    every segment) against the oracle run on the oracle's own receive buffer."""
    G, T_rank, d, f, E, k = 4, 1024, 4096, 14336, 8, 2
    pl = np.repeat(np.arange(G), E // G).astype(np.int32)
    grp, weights, xs, lgs = make_group(77, G, T_rank, d, f, E, k, "bf16", pl)
    grp.forward([to_device(x) for x in xs], [torch.from_numpy(l).cuda() for l in lgs])
    torch.cuda.synchronize()
    got = grp.received[0]
    dsps = [O.dispatch(xs[r], O.topk_gate(lgs[r], k)[0], pl, G) for r in range(G)]
    ex = O.exchange_to(dsps, pl, 0)
    np.testing.assert_array_equal(to_host(got["recv_buf"]).reshape(ex["recv_buf"].shape), ex["recv_buf"])
    for n in ("seg_expert", "seg_counts", "seg_start"):
        np.testing.assert_array_equal(got[n].cpu().numpy(), ex[n])
    rng = np.random.default_rng(0)
    pos = []
    for c, s in zip(ex["seg_counts"], ex["seg_start"]):
        if c:
            pos += [int(s), int(s + c - 1)] + (s + rng.integers(0, c, 6)).tolist()
    pos = np.unique(np.array(pos, dtype=np.int64))
    ref = O.expert_ffn_segments(ex["recv_buf"], *weights, ex["seg_expert"], ex["seg_counts"], ex["seg_start"], positions=pos)
    out = as_f64(to_host(got["out"][torch.from_numpy(pos).cuda()]))
    assert rel_err(out, ref[pos]) <= TOL_BF16
