"""moe_layer_forward against the four calls it stands for, bit for bit: every size where its merged kernels can go
wrong (one token, a token per workgroup and more, slices of the in-workgroup sort, the last sizes of the fused front
and of the decode-sized combine and the first ones past them), each lane layout of the gate, ragged expert counts."""
import numpy as np
import pytest
import torch

from paper_2502_06643_amd import binding as B
from paper_2502_06643_amd import synth
from paper_2502_06643_amd.layer import MoELayer, to_device

pytestmark = pytest.mark.gpu

OUTPUTS = ("topk_idx", "topk_w", "send_buf", "perm", "inv_perm", "expert_counts", "expert_start", "gpu_counts", "gpu_offsets", "ffn_out", "y")


@pytest.mark.parametrize("dtype,T,d,f,E,k,G,local", [
    ("bf16", 1, 64, 64, 8, 2, 1, -1),
    ("bf16", 80, 1088, 128, 8, 2, 4, 2),          # 160 routes: the last decode-sized batch, columns past a workgroup's 1024
    ("bf16", 81, 64, 128, 8, 2, 4, 2),            # the first one past it
    ("bf16", 10, 128, 64, 256, 16, 8, 3),         # 16 lanes per token, 16 routes per token
    ("bf16", 255, 64, 64, 5, 3, 2, 1),            # logit rows that are no multiple of 16 bytes
    ("bf16", 257, 64, 64, 64, 6, 8, 7),           # past the fused front (FUSED_FRONT below has its edges): gate and index kernels
    ("bf16", 2048, 64, 64, 64, 6, 8, 0),
    ("bf16", 2049, 64, 64, 64, 6, 8, 0),
    ("bf16", 6144, 4096, 64, 8, 2, 1, -1),        # rows of 8 KB
    ("bf16", 512, 64, 64, 200, 1, 3, -1),         # 16 lanes per token
    ("bf16", 8192, 64, 64, 3, 1, 1, -1),
    ("bf16", 8193, 64, 64, 3, 2, 2, 1),           # the plan comes from the one-workgroup index kernel: 16386 routes are past it, ...
    ("bf16", 8192, 64, 64, 100, 2, 5, 1),         # ... 16384 the last
    ("bf16", 20000, 64, 64, 256, 2, 256, 255),    # ... and from the rank kernel, widest tables
    ("bf16", 87381, 64, 64, 64, 6, 1, -1),        # 256 chunks of two steps and the plan: more workgroups than compute units, ...
    ("bf16", 262144, 64, 64, 16, 2, 1, -1),       # ... with ranks counted in lanes
    ("bf16", 100000, 64, 64, 33, 4, 2, 1),        # 196 of them
    ("f32", 9000, 16, 16, 8, 2, 1, -1),
    ("f32", 1, 4, 4, 1, 1, 1, -1),
    ("f32", 256, 128, 256, 8, 2, 4, 0),
    ("f32", 1025, 36, 100, 9, 2, 2, 1),
])
def test_forward_equals_the_four_calls(lib, dtype, T, d, f, E, k, G, local):
    check_forward(dtype, T, d, f, E, k, G, local)


FUSED_FRONT = [  # the last sizes of the fused front and the first ones past it
    ((257, 64, 8, 2, 4, 1), True),                # one workgroup owns two tokens
    ((256, 64, 64, 6, 8, 7), True), ((257, 64, 64, 6, 8, 7), False),            # one gate pass of 4 lanes per token
    ((512, 64, 33, 2, 2, 0), True), ((513, 64, 33, 2, 2, 0), False),            # two of them up to top-2
    ((64, 64, 256, 16, 8, 3), True), ((65, 64, 256, 16, 8, 3), False),          # 16 lanes per token
    ((128, 64, 200, 1, 3, -1), True), ((129, 64, 200, 1, 3, -1), False),
    ((6144, 1024, 8, 2, 1, -1), True), ((6145, 64, 8, 1, 1, -1), False),        # six passes of one lane; 25 tokens per workgroup, more rows than are prefetched
    ((4608, 4096, 8, 2, 1, -1), True), ((4609, 4096, 8, 2, 1, -1), False),      # 72 MB of rows
    ((1536, 64, 8, 8, 2, 1), True), ((1537, 64, 8, 8, 2, 1), False),            # 12288 routes
]


@pytest.mark.parametrize("shape,fused", FUSED_FRONT)
def test_where_the_front_is_fused(lib, shape, fused):
    T, d, E, k, G, local = shape
    B.moe_timing_begin(1 << B.KERNEL_NAMES.index("front"), 64)
    check_forward("bf16", T, d, 64, E, k, G, local)
    assert B.moe_timing_end()[1]["front"] == (2 if fused else 0)


@pytest.mark.parametrize("T,E,k", [(100, 8, 2), (9000, 8, 2), (20000, 256, 2)])      # fused front, histograms of one tile and of 40 KB
def test_one_buffer_for_both_workspaces(lib, T, E, k):
    check_forward("bf16", T, 64, 64, E, k, 4, 1, one_workspace=True)


@pytest.mark.parametrize("T,d,f,E,k,G,local,up,down", [
    (2700, 4096, 512, 16, 6, 8, 0, True, False),        # one workgroup's index kernel; the up projection takes all
    (9000, 2048, 1024, 32, 4, 4, 1, True, True),        # rank kernel; both projections take some
    (11001, 1344, 256, 16, 4, 4, 1, True, False),       # 168 pieces a row
    (4000, 4096, 512, 32, 3, 8, 3, True, False),        # 512 pieces a row
    (2750, 4096, 2048, 16, 4, 16, 2, True, False),      # the down projection's tiles are cut along k
    (2100, 1280, 64, 16, 16, 200, 199, True, False),    # no expert here, 16 routes per token
    (26000, 1280, 64, 32, 4, 8, 0, True, True),         # more than they can take
    (8192, 2048, 1408, 64, 6, 8, 5, False, False),      # tiles on more than three quarters of the compute units
    (14000, 2048, 384, 8, 3, 2, 0, False, False),       # on nearly all
    (12000, 1216, 512, 16, 4, 4, 0, None, None),        # reductions too short to ask
    (14000, 2048, 512, 16, 2, 4, 0, None, None),        # two routes a token
    (2700, 2048, 1408, 64, 6, 8, 0, None, None),        # few rows
])
def test_rows_copied_beside_the_projections(lib, T, d, f, E, k, G, local, up, down):
    plan = check_forward("bf16", T, d, f, E, k, G, local).ffn_ws[:64].view(torch.int32).cpu()
    if up is not None:                             # what the plan leaves to the two projections
        assert (int(plan[8]) > 0) == up and (int(plan[9]) > 0) == down and int(plan[8]) + int(plan[9]) <= T
    else:                                          # nobody has asked
        assert plan[8:12].tolist() == [0x03030303] * 4


def test_rows_copied_beside_the_projections_of_experts_mapped_nowhere(lib):
    """Experts on GPUs that do not exist come first and last in the sorted order; their rows are copied like any other GPU's."""
    pl = np.array([3, -1, 1, 4, 0, -7, 2, 1, 100, 0, 1, 3, 2, -1, 2, 4], dtype=np.int32)
    plan = check_forward("bf16", 4500, 2048, 512, 16, 6, 4, 1, placement=pl).ffn_ws[:64].view(torch.int32).cpu()
    assert int(plan[8]) > 0 and int(plan[10]) > 0


@pytest.mark.parametrize("shared", ["x and ffn_out", "x and H", "inv_perm and H", "send_buf and ffn_out, shifted", "send_buf is ffn_out",
                                    "perm and send_buf"])
def test_outputs_in_the_memory_of_the_inputs(lib, shared):
    """Memory that the four calls may share, because each has read it when the next writes it, or writes other rows of it: the same
    results, and nobody asks the projections to copy rows (but for the send buffer as ffn_out).  In a call with memory of its own
    for everything both of them copy rows that lie under what they write here."""
    T, d, f, E, k, G, local = 6000, 2048, 896, 32, 6, 4, 0
    N, row = T * k, d * 2
    rng = np.random.default_rng(T + E)
    pl = (np.arange(E) * G // E).astype(np.int32)
    x = to_device(synth.normal(T, 0, (T, d), 1.0, "bf16"))
    lg = torch.from_numpy(rng.standard_normal((T, E)).astype(np.float32)).cuda()
    w = [to_device(synth.normal(T, i, s, s[1] ** -0.5, "bf16")) for i, s in ((2, (E, d, f)), (3, (E, d, f)), (4, (E, f, d)))]
    got, want = (MoELayer(T, d, f, E, k, G, local, "bf16") for _ in range(2))
    for L in (got, want):
        L.set_placement(pl)
        L.set_weights(*w)
    want.forward(x, lg)
    up, down, begin, end = want.ffn_ws[:64].view(torch.int32).cpu().tolist()[8:12]
    assert up > 0 and down > 0 and begin == 0 and end > up + 1000      # this GPU's rows come first
    send = want.send_buf.clone()
    got.ffn_ws.fill_(3)
    if shared == "x and ffn_out":                  # rows of x from `up` on lie under the down projection's
        got.ffn_out[:T].copy_(x)
        xs = got.ffn_out[:T]
    elif shared == "x and H":                      # the first ones lie under the up projection's (H follows the plan's 8192 bytes)
        xs = got.ffn_ws[8192:8192 + T * row].view(torch.bfloat16).view(T, d)
        xs.copy_(x)
    elif shared == "inv_perm and H":               # under the rows of other GPUs, which the up projection leaves alone
        at = 8192 + (end * f * 2 + 255) // 256 * 256
        got.inv_perm, xs = got.ffn_ws[at:at + N * 4].view(torch.int32), x
    elif shared == "perm and send_buf":            # a sorted order that nobody wants, under this GPU's rows
        got.perm, xs = got.send_buf.view(-1)[:2 * N].view(torch.int32), x
    else:                                          # the down projection's rows where other GPUs' send rows, or its own, are
        shift = end if shared.endswith("shifted") else 0
        memory = torch.zeros((N + shift, d), dtype=torch.bfloat16, device="cuda")
        got.send_buf, got.ffn_out, xs = memory[:N], memory[shift:], x
        send[shift:shift + end] = want.ffn_out[:end]
    got.forward(xs, lg)
    torch.cuda.synchronize()
    assert torch.equal(got.y, want.y) and torch.equal(got.send_buf, send)
    asked = got.ffn_ws[:64].view(torch.int32).cpu().tolist()[8:12] != [0x03030303] * 4
    assert asked == (shared == "send_buf is ffn_out")


@pytest.mark.parametrize("T,E,k,G,local", [
    (800, 8, 2, 1, -1), (3000, 8, 2, 1, -1), (5000, 8, 2, 2, 1),           # written by the front; more and fewer buckets of one row tile
    (900, 128, 4, 1, -1), (1300, 16, 4, 1, -1), (2103, 32, 2, 2, 0), (700, 256, 4, 3, 1),        # by the one-workgroup index kernel
    (8000, 64, 6, 1, -1), (9000, 8, 2, 1, -1), (20000, 256, 2, 1, -1),     # by the rank kernel
])
def test_tiles_counted_by_the_plan(lib, T, E, k, G, local):
    """The plan's header: row tiles of 256, those of at most 128 rows, and those of buckets of several tiles if the buckets of one are
    at least as many (else 0)."""
    L = check_forward("bf16", T, 64, 64, E, k, G, local)
    counts = L.expert_counts.cpu().numpy()
    if local >= 0:
        counts = counts[L.placement.cpu().numpy() == local]
    counts = counts[counts > 0]
    tiles, single = -(-counts // 256), int((counts <= 256).sum())
    plan = L.ffn_ws[:64].view(torch.int32).cpu().tolist()
    assert plan[0] == len(counts) and plan[2] == tiles.sum()
    assert plan[4] == 1 + ((counts - 1) % 256 < 128).sum()
    assert plan[12] == (tiles.sum() - single if 2 * single >= tiles.sum() else 0)


def check_forward(dtype, T, d, f, E, k, G, local, one_workspace=False, placement=None):
    rng = np.random.default_rng(T + E)
    pl = rng.integers(0, G, E).astype(np.int32) if placement is None else placement
    x = to_device(synth.normal(T, 0, (T, d), 1.0, dtype))
    lg = rng.standard_normal((T, E)).astype(np.float32)
    lg[T // 2] = np.round(lg[T // 2])              # ties
    lg = torch.from_numpy(lg - np.log(np.arange(1, E + 1)).astype(np.float32)[None, :]).cuda()
    w = [to_device(synth.normal(T, i, s, s[1] ** -0.5, dtype)) for i, s in ((2, (E, d, f)), (3, (E, d, f)), (4, (E, f, d)))]
    got, want = (MoELayer(T, d, f, E, k, G, local, dtype) for _ in range(2))
    for L in (got, want):
        L.set_placement(pl)
        L.set_weights(*w)
        for n in OUTPUTS:
            getattr(L, n).fill_(3)                 # what a call leaves untouched must be the same too
    got.ffn_ws.fill_(3)
    if one_workspace:
        got.dispatch_ws = got.ffn_ws
    want.gate(lg)
    want.dispatch(x)
    want.ffn()
    want.combine()
    for rep in range(2):                           # the second call finds the first one's workspaces
        got.forward(x, lg)
        torch.cuda.synchronize()
        for n in OUTPUTS:
            a, b = (getattr(L, n).reshape(-1).view(torch.uint8) for L in (got, want))
            assert torch.equal(a, b), f"call {rep}: {n}"
    return got


def test_forward_reports_bad_arguments(lib):
    L = MoELayer(4, 64, 64, 8, 2, 1, -1, "bf16")
    L.set_placement(np.zeros(8, dtype=np.int32))
    L.set_weights(*[torch.zeros(s, dtype=torch.bfloat16, device="cuda") for s in ((8, 64, 64),) * 3])
    x, lg = torch.zeros((4, 64), dtype=torch.bfloat16, device="cuda"), torch.zeros((4, 8), device="cuda")
    with pytest.raises(ValueError):
        L.forward(x.t(), lg)
    with pytest.raises(B.MoeError):
        L.forward(None, lg)
    L.ffn_ws = L.ffn_ws[:256]
    with pytest.raises(B.MoeError):
        L.forward(x, lg)
