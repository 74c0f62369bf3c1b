"""The plane-split matrix-core kernels at the sizes where they can go wrong: chunk and segment
edges, every tile form, the padded head size, exact scaling, non-finite inputs."""
import ctypes

import numpy as np
import pytest
import torch

from la_testlib import (TOL, excess, gpu_backward, gpu_backward_saved, gpu_forward,
                        gpu_forward_save, run_gpu, scratch, to_f64, upload_case)

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def la():
    import paper_2510_21956_amd as la
    la.load_library()
    return la



def _qknorm_forward(la, dev, a, b, causal):
    Q = dev["Q"]
    B, H, N, D = Q.shape
    dt = la.LA_F32 if Q.dtype == torch.float32 else la.LA_BF16
    O, G = torch.empty_like(Q), torch.empty((B, H, N), device="cuda")
    la.la_forward_qknorm(Q, dev["K"], dev["V"], O, G, a, b, causal,
                         scratch(la.la_workspace_bytes(B, H, N, D, dt, causal, 0), "cuda"))
    return O, G


def _qknorm_backward(la, dev, O, G, a, b, causal):
    Q = dev["Q"]
    B, H, N, D = Q.shape
    dt = la.LA_F32 if Q.dtype == torch.float32 else la.LA_BF16
    grads = [torch.empty_like(Q) for _ in range(3)]
    la.la_backward_qknorm(Q, dev["K"], dev["V"], O, G, dev["dO"], *grads, a, b, causal,
                          scratch(la.la_workspace_bytes(B, H, N, D, dt, causal, 1), "cuda"))
    return tuple(grads)


def _run_qknorm(la, dev, a, b, causal):
    O, G = _qknorm_forward(la, dev, a, b, causal)
    return (O, G) + _qknorm_backward(la, dev, O, G, a, b, causal)


# one row, either side of a chunk (32), of a segment of two chunks (64) and of three segments
@pytest.mark.parametrize("N", [1, 31, 33, 64, 65, 161])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("D", [16, 32, 64, 128])
def test_edges_against_plain_alu(la, D, dtype, N):
    """Every output against the plain-ALU kernels on the same inputs, masked and not, plain and
    normalising, both backward passes on the same O and g; the tolerance is the parity tests' own
    (twice, as both sides may use it up)."""
    dev, _ = upload_case(1, 2, N, D, dtype, 4200 + D + N, [0, 1])
    for causal in (True, False):
        for fwd, bwd in ((gpu_forward, gpu_backward), (_qknorm_forward, _qknorm_backward)):
            try:
                la.la_debug_override(64, 0)
                O, G = fwd(la, dev, 1.0, 0.5, causal)
                got = (O, G) + tuple(bwd(la, dev, O, G, 1.0, 0.5, causal))
                la.la_debug_override(64, 1)
                want = tuple(fwd(la, dev, 1.0, 0.5, causal)) + \
                    tuple(bwd(la, dev, O, G, 1.0, 0.5, causal))
            finally:
                la.la_debug_override(0, 0)
            for name, x, y in zip(("O", "G", "dQ", "dK", "dV"), got, want):
                # N = 1: dQ = dK = 0 exactly; rounding noise at the scale of V, dO ~ 1
                floor = 2 * TOL[dtype] if N == 1 and name in ("dQ", "dK") else 0.0
                e = excess(to_f64(x), to_f64(y), 2 * (TOL["f32"] if name == "G" else TOL[dtype]), floor)
                assert e <= 1.0, (D, dtype, N, causal, fwd.__name__, name, e)


# segments of an even and an odd number of chunks, the last chunk of 1 and of 31 rows; the rows with a
# second plane (132, 137, 260 of them) end inside a chunk
@pytest.mark.parametrize("N", [1057, 1103, 2080])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("D", [32, 64, 128])
def test_sweeps_over_many_chunks(la, D, dtype, N):
    """The sweeps of the backward pass on the kernels' own cuts, both handed-over and own sums, against the
    plain-ALU kernels on the same O and g; tolerance as above."""
    dev, _ = upload_case(1, 3, N, D, dtype, 5100 + D + N, [0])
    O, G, saved = gpu_forward_save(la, dev, 1.0, 0.5, True)
    got = (gpu_backward(la, dev, O, G, 1.0, 0.5, True),
           gpu_backward_saved(la, dev, O, G, saved, 1.0, 0.5, True))
    try:
        la.la_debug_override(0, 1)
        want = gpu_backward(la, dev, O, G, 1.0, 0.5, True)
    finally:
        la.la_debug_override(0, 0)
    for grads in got:
        for name, x, y in zip(("dQ", "dK", "dV"), grads, want):
            e = excess(to_f64(x), to_f64(y), 2 * TOL[dtype])
            assert e <= 1.0, (D, dtype, N, name, e)


@pytest.mark.parametrize("D,norm", [(16, False), (16, True), (32, True), (64, True), (128, True)])
@pytest.mark.parametrize("N", [1057, 1103])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_normalising_and_padded_sweeps_over_many_chunks(la, dtype, N, D, norm):
    """The same for the forms with factors per row and for head size 16: rows requested two chunks ahead and
    factors posted by one half of a workgroup come round several times a segment."""
    dev, _ = upload_case(1, 3, N, D, dtype, 5700 + D + N, [0], normalise=not norm)
    fwd, bwd = (_qknorm_forward, _qknorm_backward) if norm else (gpu_forward, gpu_backward)
    O, G = fwd(la, dev, 1.0, 0.5, True)
    got = bwd(la, dev, O, G, 1.0, 0.5, True)
    try:
        la.la_debug_override(0, 1)
        want = fwd(la, dev, 1.0, 0.5, True) + tuple(bwd(la, dev, O, G, 1.0, 0.5, True))
    finally:
        la.la_debug_override(0, 0)
    for name, x, y in zip(("O", "G", "dQ", "dK", "dV"), (O, G) + tuple(got), want):
        e = excess(to_f64(x), to_f64(y), 2 * (TOL["f32"] if name == "G" else TOL[dtype]))
        assert e <= 1.0, (D, dtype, N, norm, name, e)


@pytest.mark.parametrize("N", [33, 700])  # one segment, three
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_hand_over_at_head_size_256(la, dtype, causal, N):
    """The four passes' sums handed over: O, G as without, gradients within the parity tolerance of those on
    the backward pass's own sums (twice, as both may use it up).  Without a buffer, or with a short one,
    the pair is la_forward and la_backward to the bit."""
    dev, _ = upload_case(1, 3, N, 256, dtype, 6400 + N, [0])
    O, G, saved = gpu_forward_save(la, dev, 1.0, 0.5, causal)
    assert saved is not None
    O2, G2 = gpu_forward(la, dev, 1.0, 0.5, causal)
    assert torch.equal(O, O2) and torch.equal(G, G2)
    want = gpu_backward(la, dev, O, G, 1.0, 0.5, causal)
    for name, x, y in zip(("dQ", "dK", "dV"), gpu_backward_saved(la, dev, O, G, saved, 1.0, 0.5, causal), want):
        e = excess(to_f64(x), to_f64(y), 2 * TOL[dtype])
        assert e <= 1.0, (dtype, causal, N, name, e)
    for none in (None, saved[:256]):
        wf = scratch(la.la_workspace_bytes(1, 3, N, 256, la.LA_F32 if dtype == "f32" else la.LA_BF16, causal, 0),
                     "cuda")
        la.la_forward_save(dev["Q"], dev["K"], dev["V"], O2, G2, 1.0, 0.5, causal, wf, none)
        got = gpu_backward_saved(la, dev, O2, G2, none, 1.0, 0.5, causal)
        assert torch.equal(O, O2) and all(torch.equal(x, y) for x, y in zip(got, want))


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_sums_at_head_size_256_are_used_only_where_they_were_written(la, dtype, causal):
    """The forward call succeeds without a hand-over buffer, so the backward call may be given one that holds
    something else: memory no forward pass wrote, sums of other inputs, of the other mask.  Gradients are
    then those of la_backward to the bit, slice by slice; a buffer that does hold is read."""
    B, H, N, D = 1, 3, 700, 256
    code = la.LA_F32 if dtype == "f32" else la.LA_BF16
    dev, _ = upload_case(B, H, N, D, dtype, 6600, [0])
    other, _ = upload_case(B, H, N, D, dtype, 6601, [0])
    _, _, foreign = gpu_forward_save(la, other, 1.0, 0.5, causal)
    _, _, masked_otherwise = gpu_forward_save(la, dev, 1.0, 0.5, not causal)
    O, G = (torch.full_like(x, float("nan")) for x in gpu_forward(la, dev, 1.0, 0.5, causal))
    wf = scratch(la.la_workspace_bytes(B, H, N, D, code, causal, 0), "cuda")
    la.la_forward_save(dev["Q"], dev["K"], dev["V"], O, G, 1.0, 0.5, causal, wf, None)
    want = gpu_backward(la, dev, O, G, 1.0, 0.5, causal)
    for saved in (torch.zeros_like(foreign), torch.full_like(foreign, 0xFF), foreign, masked_otherwise):
        got = gpu_backward_saved(la, dev, O, G, saved, 1.0, 0.5, causal)
        assert all(torch.equal(x, y) for x, y in zip(got, want)), (dtype, causal)
    # one slice's inputs changed since: that slice as without, the others on the sums
    _, _, saved = gpu_forward_save(la, dev, 1.0, 0.5, causal)
    kept = gpu_backward_saved(la, dev, O, G, saved, 1.0, 0.5, causal)
    for n in ("Q", "K", "V"):
        dev[n][0, 1].copy_(other[n][0, 1])
    O, G = gpu_forward(la, dev, 1.0, 0.5, causal)
    want = gpu_backward(la, dev, O, G, 1.0, 0.5, causal)
    got = gpu_backward_saved(la, dev, O, G, saved, 1.0, 0.5, causal)
    for x, y, z in zip(got, want, kept):
        assert torch.equal(x[0, 1], y[0, 1]) and torch.equal(x[0, 0], z[0, 0]) and torch.equal(x[0, 2], z[0, 2])
    # the sums are read: poisoned ones show (the first slice's of the first of the four passes: three segments)
    saved[:3 * (128 * 128 + 128) * 4] = 0xFF
    got = gpu_backward_saved(la, dev, O, G, saved, 1.0, 0.5, causal)
    assert torch.isnan(got[0][0, 0].float()).any()


@pytest.mark.parametrize("handed", [True, False])
@pytest.mark.parametrize("causal", [True, False])
def test_trace_at_head_size_256_reaches_the_last_kernel(la, causal, handed):
    """Forward, backward and recomputing backward passes: every kernel in an entry, up to the last."""
    dev, _ = upload_case(1, 2, 700, 256, "f32", 6900, [0])
    O, G, saved = gpu_forward_save(la, dev, 1.0, 0.5, causal)
    grads = [torch.empty_like(O) for _ in range(3)]

    def names(call):
        events = [torch.cuda.Event(enable_timing=True) for _ in range(la.LA_MAX_TRACE + 4)]
        for e in events:
            e.record()
        tr = la.la_trace()
        tr.events = (ctypes.c_void_p * len(events))(*(e.cuda_event for e in events))
        tr.capacity = len(events)
        call(tr)
        torch.cuda.synchronize()
        assert tr.recorded - 1 <= la.LA_MAX_TRACE
        return [tr.names[k].decode() for k in range(tr.recorded - 1)]

    def ws(which):
        return scratch(la.la_workspace_bytes(1, 2, 700, 256, la.LA_F32, causal, which), "cuda")
    own = ["bwd_state", "scan_slots"]
    sums = ["check_witness", "bwd_state_scan"] if handed else own
    sweeps = ["bwd_dq", "bwd_dq", "scan_slots_rev", "bwd_dkv", "bwd_dkv"]
    args = dev["Q"], dev["K"], dev["V"]
    kept = saved if handed else None
    assert names(lambda tr: la.la_forward_save(*args, O, G, 1.0, 0.5, causal, ws(0), kept, None, tr)) == \
        ["fwd_state", "scan_slots", "fwd_apply", "fwd_apply"] + ["leave_witness"] * handed
    for again in (0, 1):
        og = (None, None) if again else (O, G)
        assert names(lambda tr: la.la_backward_saved(*args, *og, dev["dO"], *grads, 1.0, 0.5, causal, ws(1 + again), kept,
                                                     None, tr)) == ["fwd_again"] * again + sums + sweeps


@pytest.mark.parametrize("causal", [True, False])
def test_hand_over_at_head_size_256_in_a_graph(la, causal):
    """The pair captured once: every replay, on new inputs and with eager calls in between, gives the eager
    pair's bits; a replay of the backward pass alone on new inputs forms its own sums."""
    B, H, N, D = 1, 2, 700, 256
    draws = [upload_case(B, H, N, D, "bf16", 6800 + k, [0])[0] for k in range(3)]
    dev = {n: x.clone() for n, x in draws[0].items()}
    O, G, saved = gpu_forward_save(la, dev, 1.0, 0.5, causal)
    ws = [scratch(la.la_workspace_bytes(B, H, N, D, la.LA_BF16, causal, w), "cuda") for w in (0, 1)]
    grads = [torch.empty_like(O) for _ in range(3)]

    def forward():
        la.la_forward_save(dev["Q"], dev["K"], dev["V"], O, G, 1.0, 0.5, causal, ws[0], saved)

    def backward():
        la.la_backward_saved(dev["Q"], dev["K"], dev["V"], O, G, dev["dO"], *grads, 1.0, 0.5, causal, ws[1], saved)
    fwd, bwd = torch.cuda.CUDAGraph(), torch.cuda.CUDAGraph()
    for graph, call in ((fwd, forward), (bwd, backward)):
        with torch.cuda.graph(graph):
            call()
    for k in (1, 2, 0, 1):
        for n in dev:
            dev[n].copy_(draws[k][n])
        Oe, Ge, se = gpu_forward_save(la, dev, 1.0, 0.5, causal)
        own = gpu_backward(la, dev, Oe, Ge, 1.0, 0.5, causal)
        want = gpu_backward_saved(la, dev, Oe, Ge, se, 1.0, 0.5, causal)
        O.copy_(Oe)
        G.copy_(Ge)
        bwd.replay()
        assert all(torch.equal(x, y) for x, y in zip(grads, own)), (causal, k)
        O.zero_()
        fwd.replay()
        bwd.replay()
        assert torch.equal(O, Oe) and torch.equal(G, Ge)
        assert all(torch.equal(x, y) for x, y in zip(grads, want)), (causal, k)


def test_hand_over_buffer_that_overlaps_another_at_head_size_256(la):
    """Left unused by both calls, as any buffer was before there was a hand-over at this head size."""
    B, H, N, D = 1, 2, 700, 256
    dev, _ = upload_case(B, H, N, D, "f32", 6700, [0])
    args = dev["Q"], dev["K"], dev["V"]
    ns = la.la_saved_state_bytes(B, H, N, D, la.LA_F32, True)
    nb = [la.la_workspace_bytes(B, H, N, D, la.LA_F32, True, w) for w in (0, 1)]
    ws = scratch(max(nb) + ns, "cuda")
    O, G = gpu_forward(la, dev, 1.0, 0.5, True)
    want = gpu_backward(la, dev, O, G, 1.0, 0.5, True)
    O2, G2 = torch.empty_like(O), torch.empty_like(G)
    grads = [torch.empty_like(O) for _ in range(3)]
    for at in (0, nb[1] // 2 // 256 * 256):  # at the workspace's start and inside it
        la.la_forward_save(*args, O2, G2, 1.0, 0.5, True, ws[:nb[0]], ws[at:at + ns])
        la.la_backward_saved(*args, O2, G2, dev["dO"], *grads, 1.0, 0.5, True, ws[:nb[1]], ws[at:at + ns])
        assert torch.equal(O, O2) and torch.equal(G, G2)
        assert all(torch.equal(x, y) for x, y in zip(grads, want))


def test_descending_sums_lose_no_small_products(la):
    """bf16, D = 128, one segment: R starts at 2^23 with the last row, and every 16 rows add a product of 1/2,
    which an instruction that adds onto R cuts off and 32 rows on an accumulator of their own keep.  dK and
    dV of the first rows are the difference of two entries of R, one of them without the additions: exact but
    for the rounding of R's second plane and of the result, 2^-9 each."""
    N, D = 8192, 128
    big, i = 2.0 ** 12, torch.arange(0, N, 16, device="cuda")
    Q, K, V, dO = (torch.zeros((1, 1, N, D), device="cuda", dtype=torch.bfloat16) for _ in range(4))
    Q[0, 0, i, 0], dO[0, 0, i, 0] = 1.0, 0.5       # into R[0, 0] alone
    Q[0, 0, -1, :2], dO[0, 0, -1, :2] = big, big / 2   # 2^23 into R[0..1, 0..1]
    V[..., 0], V[..., 1] = 1.0, -1.0               # dK[:, 0] reads R[0, 0] - R[0, 1]
    K[..., 0], K[..., 1] = 1.0, -1.0               # dV[:, 0] reads R[0, 0] - R[1, 0]
    O, G = torch.zeros_like(Q), torch.ones((1, 1, N), device="cuda")
    try:
        la.la_debug_override(N, 0)
        dQ, dK, dV = gpu_backward(la, {"Q": Q, "K": K, "V": V, "dO": dO}, O, G, 0.0, 1.0, True)
    finally:
        la.la_debug_override(0, 0)
    want = 0.5 * torch.flip(torch.cumsum(torch.flip((torch.arange(N) % 16 == 0).double(), [0]), 0), [0])[:64]
    for name, x in (("dK", dK), ("dV", dV)):
        got = x[0, 0, :64, 0].double().cpu()
        assert (got - want).abs().max() <= want.max() * 2.0 ** -8, (name, got[0].item(), want[0].item())


@pytest.mark.parametrize("D", [64, 128])
def test_fp32_is_fp32(la, oracle_mod, D):
    """Six bf16 products a float product keep 24 bits: the 2-norm error against 64 bits stays at
    a few roundings of the running sums (N / 32 = 64 additions, sqrt(64) 2^-25 = 2.4e-7)."""
    N, slices = 2048, [0, 1]
    dev, ref = upload_case(1, 2, N, D, "f32", 77 + D, slices)
    O, G, dQ, dK, dV = run_gpu(la, dev, 1.0, 0.5, True)
    Or, Gr = oracle_mod.forward_rec(ref["Q"], ref["K"], ref["V"], 1.0, 0.5, True)
    want = (Or, Gr) + tuple(oracle_mod.backward_rec(ref["Q"], ref["K"], ref["V"], Or, Gr, ref["dO"],
                                                    1.0, 0.5, True))
    for name, x, y in zip(("O", "G", "dQ", "dK", "dV"), (O, G, dQ, dK, dV), want):
        x = to_f64(x).reshape(y.shape)
        e = np.linalg.norm(x - y) / np.linalg.norm(y)
        assert e <= 2.4e-7, (name, e)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_powers_of_two_scale_exactly(la, dtype):
    """V and dO enter linearly and every plane scales with its value, so a power of two goes
    through all kernels without touching a bit.  (From 2^-109 on the third plane is subnormal and
    bits are lost; sums of 200 rows of 4 sigma reach the largest float at 2^117.)"""
    dev, _ = upload_case(1, 2, 200, 64, dtype, 9, [0, 1])
    base = run_gpu(la, dev, 1.0, 0.5, True)
    for p in (-90, -60, 60, 110):
        s = 2.0 ** p
        d2 = dict(dev)
        d2["V"] = dev["V"] * s
        O, _, _, _, _ = run_gpu(la, d2, 1.0, 0.5, True)
        assert torch.equal(O, base[0] * s), ("O", p)
        d3 = dict(dev)
        d3["dO"] = dev["dO"] * s
        got = run_gpu(la, d3, 1.0, 0.5, True)
        for name, x, y in zip(("dQ", "dK", "dV"), got[2:], base[2:]):
            assert torch.equal(x, y * s), (name, p)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("D", [16, 64, 128])
def test_nonfinite_stays_in_its_column(la, D, dtype):
    """An infinity in one column of V reaches no other column of O, and in its own no chunk of 32 rows
    before its row's.  (The rows of that chunk before it meet it times the zeros above the diagonal.)"""
    dev, _ = upload_case(1, 1, 150, D, dtype, 31, [0])
    clean = run_gpu(la, dev, 1.0, 0.5, True)[0]
    V = dev["V"].clone()
    V[0, 0, 40, 5] = float("inf")
    O = run_gpu(la, dict(dev, V=V), 1.0, 0.5, True)[0]
    keep = [j for j in range(D) if j != 5]
    assert torch.equal(O[..., keep], clean[..., keep])
    assert torch.equal(O[0, 0, :32, 5], clean[0, 0, :32, 5])
    assert not torch.isfinite(O[0, 0, 40:, 5].float()).any()


def test_static_forward_head_size_16_many_slices(la):
    """8000 slices at D = 16: the padded tiles' states exceed the static scratch, the plain-ALU
    kernels' fit, and the call is served as it was."""
    B, H, N, D = 80, 100, 6, 16
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)
    Q, K, V = (torch.randn((B, H, N, D), device="cuda", generator=gen) * 0.25 for _ in range(3))
    assert la.la_workspace_bytes(B, H, N, D, la.LA_F32, True, 0) > la.LA_STATIC_SCRATCH_BYTES
    O, G = torch.empty_like(Q), torch.empty((B, H, N), device="cuda")
    la.la_forward_static(Q, K, V, O, G, 1.0, 0.5, True)
    P = torch.tril(1.0 + 0.5 * torch.matmul(Q.double(), K.double().transpose(2, 3).contiguous()))
    want = torch.matmul(P, V.double()) / P.sum(3, keepdim=True)
    assert excess(to_f64(O), to_f64(want), TOL["f32"]) <= 1.0
    assert excess(to_f64(G), to_f64(P.sum(3)), TOL["f32"]) <= 1.0


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("N", [250, 4000])
def test_head_size_16_bf16_has_32_bit_intermediates(la, N, causal):
    """bf16 at D = 16: nothing but the outputs is rounded to bf16, so that on the same O and g they
    are the plain-ALU kernels' but for values that lie within a few fp32 roundings of a tie.
    Two fp32 evaluations differ by some 1e-6 of a value (ten times that in dQ, dK, which are
    differences); a bf16 interval is 2^-8 of it, so well under 1 % of the values fall on either
    side of a tie.  An intermediate in one bf16 plane makes it 5 to 50 %."""
    dev, _ = upload_case(1, 4, N, 16, "bf16", 77, [])
    try:
        O, G = gpu_forward(la, dev, 1.0, 0.5, causal)
        got = (O,) + gpu_backward(la, dev, O, G, 1.0, 0.5, causal)
        la.la_debug_override(0, 1)
        want = (gpu_forward(la, dev, 1.0, 0.5, causal)[0],) + gpu_backward(la, dev, O, G, 1.0, 0.5,
                                                                          causal)
    finally:
        la.la_debug_override(0, 0)
    for name, x, y in zip(("O", "dQ", "dK", "dV"), got, want):
        share = float((x != y).float().mean())
        assert share <= 0.01, (name, share)


@pytest.mark.parametrize("p", [-68, 58])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("D", [16, 32, 64, 128])
def test_qknorm_takes_any_row_length(la, D, dtype, p):
    """Rows of Q and K scaled by a power of two: the same O, g and dV, dQ and dK scaled back.  At
    2^-68 a row's squared length is subnormal (2^-134 D, in steps of 2^-149: 2^-11 at worst, far
    below the bf16 tolerance; the fp32 rows are scaled by 2^-60, where it is not)."""
    if dtype == "f32":
        p = max(p, -60)
    dev, _ = upload_case(1, 2, 200, D, dtype, 9, [0, 1], normalise=False)
    base = _run_qknorm(la, dev, 1.0, 0.5, True)
    s = 2.0 ** p
    got = _run_qknorm(la, dict(dev, Q=dev["Q"] * s, K=dev["K"] * s), 1.0, 0.5, True)
    for name, x, y in zip(("O", "G", "dQ", "dK", "dV"), got, base):
        x = to_f64(x) * (s if name in ("dQ", "dK") else 1.0)
        assert excess(x, to_f64(y), TOL[dtype]) <= 1.0, (name, p)


@pytest.mark.parametrize("sign", [1.0, -1.0])
@pytest.mark.parametrize("D", [16, 32, 64, 128])
def test_fp32_infinity_keeps_its_sign(la, D, sign):
    """An infinite value of row 40 is +-infinity in rows 40 to 63 of O, the rest of its chunk, where
    every weight 1 + 0.5 q.k is positive, and it spoils the later rows of its column.  (D = 256 adds
    the weight up from two halves of either sign.)"""
    dev, _ = upload_case(1, 1, 150, D, "f32", 31, [0])
    V = dev["V"].clone()
    V[0, 0, 40, 5] = sign * float("inf")
    O = run_gpu(la, dict(dev, V=V), 1.0, 0.5, True)[0][0, 0, :, 5]
    assert torch.isfinite(O[:32]).all()
    assert (O[40:64] == sign * float("inf")).all()
    assert not torch.isfinite(O[64:]).any()


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("D", [16, 32, 64, 128, 256])
def test_largest_floats(la, D, causal):
    """A float that no bf16 reaches (3.4e38; the last bf16 is 3.39e38, and from 3.396e38 on a float
    rounds to infinity) in V and in dO, with weights a = 1/4: o_i is the mean of the rows it sees,
    dv_n the sum of dO_i / (their number) over the rows that see it."""
    N, top = 150, 3.4e38
    dev, _ = upload_case(1, 1, N, D, "f32", 32, [0])
    V = dev["V"] * 0.01
    V[0, 0, 40, 5] = -top
    O, _, _, _, _ = run_gpu(la, dict(dev, V=V), 0.25, 0.0, causal)
    n = torch.arange(1, N + 1, device="cuda", dtype=torch.float64)
    want = V[0, 0].double().cumsum(0) / n[:, None] if causal else V[0, 0].double().mean(0).expand(N, D)
    keep = torch.arange(N, device="cuda") >= (40 if causal else 0)  # rows that see row 40
    assert excess(to_f64(O[0, 0, keep, 5]), to_f64(want[keep, 5]), TOL["f32"]) <= 1.0

    V, dO = dev["V"] * 0.01, dev["dO"].clone()
    dO[0, 0, 40, 5] = top
    dV = run_gpu(la, dict(dev, V=V, dO=dO), 0.25, 0.0, causal)[4]
    x = dO[0, 0].double() / (n if causal else float(N) * torch.ones_like(n))[:, None]
    want = x.flip(0).cumsum(0).flip(0) if causal else x.sum(0).expand(N, D)
    keep = torch.arange(N, device="cuda") <= (40 if causal else N)
    assert excess(to_f64(dV[0, 0, keep, 5]), to_f64(want[keep, 5]), TOL["f32"]) <= 1.0


@pytest.mark.parametrize("D", [32, 64, 128])
def test_unmasked_sums_keep_24_bits(la, oracle_mod, D):
    """Without the mask O is mostly p / N and dV mostly w, sums over all rows: they carry what
    their additions lose, so that what is left are the roundings of p, of the two terms, their sum,
    1/g and the product: five of 2^-24 / sqrt(3) rms at most, 7.7e-8 (plain sums: 2.3e-7 to 2.9e-7)."""
    N, slices = 20000, [0, 1, 2, 3]
    dev, ref = upload_case(1, 4, N, D, "f32", 770 + D, slices)
    O, G, _, _, dV = run_gpu(la, dev, 1.0, 0.5, False)
    Or, Gr = oracle_mod.forward_rec(ref["Q"], ref["K"], ref["V"], 1.0, 0.5, False)
    dVr = oracle_mod.backward_rec(ref["Q"], ref["K"], ref["V"], Or, Gr, ref["dO"], 1.0, 0.5, False)[2]
    for name, x, y in (("O", O, Or), ("dV", dV, dVr)):
        e = np.linalg.norm(to_f64(x).reshape(y.shape) - y) / np.linalg.norm(y)
        assert e <= 7.7e-8, (name, e)


def test_prefill_sums_bf16(la):
    """The state after a bf16 prompt: every product is exact in fp32, and a segment's S takes one
    rounded addition per 64 rows, here 64 of them.  A sum of n like terms grows as sqrt(i), so its n
    roundings (2^-24 / sqrt(3) rms of the sum then held) come to sqrt(n / 2) 3.4e-8 = 1.9e-7 of it at
    the end; the rows within an instruction add half as much."""
    B, H, N, D = 16, 16, 4096, 128
    gen = torch.Generator(device="cuda")
    gen.manual_seed(8)
    K, V = (torch.randn((B, H, N, D), device="cuda", generator=gen).bfloat16() for _ in range(2))
    state = torch.zeros((B * H, la.la_decode_state_bytes(B, H, D) // 4 // (B * H)), device="cuda")
    la.la_decode_prefill(K, V, state, 0,
                         scratch(la.la_workspace_bytes(B, H, N, D, la.LA_BF16, False, 0), "cuda"))
    k, v, st = K[0].double(), V[0].double(), state[:H].double()
    want = {"S": torch.matmul(k.transpose(1, 2).contiguous(), v).reshape(H, -1), "z": k.sum(1), "p": v.sum(1)}
    got = {"S": st[:, :D * D], "z": st[:, D * D:D * D + D], "p": st[:, D * D + D:D * D + 2 * D]}
    for name, bound in (("S", 2.1e-7), ("z", 6e-8), ("p", 6e-8)):
        e = float((got[name] - want[name]).norm() / want[name].norm())
        assert e <= bound, (name, e)


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("norm", [False, True])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("D", [16, 32, 64, 128])
def test_runs_are_bitwise_alike(la, D, dtype, norm, causal):
    """Several runs on the same inputs, every mode of the kernels: the same bits each time."""
    dev, _ = upload_case(2, 3, 1100, D, dtype, 99 + D, [])
    run = _run_qknorm if norm else run_gpu
    first = run(la, dev, 1.0, 0.5, causal)
    for _ in range(4):
        for name, x, y in zip(("O", "G", "dQ", "dK", "dV"), run(la, dev, 1.0, 0.5, causal), first):
            assert torch.equal(x, y), name


# evened-out segments (D = 64); four, two and one workgroup a CU for the rows (D = 128); more slices
# than compute units
@pytest.mark.parametrize("B,H,N,D", [(8, 24, 1000, 64), (8, 24, 900, 128), (4, 20, 1000, 128),
                                     (8, 24, 300, 128), (32, 32, 70, 32)])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_unmasked_cuts(la, B, H, N, D, dtype):
    """Without the mask the rows of the forward pass are cut by a rule of their own: every row is
    written, and the sums handed over serve the backward pass like recomputed ones."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(B * N + D)
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    dev = {n: (torch.randn((B, H, N, D), device="cuda", generator=gen) * sc).to(td)
           for n, sc in (("Q", D ** -0.5), ("K", D ** -0.5), ("V", 1.0), ("dO", 1.0))}
    O, G, saved = gpu_forward_save(la, dev, 1.0, 0.5, False)
    q, k, v = (dev[n].double() for n in ("Q", "K", "V"))
    S = torch.matmul(k.transpose(2, 3).contiguous(), v)
    g = N + 0.5 * torch.matmul(q, k.sum(2).unsqueeze(3)).squeeze(3)
    want = (v.sum(2, keepdim=True) + 0.5 * torch.matmul(q, S)) / g.unsqueeze(3)
    assert excess(to_f64(O), to_f64(want), TOL[dtype]) <= 1.0
    assert excess(to_f64(G), to_f64(g), TOL["f32"]) <= 1.0
    got = gpu_backward_saved(la, dev, O, G, saved, 1.0, 0.5, False)
    for x, y in zip(got, gpu_backward(la, dev, O, G, 1.0, 0.5, False)):
        assert excess(to_f64(x), to_f64(y), TOL[dtype]) <= 1.0


# K and V beyond the last-level cache (256 MB): the sums of 32-row chunks, with a ragged last one, in three segments
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("D", [16, 32, 64, 128])
def test_sums_of_large_tensors(la, D, dtype):
    """The last slices of a problem whose K and V exceed the last-level cache come out as they do by themselves, bit by
    bit in segments of the same length: passes with and without the mask, plain and normalising, and prompt states."""
    N, (td, dt) = 3001, (torch.float32, la.LA_F32) if dtype == "f32" else (torch.bfloat16, la.LA_BF16)
    H = (256 << 20) // (2 * td.itemsize * N * D) + 1
    gen = torch.Generator(device="cuda")
    gen.manual_seed(D)
    big = {n: torch.randn((1, H, N, D), device="cuda", generator=gen).to(td) for n in ("Q", "K", "V", "dO")}
    for n in "QK":
        big[n] *= D ** -0.5
    own = {n: x[:, -2:].contiguous() for n, x in big.items()}
    la.la_debug_override(1024, 0)
    try:
        for causal in (True, False):
            for fwd, bwd in ((gpu_forward, gpu_backward), (_qknorm_forward, _qknorm_backward)):
                got, want = fwd(la, big, 1.0, 0.5, causal), fwd(la, own, 1.0, 0.5, causal)
                got += bwd(la, big, *got, 1.0, 0.5, causal)
                want += bwd(la, own, *want, 1.0, 0.5, causal)
                for name, x, y in zip(("O", "G", "dQ", "dK", "dV"), got, want):
                    assert torch.equal(x[:, -2:], y), (D, dtype, causal, fwd.__name__, name)
        states = []
        for x in (big, own):
            h = x["K"].shape[1]
            states.append(torch.zeros(la.la_decode_state_bytes(1, h, D) // 4, device="cuda"))  # has padding
            la.la_decode_prefill(x["K"], x["V"], states[-1], 0,
                                 scratch(la.la_workspace_bytes(1, h, N, D, dt, 0, 0), "cuda"))
        assert torch.equal(states[0][-states[1].numel():], states[1])
    finally:
        la.la_debug_override(0, 0)
