"""GPU parity of the incremental (decode) entry points against the oracle's incremental form
(App. B.1), which the CPU tests pin to the definition."""
import numpy as np
import pytest
import torch

import la_workloads as wl
from la_testlib import TOL, excess, scratch, to_device, to_f64, torch_dtype

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def la():
    import paper_2510_21956_amd as la_mod
    la_mod.load_library()
    assert torch.cuda.is_available()
    la_mod.la_debug_override(0, 0)
    return la_mod


def draw(BH, N, D, dtype, seed):
    bits = {n: [] for n in ("Q", "K", "V")}
    vals = {n: [] for n in ("Q", "K", "V")}
    for s in range(BH):
        sl = wl.make_slice(N, D, dtype, seed, s)
        for n in bits:
            bits[n].append(sl[n][0])
            vals[n].append(sl[n][1])
    dev = {n: to_device(np.stack(bits[n]), dtype) for n in bits}
    ref = {n: np.stack(vals[n]) for n in vals}
    return dev, ref


def canonical_state(state, BH, D):
    """[S | z | p | count] of every slice from the library's padded state."""
    return to_f64(state.view(BH, -1)[:, :D * D + 2 * D + 1])


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("D", [16, 32, 64, 128, 256])
def test_decode_steps(oracle_mod, la, D, dtype):
    """A sequence fed in pieces of 1, 5, 1, 2, ... rows with the state carried over: every
    output row and the final state against the oracle; a = 1, b = 0.5 and a = 2, b = -0.7."""
    B, H = 2, 3
    BH = B * H
    steps = [1, 5, 1, 2, 16, 1, 7]
    N = sum(steps)
    tol = TOL[dtype]
    td = torch_dtype(dtype)
    dev, ref = draw(BH, N, D, dtype, 600 + D)
    for a, b in ((1.0, 0.5), (2.0, -0.7)):
        print("case decode D=%d %s a=%g b=%g" % (D, dtype, a, b), flush=True)
        state = torch.zeros(la.la_decode_state_bytes(B, H, D) // 4, dtype=torch.float32,
                            device="cuda")
        st_ref = np.zeros((BH, oracle_mod.decode_state_floats(D)))
        at = 0
        for T in steps:
            q, k, v = (dev[n][:, at:at + T].reshape(B, H, T, D).contiguous() for n in "QKV")
            o = torch.full((B, H, T, D), float("nan"), dtype=td, device="cuda")
            g = torch.full((B, H, T), float("nan"), dtype=torch.float32, device="cuda")
            la.la_decode_step(q, k, v, o, g, state, a, b)
            torch.cuda.synchronize()
            o_ref, g_ref = oracle_mod.decode(ref["Q"][:, at:at + T], ref["K"][:, at:at + T],
                                             ref["V"][:, at:at + T], st_ref, a, b)
            eo = excess(to_f64(o.reshape(BH, T, D)), o_ref, tol)
            eg = excess(to_f64(g.reshape(BH, T)), g_ref, TOL["f32"])
            assert eo <= 1.0 and eg <= 1.0, (at, T, eo, eg)
            at += T
        # the state is float32 whatever the I/O type
        es = excess(canonical_state(state, BH, D), st_ref, TOL["f32"])
        print("  final state excess", round(es, 4), flush=True)
        assert es <= 1.0


@pytest.mark.parametrize("dtype,D,N0", [("f32", 64, 700), ("bf16", 128, 1000), ("f32", 32, 300),
                                        ("f32", 256, 700), ("bf16", 256, 400)])
def test_prefill_then_decode(oracle_mod, la, dtype, D, N0):
    """la_decode_prefill over a prompt (in two parts, the second accumulated), then single
    decode steps: outputs must equal the rows of the causal forward pass over the whole
    sequence (oracle: running sums), and la_forward's own rows on the GPU within tolerance."""
    B, H, extra = 1, 4, 6
    BH, N = B * H, N0 + extra
    tol = TOL[dtype]
    td = torch_dtype(dtype)
    dev, ref = draw(BH, N, D, dtype, 900 + D)
    a, b = 1.0, 0.5
    dt = la.LA_F32 if dtype == "f32" else la.LA_BF16
    state = torch.full((la.la_decode_state_bytes(B, H, D) // 4,), float("nan"),
                       dtype=torch.float32, device="cuda")
    cut = 192  # first part: overwrite; second part: accumulate
    for lo, hi, acc in ((0, cut, 0), (cut, N0, 1)):
        K = dev["K"][:, lo:hi].reshape(B, H, hi - lo, D).contiguous()
        V = dev["V"][:, lo:hi].reshape(B, H, hi - lo, D).contiguous()
        ws = scratch(la.la_workspace_bytes(B, H, hi - lo, D, dt, 0, 0), "cuda")
        la.la_decode_prefill(K, V, state, acc, ws)
    O_ref, G_ref = oracle_mod.forward_rec(ref["Q"], ref["K"], ref["V"], a, b, True)
    for t in range(N0, N):
        q, k, v = (dev[n][:, t:t + 1].reshape(B, H, 1, D).contiguous() for n in "QKV")
        o = torch.full((B, H, 1, D), float("nan"), dtype=td, device="cuda")
        g = torch.full((B, H, 1), float("nan"), dtype=torch.float32, device="cuda")
        la.la_decode_step(q, k, v, o, g, state, a, b)
        torch.cuda.synchronize()
        eo = excess(to_f64(o.reshape(BH, D)), O_ref[:, t], tol)
        eg = excess(to_f64(g.reshape(BH)), G_ref[:, t], TOL["f32"])
        print("prefill+decode", dtype, D, "row", t, round(eo, 4), round(eg, 4), flush=True)
        assert eo <= 1.0 and eg <= 1.0


def test_decode_argument_errors(la):
    B, H, T, D = 1, 2, 1, 64
    q = torch.zeros((B, H, T, D), device="cuda")
    st = torch.zeros(la.la_decode_state_bytes(B, H, D) // 4, device="cuda")
    with pytest.raises(la.LaError) as e:
        la.la_decode_step(q, q.clone(), q.clone(), q.clone(), None, st[:64], 1.0, 0.5)
    assert e.value.code == 5
    with pytest.raises(la.LaError) as e:
        la.la_decode_step(q, q.clone(), q.clone(), q, None, st, 1.0, 0.5)
    assert e.value.code == 7
    q48 = torch.zeros((B, H, T, 48), device="cuda")
    with pytest.raises(la.LaError) as e:
        la.la_decode_step(q48, q48.clone(), q48.clone(), q48.clone(), None, st, 1.0, 0.5)
    assert e.value.code == 3
    assert la.la_decode_state_bytes(1, 1, 48) == 0


# one slot a slice, a batch of sixteen and one more, either side of the change to runs of slots (5 at 33, the last one
# empty), more than a batch in a run
@pytest.mark.parametrize("nseg", [1, 16, 17, 32, 33, 50, 259])
@pytest.mark.parametrize("D", [16, 64, 256])
def test_prefill_adds_any_number_of_slots(la, D, nseg):
    B, H, N = 1, 2, 64 * nseg - 3
    dev, ref = draw(B * H, N, D, "f32", 900 + nseg)
    K, V = dev["K"].view(B, H, N, D), dev["V"].view(B, H, N, D)
    state = torch.zeros(la.la_decode_state_bytes(B, H, D) // 4, device="cuda")
    try:
        la.la_debug_override(64, 0)
        ws = scratch(la.la_workspace_bytes(B, H, N, D, la.LA_F32, False, 0), "cuda")
        la.la_decode_prefill(K, V, state, 0, ws)
        once = canonical_state(state, B * H, D)
        la.la_decode_prefill(K, V, state, 1, ws)
        twice = canonical_state(state, B * H, D)
    finally:
        la.la_debug_override(0, 0)
    k, v = ref["K"], ref["V"]
    want = np.concatenate([np.einsum("bnr,bnj->brj", k, v).reshape(B * H, -1), k.sum(1), v.sum(1),
                           np.full((B * H, 1), float(N))], axis=1)
    assert excess(once, want, TOL["f32"]) <= 1.0
    assert np.array_equal(twice, 2.0 * once)


# bf16: shorter than a prompt's shortest segments, prompts in one segment and in several of their own, more than a round
@pytest.mark.parametrize("BH,N,D", [(3, 70, 32), (2, 257, 64), (5, 700, 128), (300, 90, 128), (140, 400, 128)])
def test_prefill_in_segments_of_its_own(la, BH, N, D):
    dev, ref = draw(BH, N, D, "bf16", 960 + N)
    K, V = dev["K"].view(1, BH, N, D), dev["V"].view(1, BH, N, D)
    state = torch.zeros(la.la_decode_state_bytes(1, BH, D) // 4, device="cuda")
    ws = scratch(la.la_workspace_bytes(1, BH, N, D, la.LA_BF16, False, 0), "cuda")
    la.la_decode_prefill(K, V, state, 0, ws)
    k, v = ref["K"], ref["V"]
    want = np.concatenate([np.matmul(k.transpose(0, 2, 1), v).reshape(BH, -1), k.sum(1), v.sum(1),
                           np.full((BH, 1), float(N))], axis=1)
    assert excess(canonical_state(state, BH, D), want, TOL["f32"]) <= 1.0


def test_prefill_one_block_after_another(la):
    """fp32 at head size 256 where the four blocks do not share a launch: set, then added to."""
    BH, N, D = 66, 1000, 256
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)
    K, V = (torch.randn((1, BH, N, D), device="cuda", generator=gen) for _ in range(2))
    state = torch.zeros(la.la_decode_state_bytes(1, BH, D) // 4, device="cuda")
    ws = scratch(la.la_workspace_bytes(1, BH, 4 * N, D, la.LA_F32, False, 0), "cuda")
    long = [torch.cat([x] * 4, 2) for x in (K, V)]  # 4000 rows: one block after another
    la.la_decode_prefill(*long, state, 0, ws)
    once = canonical_state(state, BH, D)
    la.la_decode_prefill(*long, state, 1, ws)
    assert np.array_equal(canonical_state(state, BH, D), 2.0 * once)
    k, v = K[0].double(), V[0].double()
    want = torch.cat([torch.stack([x.t().contiguous() @ y for x, y in zip(k, v)]).flatten(1), k.sum(1), v.sum(1),
                      torch.full((BH, 1), float(N), device="cuda", dtype=torch.float64)], 1) * 4
    assert excess(once, want.cpu().numpy(), TOL["f32"]) <= 1.0


def _outcome(call):
    try:
        call()
    except Exception as e:  # noqa: BLE001 -- the type and the text are what is compared
        return type(e), str(e)
    return None


def test_native_marshalling_refuses_what_python_refuses(la, monkeypatch):
    """Every form of a bad argument, through the native functions and through the Python ones: the same
    exception with the same text; and the good calls give the same bits."""
    from paper_2510_21956_amd import binding
    assert binding._native is not None, "_marshal.so is not built"
    B, H, N, D = 2, 3, 40, 32
    gen = torch.Generator(device="cuda")
    gen.manual_seed(11)
    x = [torch.randn((B, H, N, D), device="cuda", generator=gen) for _ in range(9)]
    G = torch.empty((B, H, N), device="cuda")
    ws = torch.empty(1 << 22, dtype=torch.uint8, device="cuda")
    st = torch.zeros(la.la_decode_state_bytes(B, H, D) // 4, device="cuda")
    good = {"f": [x[0], x[1], x[2], x[3], G, 1.0, 0.5, True, ws, None],
            "b": [x[0], x[1], x[2], x[3], G, x[4], x[5], x[6], x[7], 1, 0.5, 1, ws, None],
            "d": [x[0], x[1], x[2], x[3], G, st, 1.0, 0.5], "p": [x[0], x[1], st, 0, ws]}
    funcs = {"f": [la.la_forward_save, la.la_forward_qknorm_save,
                   lambda *a: la.la_forward(*a[:-1]), lambda *a: la.la_forward_qknorm(*a[:-1])],
             "b": [la.la_backward_saved, la.la_backward_qknorm_saved,
                   lambda *a: la.la_backward(*a[:-1]), lambda *a: la.la_backward_qknorm(*a[:-1])],
             "d": [la.la_decode_step], "p": [la.la_decode_prefill]}

    class Scattered(torch.Tensor):  # a subclass answers for itself
        def is_contiguous(self, *args, **kwargs):
            return False

    bad = [None, x[0].as_subclass(Scattered), x[0].transpose(1, 2), x[0][0], x[0].cpu(), x[0].half(), x[0].to(torch.bfloat16),
           x[0][:, :, :20].contiguous(), x[0].double(), "text", 3, G.double(), ws[:256], ws[8:]]
    for key, args in good.items():
        n = len(args)
        calls = [args] + [args[:i] + [v] + args[i + 1:] for i in range(n) for v in bad]
        # a short, host or misaligned buffer may be taken where a tensor is optional; only the outcome counts
        for fn in funcs[key]:
            for c in calls:
                native = _outcome(lambda: fn(*c))
                with monkeypatch.context() as m:
                    m.setattr(binding, "_native", None)
                    assert _outcome(lambda: fn(*c)) == native, (key, [type(v) for v in c])
    torch.cuda.synchronize()
    saved = torch.empty(la.la_saved_state_bytes(B, H, N, D, la.LA_F32, True), dtype=torch.uint8, device="cuda")
    out = []
    for native in (binding._native, None):
        with monkeypatch.context() as m:
            m.setattr(binding, "_native", native)
            O, dQ, dK, dV = (torch.full_like(x[0], float("nan")) for _ in range(4))
            s2 = torch.zeros_like(st)
            g = torch.full_like(G, float("nan"))
            la.la_forward_save(x[0], x[1], x[2], O, g, 1.0, 0.05, True, ws, saved)
            la.la_backward_saved(x[0], x[1], x[2], O, g, x[4], dQ, dK, dV, 1.0, 0.05, True, ws, saved)
            la.la_decode_prefill(x[1], x[2], s2, 0, ws)
            o1, g1 = torch.empty((B, H, 1, D), device="cuda"), torch.empty((B, H, 1), device="cuda")
            q1 = [t[:, :, :1].contiguous() for t in x[:3]]
            la.la_decode_step(*q1, o1, g1, s2, 1.0, 0.05, stream=torch.cuda.current_stream())
            out.append([O, g, dQ, dK, dV, s2, o1, g1])
    assert all(torch.equal(a, b) for a, b in zip(*out))


@pytest.mark.parametrize("dtype", [torch.float16, torch.float64, torch.int32])
def test_calls_in_another_type_are_refused_in_the_same_words(la, monkeypatch, dtype):
    """Every tensor of the call in a type the library does not take: nothing stops the checks before the type
    itself is refused."""
    from paper_2510_21956_amd import binding
    assert binding._native is not None, "_marshal.so is not built"
    x = torch.zeros((1, 2, 8, 16), device="cuda", dtype=dtype)
    G, st = torch.zeros((1, 2, 8), device="cuda"), torch.zeros(1 << 12, device="cuda")
    ws = torch.zeros(1 << 16, dtype=torch.uint8, device="cuda")
    for call in (lambda: la.la_forward(x, x, x, x, G, 1.0, 0.5, True, ws),
                 lambda: la.la_backward(x, x, x, x, G, x, x, x, x, 1.0, 0.5, True, ws),
                 lambda: la.la_decode_step(x, x, x, x, G, st, 1.0, 0.5),
                 lambda: la.la_decode_prefill(x, x, st, 0, ws)):
        native = _outcome(call)
        with monkeypatch.context() as m:
            m.setattr(binding, "_native", None)
            assert native == _outcome(call) == (TypeError, "Q/K/V must be float32 or bfloat16, got %s" % dtype)


def test_stream_handles_are_taken_as_ctypes_takes_them(la):
    """A stream object may hold its handle as a number, as a ctypes pointer or, for the default stream, as None."""
    import ctypes
    q = [torch.randn((1, 2, 1, 16), device="cuda") for _ in range(3)]
    out = []
    for handle in (0, None, ctypes.c_void_p(0), ctypes.c_void_p(torch.cuda.default_stream().cuda_stream)):
        o, st = torch.zeros_like(q[0]), torch.zeros(la.la_decode_state_bytes(1, 2, 16) // 4, device="cuda")
        la.la_decode_step(*q, o, None, st, 1.0, 0.5, stream=type("Stream", (), {"cuda_stream": handle})())
        torch.cuda.synchronize()
        out.append(o)
    assert out[0].abs().sum() > 0 and all(torch.equal(out[0], o) for o in out)
