"""The work this library is used for, as cases that can be timed and checked.

A case is one call sequence of a user's program through the package's public entry points:

  step     a training step of a program that manages its own buffers: la_forward_save, then
           la_backward_saved with the sums the forward pass handed over
  train    the same through the autograd wrapper (linear_attention and torch.autograd.grad),
           with or without the normalisation of the Q and K rows inside the kernels
  forward  la_forward alone
  prefill  a prompt in a serving program: la_forward without G, then la_decode_prefill
  decode   la_decode_step: T new rows per slice on a carried state

Values follow the recipe of la_workloads.py: Q, K Gaussian with rows of unit length (raw rows
where the kernels normalise them), V and dO Gaussian, kernel f(x) = 1 + 0.5 x.
"""
import math

import torch

import paper_2510_21956_amd as la

A, BCOEF = 1.0, 0.5
PROMPT = 512  # rows already in the state a decode case starts from


def _case(name, kind, B, H, N, D, dtype, causal=True, norm=False):
    return {"name": name, "kind": kind, "B": B, "H": H, "N": N, "D": D, "dtype": dtype,
            "causal": causal, "norm": norm}


def listed():
    return [
        # the smallest training step (a unit test's layer, a toy model): launches and latency
        _case("train_f32_tiny", "train", 1, 1, 256, 16, "f32"),
        # one token for every sequence of a serving batch
        _case("decode_bf16_d128", "decode", 8, 16, 1, 128, "bf16"),
        # a ragged prompt in a serving program
        _case("prefill_bf16_d128_ragged", "prefill", 2, 16, 3001, 128, "bf16"),
        # the headline layer: fp32, head size 64
        _case("step_f32_d64", "step", 4, 16, 4096, 64, "f32"),
        # without the mask: an encoder layer over a long sequence
        _case("step_f32_d64_unmasked", "step", 8, 8, 16384, 64, "f32", causal=False),
        # one attention layer of an LLM training step
        _case("step_bf16_d128", "step", 8, 16, 2048, 128, "bf16"),
        # a long-context training step: few slices, very long sequences
        _case("step_bf16_d128_long", "step", 1, 16, 131072, 128, "bf16"),
        # odd sizes in bf16 at the smaller head size
        _case("step_bf16_d64_ragged", "step", 3, 12, 5003, 64, "bf16"),
        # the paper's layer benchmark: forward pass at N = 10^4
        _case("forward_f32_d128_paper", "forward", 4, 16, 10000, 128, "f32"),
        # the short end of the paper's sequence-length sweep
        _case("step_f32_d128_short", "step", 4, 16, 1000, 128, "f32"),
        # the top of the paper's head-size sweep
        _case("step_f32_d256_paper", "step", 4, 16, 4096, 256, "f32"),
        # an LLM layer through autograd with the Q, K normalisation of the paper inside
        _case("train_norm_bf16_d128", "train", 8, 16, 2048, 128, "bf16", norm=True),
    ]


def draw(rng):
    kind = rng.choice(["step", "step", "train", "train", "forward", "prefill", "decode"])
    D = rng.choice([16, 32, 64, 64, 128, 128, 128, 256])
    dtype = rng.choice(["f32", "bf16"])
    B, H = rng.randint(1, 8), rng.randint(1, 24)
    causal, norm = True, False
    if kind == "decode":
        N = rng.choice([1, 1, 1, 2, 3, 5, 8])
    else:
        # at most the token-heads x D^2 and the token-heads of the largest listed cases
        # (head size 16 runs on kernels of its own, sized for small problems)
        cap = min(1.2e10 / (D * D), 2.0e6 if D > 16 else 2.5e5)
        N = max(1, int(round(math.exp(rng.uniform(math.log(30), math.log(60000))))))
        while B * H * N > cap and B * H > 1:
            if B > 1:
                B -= 1
            else:
                H -= 1
        N = int(min(N, cap))
        if kind != "prefill":
            causal = rng.random() < 0.75
        norm = kind == "train" and D <= 128 and rng.random() < 0.6
    return {"kind": kind, "B": B, "H": H, "N": N, "D": D, "dtype": dtype, "causal": causal,
            "norm": norm}


def _inputs(case, seed):
    """Q, K, V, dO as a program holds them (float32 or bfloat16, [B, H, N, D])."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed) * 7919 + 17)
    td = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    shape = (case["B"], case["H"], case["N"], case["D"])
    out = []
    for name in ("Q", "K", "V", "dO"):
        x = torch.randn(shape, device="cuda", dtype=torch.float32, generator=gen)
        if name in ("Q", "K"):
            if case["norm"]:
                x = x * (3.0 if name == "Q" else 0.25)
            else:
                x = x / x.norm(dim=-1, keepdim=True)
        out.append(x.to(td))
    return out


def _decode_state(case, seed):
    """[S | z | p | count] of a prompt of PROMPT rows, one row of floats per slice."""
    B, H, D = case["B"], case["H"], case["D"]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed) * 104729 + 5)
    K = torch.randn((B * H, PROMPT, D), device="cuda", dtype=torch.float32, generator=gen)
    V = torch.randn((B * H, PROMPT, D), device="cuda", dtype=torch.float32, generator=gen)
    K = (K / K.norm(dim=-1, keepdim=True)).double()
    V = V.double()
    row = la.la_decode_state_bytes(B, H, D) // 4 // (B * H)
    st = torch.zeros((B * H, row), device="cuda", dtype=torch.float32)
    st[:, :D * D] = torch.matmul(K.transpose(1, 2).contiguous(), V).reshape(B * H, D * D)
    st[:, D * D:D * D + D] = K.sum(1)
    st[:, D * D + D:D * D + 2 * D] = V.sum(1)
    st[:, D * D + 2 * D] = float(PROMPT)
    return st


def _workspace(case, which):
    dt = la.LA_F32 if case["dtype"] == "f32" else la.LA_BF16
    n = la.la_workspace_bytes(case["B"], case["H"], case["N"], case["D"], dt, case["causal"], which)
    return torch.empty(max(n, 256), dtype=torch.uint8, device="cuda")


def prepare(case, seed):
    B, H, N, D = case["B"], case["H"], case["N"], case["D"]
    kind = case["kind"]
    Q, K, V, dO = _inputs(case, seed)
    s = {"case": case, "Q": Q, "K": K, "V": V}
    if kind == "train":
        for x in (Q, K, V):
            x.requires_grad_(True)
        s["dO"] = dO
        return s
    s["O"] = torch.empty_like(Q)
    s["G"] = torch.empty((B, H, N), dtype=torch.float32, device="cuda")
    if kind == "decode":
        s["state"] = _decode_state(case, seed)
        return s
    s["wf"] = _workspace(case, 0)
    if kind == "prefill":
        s["state"] = torch.zeros((B * H, la.la_decode_state_bytes(B, H, D) // 4 // (B * H)),
                                 dtype=torch.float32, device="cuda")
        s["ws"] = _workspace(dict(case, causal=False), 0)
    if kind == "step":
        s["dO"] = dO
        dt = la.LA_F32 if case["dtype"] == "f32" else la.LA_BF16
        ns = la.la_saved_state_bytes(B, H, N, D, dt, case["causal"])
        s["saved"] = torch.empty(ns, dtype=torch.uint8, device="cuda") if ns else None
        s["wb"] = _workspace(case, 1)
        for n in ("dQ", "dK", "dV"):
            s[n] = torch.empty_like(Q)
    return s


def run(s):
    c = s["case"]
    kind, causal = c["kind"], c["causal"]
    if kind == "step":
        la.la_forward_save(s["Q"], s["K"], s["V"], s["O"], s["G"], A, BCOEF, causal, s["wf"],
                           s["saved"])
        la.la_backward_saved(s["Q"], s["K"], s["V"], s["O"], s["G"], s["dO"], s["dQ"], s["dK"],
                             s["dV"], A, BCOEF, causal, s["wb"], s["saved"])
        return [s["O"], s["G"], s["dQ"], s["dK"], s["dV"]]
    if kind == "train":
        O = la.linear_attention(s["Q"], s["K"], s["V"], A, BCOEF, causal, c["norm"])
        dQ, dK, dV = torch.autograd.grad(O, (s["Q"], s["K"], s["V"]), s["dO"])
        return [O.detach(), dQ, dK, dV]
    if kind == "forward":
        la.la_forward(s["Q"], s["K"], s["V"], s["O"], s["G"], A, BCOEF, causal, s["wf"])
        return [s["O"], s["G"]]
    if kind == "prefill":
        la.la_forward(s["Q"], s["K"], s["V"], s["O"], None, A, BCOEF, True, s["wf"])
        la.la_decode_prefill(s["K"], s["V"], s["state"], 0, s["ws"])
        return [s["O"], s["state"]]
    la.la_decode_step(s["Q"], s["K"], s["V"], s["O"], s["G"], s["state"], A, BCOEF)
    return [s["O"], s["G"], s["state"]]


def work(case):
    """Per token-head, with e bytes an element: Q, K, V read and O written (4 D e), g written
    (4); a training step also reads dO and writes dQ, dK, dV (another 4 D e).  4 D^2 flops
    forward and 10 D^2 backward with the mask, the recurrence's own work (12 D^2 together
    without it).  Serving cases read and write the carried state."""
    D, e = case["D"], 4 if case["dtype"] == "f32" else 2
    T = case["B"] * case["H"] * case["N"]
    state = case["B"] * case["H"] * (D * D + 2 * D + 1) * 4
    if case["kind"] == "decode":
        return {"bytes": T * (4 * D * e + 4) + 2 * state, "flops": 4 * D * D * T}
    if case["kind"] == "prefill":
        return {"bytes": T * 4 * D * e + state, "flops": 4 * D * D * T}
    if case["kind"] == "forward":
        return {"bytes": T * (4 * D * e + 4), "flops": 4 * D * D * T}
    g = 4 if case["kind"] == "step" else 0
    return {"bytes": T * (8 * D * e + g), "flops": (14 if case["causal"] else 12) * D * D * T}


def tolerance(case):
    """Four times the largest error against exact() that was measured over the listed and some
    drawn cases (float32 8e-7: sums in another order; bfloat16 2.1e-3: the rounding of the
    outputs and of the O that the backward pass reads)."""
    return {"rel": 4e-6} if case["dtype"] == "f32" else {"rel": 8e-3}


# ---- the same in 64 bits, from the definition's running sums -----------------------------------

def _forward64(q, k, v, causal):
    n, D = q.shape[1], q.shape[2]
    if not causal:
        S, z, p = torch.matmul(k.transpose(1, 2).contiguous(), v), k.sum(1), v.sum(1)
        g = A * n + BCOEF * torch.matmul(q, z.unsqueeze(2)).squeeze(2)
        return (A * p.unsqueeze(1) + BCOEF * torch.matmul(q, S)) / g.unsqueeze(2), g
    S = q.new_zeros((q.shape[0], D, D))
    z, p = q.new_zeros((q.shape[0], 1, D)), q.new_zeros((q.shape[0], 1, D))
    O, G = torch.empty_like(q), q.new_empty(q.shape[:2])
    for i in range(0, n, 256):
        qc, kc, vc = q[:, i:i + 256], k[:, i:i + 256], v[:, i:i + 256]
        P = torch.tril(A + BCOEF * torch.matmul(qc, kc.transpose(1, 2).contiguous()))
        g = P.sum(2) + A * i + BCOEF * (qc * z).sum(2)
        O[:, i:i + 256] = (torch.matmul(P, vc) + A * p + BCOEF * torch.matmul(qc, S)) / g.unsqueeze(2)
        G[:, i:i + 256] = g
        S += torch.matmul(kc.transpose(1, 2).contiguous(), vc)
        z += kc.sum(1, keepdim=True)
        p += vc.sum(1, keepdim=True)
    return O, G


def _backward64(q, k, v, O, G, dO, causal):
    n, D = q.shape[1], q.shape[2]
    W = dO / G.unsqueeze(2)
    d = (O * W).sum(2, keepdim=True)
    if not causal:
        S, z = torch.matmul(k.transpose(1, 2).contiguous(), v), k.sum(1, keepdim=True)
        R = torch.matmul(q.transpose(1, 2).contiguous(), W)
        u, w = (d * q).sum(1, keepdim=True), W.sum(1, keepdim=True)
        dQ = BCOEF * (torch.matmul(W, S.transpose(1, 2).contiguous()) - d * z)
        dK = BCOEF * (torch.matmul(v, R.transpose(1, 2).contiguous()) - u)
        return dQ, dK, A * w + BCOEF * torch.matmul(k, R)
    S, z = q.new_zeros((q.shape[0], D, D)), q.new_zeros((q.shape[0], 1, D))
    dQ, dK, dV = torch.empty_like(q), torch.empty_like(q), torch.empty_like(q)
    starts = list(range(0, n, 256))
    for i in starts:
        s = slice(i, i + 256)
        kc, vc, wc, dc = k[:, s], v[:, s], W[:, s], d[:, s]
        C = torch.tril(torch.matmul(wc, vc.transpose(1, 2).contiguous()) - dc)
        dQ[:, s] = BCOEF * (torch.matmul(C, kc) + torch.matmul(wc, S.transpose(1, 2).contiguous())
                            - dc * z)
        S += torch.matmul(kc.transpose(1, 2).contiguous(), vc)
        z += kc.sum(1, keepdim=True)
    R = torch.zeros_like(S)
    u, w = torch.zeros_like(z), torch.zeros_like(z)
    for i in reversed(starts):
        s = slice(i, i + 256)
        qc, kc, vc, wc, dc = q[:, s], k[:, s], v[:, s], W[:, s], d[:, s]
        C = torch.tril(torch.matmul(wc, vc.transpose(1, 2).contiguous()) - dc)
        P = torch.tril(A + BCOEF * torch.matmul(qc, kc.transpose(1, 2).contiguous()))
        dK[:, s] = BCOEF * (torch.matmul(C.transpose(1, 2).contiguous(), qc)
                            + torch.matmul(vc, R.transpose(1, 2).contiguous()) - u)
        dV[:, s] = (torch.matmul(P.transpose(1, 2).contiguous(), wc) + A * w
                    + BCOEF * torch.matmul(kc, R))
        R += torch.matmul(qc.transpose(1, 2).contiguous(), wc)
        u += (dc * qc).sum(1, keepdim=True)
        w += wc.sum(1, keepdim=True)
    return dQ, dK, dV


def exact(case, seed):
    B, H, N, D = case["B"], case["H"], case["N"], case["D"]
    Q, K, V, dO = [x.double().reshape(B * H, N, D) for x in _inputs(case, seed)]
    kind, shape = case["kind"], (B, H, N, D)
    if kind == "decode":
        st = _decode_state(case, seed).double()
        S = st[:, :D * D].reshape(B * H, D, D)
        z, p = st[:, D * D:D * D + D], st[:, D * D + D:D * D + 2 * D]
        n = D * D + 2 * D
        O, G = torch.empty_like(Q), torch.empty_like(Q[:, :, 0])
        for t in range(N):
            k, v, q = K[:, t], V[:, t], Q[:, t]
            S += k.unsqueeze(2) * v.unsqueeze(1)
            z += k
            p += v
            st[:, n] += 1.0
            G[:, t] = A * st[:, n] + BCOEF * (q * z).sum(1)
            O[:, t] = (A * p + BCOEF * torch.matmul(q.unsqueeze(1), S).squeeze(1)) / G[:, t:t + 1]
        return [O.reshape(shape), G.reshape(B, H, N), st]
    if kind == "prefill":
        O, _ = _forward64(Q, K, V, True)
        st = Q.new_zeros((B * H, la.la_decode_state_bytes(B, H, D) // 4 // (B * H)))
        st[:, :D * D] = torch.matmul(K.transpose(1, 2).contiguous(), V).reshape(B * H, D * D)
        st[:, D * D:D * D + D] = K.sum(1)
        st[:, D * D + D:D * D + 2 * D] = V.sum(1)
        st[:, D * D + 2 * D] = float(N)
        return [O.reshape(shape), st]
    if case["norm"]:
        nq, nk = Q.norm(dim=2, keepdim=True), K.norm(dim=2, keepdim=True)
        Q, K = Q / nq, K / nk
    O, G = _forward64(Q, K, V, case["causal"])
    if kind == "forward":
        return [O.reshape(shape), G.reshape(B, H, N)]
    dQ, dK, dV = _backward64(Q, K, V, O, G, dO, case["causal"])
    if case["norm"]:
        dQ = (dQ - Q * (Q * dQ).sum(2, keepdim=True)) / nq
        dK = (dK - K * (K * dK).sum(2, keepdim=True)) / nk
    grads = [x.reshape(shape) for x in (dQ, dK, dV)]
    O = O.reshape(shape)
    return [O] + grads if kind == "train" else [O, G.reshape(B, H, N)] + grads
