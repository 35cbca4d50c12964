"""What users have this library do, as cases to time: the operator's layers, forward and backward, from single small
calls to the benchmark's training step, through the entry points of `paper_2503_12211_amd`.

A case is one `kind` of call and its sizes:

  forward  stl_forward without saved planes (inference), variant AUTO, optionally with GELU on the output
  train    stl_forward saving Xhat and Yhat, then stl_backward with all four gradients
  class0   one step of fitting the bases: stl_encode_weight, stl_forward, stl_backward, stl_encode_weight_backward
  mlp      stl_mlp_forward: up-projection, GELU, down-projection
  aa       stl_aa_forward saving the planes, then stl_aa_backward (attention products, both operands run-time encoded)
  ragged   stl_ragged_forward saving the planes, then stl_ragged_backward (images whose token count 4 does not divide)
  weight   stl_encode_weight, then stl_encode_weight_backward (true encoding)

Value distributions are those of `stl_synth.py`: X, dC ~ N(0, 1), What ~ N(0, 1/k), bases ~ N(0, 1/16).
"""
import math

import torch

import paper_2503_12211_amd as stl

DTYPES = {"bf16": (torch.bfloat16, stl.STL_BF16, 2), "f32": (torch.float32, stl.STL_F32, 4)}


def _case(name, kind, dtype, m, k, n, r, **more):
    c = {"kind": kind, "dtype": dtype, "m": m, "k": k, "n": n, "r": r, "batch": 1, "gelu": False, "transposed": False}
    if name:
        c = {"name": name, **c}
    c.update(more)
    return c


def listed():
    return [
        # one small layer in a serving loop: a few microseconds of work, so launches and latency count
        _case("forward_small", "forward", "bf16", 128, 512, 512, 8),
        # a handful of tokens through a full-size layer (token-by-token decoding): reading the weight planes is the work
        _case("forward_few_rows", "forward", "bf16", 64, 4096, 4096, 32),
        # an ordinary layer with its activation: one or two images, a short prompt
        _case("forward_medium_gelu", "forward", "bf16", 1024, 1024, 1024, 32, gelu=True),
        # the rank sweep's large forward at a rank where the operator is well ahead of the dense product
        _case("forward_large_r16", "forward", "bf16", 8192, 4096, 4096, 16),
        # the square timing workload at the rank of the exact basis (two 32-plane groups)
        _case("forward_square_r49", "forward", "bf16", 4096, 4096, 4096, 49),
        # the benchmark's training step
        _case("train_large", "train", "bf16", 8192, 4096, 4096, 32),
        # training a classifier head, 768 -> 1000 classes: 250 tile columns, not a multiple of 8
        _case("train_head_1000", "train", "bf16", 2048, 768, 1000, 32),
        # fitting the bases in fp32 at the size of the exact-basis check
        _case("class0_step_f32", "class0", "f32", 256, 256, 256, 49),
        # the MLP-shaped pair of the workload list
        _case("mlp_pair", "mlp", "bf16", 16384, 1024, 4096, 24),
        # attention scores Q K^T of 8 images x 12 heads, 200 tokens, head width 64, trained
        _case("attention_scores", "aa", "bf16", 200, 64, 200, 32, batch=96, transposed=True),
        # a transformer MLP layer on 64 images of 197 tokens, trained
        _case("ragged_vit", "ragged", "bf16", 197, 768, 3072, 32, batch=64),
        # true encoding of a full-size weight and its gradients
        _case("weight_encoding", "weight", "bf16", 4, 4096, 4096, 32),
    ]


def _log_int(rng, lo, hi, step):
    """A multiple of `step` in [lo, hi], uniform in its logarithm."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return min(max(int(round(v / step)) * step, -(-lo // step) * step), hi // step * step)


# Kinds in the proportion of the listed cases; ranks as in the rank sweep and the tests.
_KINDS = ["forward"] * 5 + ["train"] * 3 + ["class0", "mlp", "aa", "ragged", "weight"]
_RANKS = [8, 12, 16, 20, 24, 32, 32, 32, 40, 48, 49, 64]


def draw(rng):
    # at most about half the largest listed case (4.2e11 flop, 5e8 bytes); sizes that are no multiple of 32 (for a forward
    # pass only the widths) are those of small and middle-sized layers
    while True:
        kind = rng.choice(_KINDS)
        odd = rng.random() < 0.35
        step = 4 if odd else 64
        r = rng.choice(_RANKS)
        if kind == "class0":
            m, k, n = (_log_int(rng, 64, 1024, 4 if odd else 32) for _ in range(3))
            c = _case(None, kind, "f32", m, k, n, r)
        elif kind == "aa":
            m = _log_int(rng, 64, 1024, 4 if odd else 64)
            k, n = rng.choice([32, 64, 80, 128]), m
            tr = rng.random() < 0.5
            if not tr:
                k, n = n, k                                  # attention x values
            c = _case(None, kind, "bf16", m, k, n, rng.choice([16, 24, 32]), batch=rng.choice([8, 12, 24, 32, 48, 64, 96]),
                      transposed=tr)
        elif kind == "ragged":
            rows = rng.choice([50, 65, 145, 197, 197, 257, 577])
            c = _case(None, kind, "bf16", rows, _log_int(rng, 192, 3072, 64), _log_int(rng, 192, 3072, 64),
                      rng.choice([16, 24, 32, 49]), batch=rng.choice([4, 8, 16, 32, 64]))
        elif kind == "mlp":
            c = _case(None, kind, "bf16", _log_int(rng, 256, 16384, 4), _log_int(rng, 256, 1024, step),
                      _log_int(rng, 512, 4096, step), rng.choice([16, 24, 32, 49]))
        elif kind == "weight":
            c = _case(None, kind, "bf16", 4, _log_int(rng, 256, 4096, step), _log_int(rng, 256, 4096, step), r)
        else:
            dtype = "f32" if rng.random() < 0.15 else "bf16"
            m = _log_int(rng, 16, 8192, 4 if kind == "forward" or odd else 32)
            k, n = _log_int(rng, 256, 4096, step), _log_int(rng, 256, 4096, step)
            c = _case(None, kind, dtype, m, k, n, r, gelu=kind == "forward" and dtype == "bf16" and rng.random() < 0.3)
        w = work(c)
        small = c["dtype"] == "f32" or any(c[s] % 32 for s in (("m", "k", "n") if kind in ("train", "aa") else ("k", "n")))
        if w["bytes"] <= 4e8 and w["flops"] <= (4e9 if small else 2e11):
            return c


def work(case):
    m, k, n, r, b = (case[s] for s in ("m", "k", "n", "r", "batch"))
    es = DTYPES[case["dtype"]][2]
    if case["kind"] == "ragged":
        m_all, M = b * m, b * (-(-m // 4))
    else:
        m_all, M = b * m, b * (m // 4)
    K, N = k // 4, n // 4
    What, basis = r * K * N, 16 * r
    gemm, enc_k, enc_n = 2 * r * M * K * N, 32 * r * M * K, 32 * r * M * N
    if case["kind"] == "forward":
        return {"bytes": es * (m * k + What + m * n + 2 * basis), "flops": gemm + enc_k + enc_n}
    if case["kind"] in ("train", "ragged"):
        return {"bytes": es * (2 * m_all * k + What + 2 * m_all * n + 2 * basis) + 4 * (What + 2 * basis),
                "flops": 3 * gemm + 3 * enc_k + 3 * enc_n}
    if case["kind"] == "class0":
        return {"bytes": es * (2 * m * k + k * n + 2 * m * n + 3 * basis) + 4 * 3 * basis,
                "flops": 3 * gemm + 3 * enc_k + 3 * enc_n + 2 * 32 * r * K * N}
    if case["kind"] == "mlp":
        return {"bytes": es * (2 * m * k + 2 * What + 4 * basis), "flops": 2 * gemm + 2 * enc_k + 2 * enc_n}
    if case["kind"] == "aa":
        enc_b = 32 * r * b * K * N
        return {"bytes": es * (2 * m_all * k + 2 * b * k * n + 2 * m_all * n + 3 * basis) + 4 * 3 * basis,
                "flops": 3 * gemm + 3 * enc_k + 3 * enc_n + 3 * enc_b}
    return {"bytes": es * (2 * k * n + What + basis) + 4 * (What + basis), "flops": 3 * 32 * r * K * N}


def tolerance(case):
    # Each stored intermediate and each output is rounded to the storage type once: against 64 bits 1.7e-3 to 4.2e-3
    # in bf16 (two, three or, for the stacked pair, five roundings) and 1.5e-7 to 5e-7 in fp32; the largest entry of
    # large outputs is off by 0.03 of the root mean square in bf16.
    if case["dtype"] == "f32":
        return {"rel": 3e-6, "max": 1e-4}
    return {"rel": 1.5e-2 if case["kind"] == "mlp" else 1e-2, "max": 0.15}


def _inputs(case, seed):
    """All inputs of a case as device tensors in their storage types, from the seed alone."""
    dt = DTYPES[case["dtype"]][0]
    m, k, n, r, b = (case[s] for s in ("m", "k", "n", "r", "batch"))
    g = torch.Generator(device="cuda").manual_seed(seed)

    def normal(shape, sigma=1.0, dtype=dt):
        return (torch.randn(shape, generator=g, device="cuda") * sigma).to(dtype)

    def basis():
        return normal((r, 16), 0.25)

    kind = case["kind"]
    if kind == "weight":
        return {"W": normal((k, n), k ** -0.5), "E_W": basis(), "dWhat": normal((r, k // 4, n // 4), 1.0, torch.float32)}
    if kind == "mlp":
        return {"X": normal((m, k)), "What1": normal((r, k // 4, n // 4), k ** -0.5), "E_X1": basis(), "D1": basis(),
                "What2": normal((r, n // 4, k // 4), n ** -0.5), "E_X2": basis(), "D2": basis()}
    if kind == "aa":
        B = normal((b * n, k) if case["transposed"] else (b * k, n), k ** -0.5)
        return {"A": normal((b * m, k)), "B": B, "E_A": basis(), "E_B": basis(), "D": basis(), "dC": normal((b * m, n))}
    i = {"X": normal((b * m, k)), "E_X": basis(), "D": basis()}
    if kind == "class0":
        i.update(W=normal((k, n)), E_W=basis())
    else:
        i["What"] = normal((r, k // 4, n // 4), k ** -0.5)
    if kind != "forward":
        i["dC"] = normal((b * m, n))
    if kind == "ragged" and m % 4:
        i["fold"] = torch.eye(m % 4, 4, device="cuda") + normal((m % 4, 4), 0.25, torch.float32)
    return i


def prepare(case, seed):
    dt, code, _ = DTYPES[case["dtype"]]
    m, k, n, r, b = (case[s] for s in ("m", "k", "n", "r", "batch"))
    kind = case["kind"]
    s = dict(_inputs(case, seed), kind=kind, batch=b, rows=m)
    prob = s["prob"] = stl.Problem(b * m if kind == "ragged" else m, k, n, r, code)
    K, N = k // 4, n // 4
    M = b * (-(-m // 4))

    def new(shape, dtype=dt):
        return torch.empty(shape, dtype=dtype, device="cuda")

    def like(name):
        return torch.empty_like(s[name])

    def planes(rows, cols):
        return new(stl.stl_plane_elems(rows, cols, r))

    def scratch(*sizes):
        s["ws_bytes"] = max(16, *sizes)
        s["ws"] = new(s["ws_bytes"], torch.uint8)

    def small(*names):
        for x in names:
            s[x] = new((r, 16), torch.float32)

    def need(op):
        return stl.stl_workspace_bytes(prob, op)

    if kind == "forward":
        s["C"] = new((m, n))
        s["flags"] = stl.STL_FLAG_AUTO | (stl.STL_FLAG_GELU if case["gelu"] else 0)
        scratch(stl.stl_workspace_bytes(prob, stl.STL_OP_FORWARD, s["flags"]))
    elif kind == "mlp":
        s["down"] = stl.Problem(m, n, k, r, code)
        s["C"] = like("X")
        scratch(stl.stl_mlp_workspace_bytes(prob, s["down"], stl.STL_FLAG_GELU))
    elif kind == "aa":
        s.update(C=new((b * m, n)), dA=like("A"), dB=like("B"), flags=stl.STL_FLAG_B_TRANSPOSED if case["transposed"] else 0,
                 Ahat=planes(M, K), Yhat=planes(M, N), Bhat=planes(b * N, K) if case["transposed"] else planes(b * K, N))
        small("dE_A", "dE_B", "dD")
        scratch(*(stl.stl_aa_workspace_bytes(prob, b, op) for op in (stl.STL_OP_FORWARD, stl.STL_OP_BACKWARD)))
    elif kind == "weight":
        s.update(What=new((r, K, N)), dW=like("W"))
        small("dE_W")
        scratch(need(stl.STL_OP_ENCODE_WEIGHT_BACKWARD))
    else:
        s.update(C=new((b * m, n)), dX=like("X"), Xhat=planes(M, K), Yhat=planes(M, N))
        s["dWhat"] = new((r, K, N), torch.float32)
        small("dE_X", "dD")
        if kind == "ragged":
            s.setdefault("fold", None)
            s["dfold"] = torch.empty_like(s["fold"]) if m % 4 else None
            scratch(*(stl.stl_ragged_workspace_bytes(prob, m, op) for op in (stl.STL_OP_FORWARD, stl.STL_OP_BACKWARD)))
        else:
            scratch(need(stl.STL_OP_FORWARD), need(stl.STL_OP_BACKWARD), need(stl.STL_OP_ENCODE_WEIGHT_BACKWARD))
        if kind == "class0":
            s.update(What=new((r, K, N)), dW=like("W"))
            small("dE_W")
    return s


def run(s):
    kind, prob, ws, nb = s["kind"], s["prob"], s["ws"], s["ws_bytes"]
    if kind == "forward":
        stl.stl_forward(prob, s["X"], s["What"], s["E_X"], s["D"], s["C"], None, None, ws, nb, s["flags"])
        return s["C"]
    if kind == "mlp":
        stl.stl_mlp_forward(prob, s["down"], s["X"], s["What1"], s["E_X1"], s["D1"], s["What2"], s["E_X2"], s["D2"], s["C"],
                            ws, nb, stl.STL_FLAG_GELU)
        return s["C"]
    if kind == "aa":
        stl.stl_aa_forward(prob, s["batch"], s["A"], s["B"], s["E_A"], s["E_B"], s["D"], s["C"], s["Ahat"], s["Bhat"], s["Yhat"],
                           ws, nb, s["flags"])
        stl.stl_aa_backward(prob, s["batch"], s["A"], s["B"], s["E_A"], s["E_B"], s["D"], s["dC"], s["Ahat"], s["Bhat"],
                            s["Yhat"], s["dA"], s["dB"], s["dE_A"], s["dE_B"], s["dD"], 0, ws, nb, s["flags"])
        return {x: s[x] for x in ("C", "dA", "dB", "dE_A", "dE_B", "dD")}
    if kind == "weight":
        stl.stl_encode_weight(prob, s["W"], s["E_W"], s["What"])
        stl.stl_encode_weight_backward(prob, s["W"], s["E_W"], s["dWhat"], s["dW"], s["dE_W"], 0, ws, nb)
        return {x: s[x] for x in ("What", "dW", "dE_W")}
    if kind == "ragged":
        stl.stl_ragged_forward(prob, s["rows"], s["X"], s["What"], s["E_X"], s["D"], s["fold"], s["C"], s["Xhat"], s["Yhat"], ws,
                               nb)
        stl.stl_ragged_backward(prob, s["rows"], s["X"], s["What"], s["E_X"], s["D"], s["fold"], s["dC"], s["Xhat"], s["Yhat"],
                                s["dX"], s["dWhat"], s["dE_X"], s["dD"], s["dfold"], 0, ws, nb)
        return {x: s[x] for x in ("C", "dX", "dWhat", "dE_X", "dD", "dfold")}
    if kind == "class0":
        stl.stl_encode_weight(prob, s["W"], s["E_W"], s["What"])
    stl.stl_forward(prob, s["X"], s["What"], s["E_X"], s["D"], s["C"], s["Xhat"], s["Yhat"], ws, nb)
    stl.stl_backward(prob, s["X"], s["What"], s["E_X"], s["D"], s["dC"], s["Xhat"], s["Yhat"], s["dX"], s["dWhat"], s["dE_X"],
                     s["dD"], 0, ws, nb)
    outs = ["C", "dX", "dE_X", "dD"]
    if kind == "train":
        outs.append("dWhat")
    else:
        stl.stl_encode_weight_backward(prob, s["W"], s["E_W"], s["dWhat"], s["dW"], s["dE_W"], 0, ws, nb)
        outs += ["dW", "dE_W"]
    return {x: s[x] for x in outs}


# ---- the same in 64 bits, with plain torch ---------------------------------------------------------------------------
def _tiles(A):
    a, b = A.shape
    return A.reshape(a // 4, 4, b // 4, 4).permute(0, 2, 1, 3).reshape(a // 4, b // 4, 16)


def _untile(T):
    a, b, _ = T.shape
    return T.reshape(a, b, 4, 4).permute(0, 2, 1, 3).reshape(4 * a, 4 * b)


def _encode(A, E):
    """(r, a/4, b/4) planes of the tiles of A."""
    return (_tiles(A) @ E.t()).permute(2, 0, 1).contiguous()


def _decode(Y, D):
    return _untile(Y.permute(1, 2, 0).contiguous() @ D)


def _products(A, B):
    return torch.stack([A[p] @ B[p] for p in range(A.shape[0])])


def _basis_grad(P, V):
    return P.reshape(P.shape[0], -1) @ _tiles(V).reshape(-1, 16)


def _layer(X, What, E_X, D, dC):
    """C, dX, dWhat, dE_X, dD of one layer."""
    Xhat = _encode(X, E_X)
    Yhat = _products(Xhat, What)
    dY = _encode(dC, D)
    dXhat = _products(dY, What.transpose(1, 2))
    return (_decode(Yhat, D), _decode(dXhat, E_X), _products(Xhat.transpose(1, 2), dY), _basis_grad(dXhat, X),
            _basis_grad(Yhat, dC))


def exact(case, seed):
    i = {name: t.double() for name, t in _inputs(case, seed).items()}
    kind, b, m = case["kind"], case["batch"], case["m"]
    if kind == "forward":
        C = _decode(_products(_encode(i["X"], i["E_X"]), i["What"]), i["D"])
        return torch.nn.functional.gelu(C) if case["gelu"] else C
    if kind == "mlp":
        H = _decode(_products(_encode(i["X"], i["E_X1"]), i["What1"]), i["D1"])
        return _decode(_products(_encode(torch.nn.functional.gelu(H), i["E_X2"]), i["What2"]), i["D2"])
    if kind == "weight":
        return {"What": _encode(i["W"], i["E_W"]), "dW": _decode(i["dWhat"], i["E_W"]), "dE_W": _basis_grad(i["dWhat"], i["W"])}
    if kind == "aa":
        out = {"C": [], "dA": [], "dB": [], "dE_A": 0, "dE_B": 0, "dD": 0}
        for A, B, dC in zip(i["A"].chunk(b), i["B"].chunk(b), i["dC"].chunk(b)):
            B = B.t().contiguous() if case["transposed"] else B
            C, dA, dBhat, dE_A, dD = _layer(A, _encode(B, i["E_B"]), i["E_A"], i["D"], dC)
            dB = _decode(dBhat, i["E_B"])
            out["C"].append(C)
            out["dA"].append(dA)
            out["dB"].append(dB.t() if case["transposed"] else dB)
            out["dE_A"], out["dD"] = out["dE_A"] + dE_A, out["dD"] + dD
            out["dE_B"] = out["dE_B"] + _basis_grad(dBhat, B)
        return {x: torch.cat(v) if isinstance(v, list) else v for x, v in out.items()}
    if kind == "ragged" and m % 4:
        # null rows at the end of every image; the last tile row's four output rows are folded into the real ones
        full = -(-m // 4) * 4
        keep = full - 4
        X = torch.nn.functional.pad(i["X"].reshape(b, m, -1), (0, 0, 0, full - m)).reshape(b * full, -1)
        dC = i["dC"].reshape(b, m, -1)
        dPad = torch.cat([dC[:, :keep], i["fold"].t() @ dC[:, keep:]], 1).reshape(b * full, -1)
        C, dX, dWhat, dE_X, dD = _layer(X, i["What"], i["E_X"], i["D"], dPad)
        C, dX = C.reshape(b, full, -1), dX.reshape(b, full, -1)
        tail = C[:, keep:]
        dfold = torch.stack([torch.stack([(dC[:, keep + a] * tail[:, c]).sum() for c in range(4)]) for a in range(m % 4)])
        return {"C": torch.cat([C[:, :keep], i["fold"] @ tail], 1).reshape(b * m, -1), "dX": dX[:, :m].reshape(b * m, -1),
                "dWhat": dWhat, "dE_X": dE_X, "dD": dD, "dfold": dfold}
    What = _encode(i["W"], i["E_W"]) if kind == "class0" else i["What"]
    C, dX, dWhat, dE_X, dD = _layer(i["X"], What, i["E_X"], i["D"], i["dC"])
    out = {"C": C, "dX": dX, "dE_X": dE_X, "dD": dD}
    if kind == "class0":
        out.update(dW=_decode(dWhat, i["E_W"]), dE_W=_basis_grad(dWhat, i["W"]))
    else:
        out["dWhat"] = dWhat
        if kind == "ragged":
            out["dfold"] = None
    return out
