"""The work that users of this library have it do, as cases that can be timed and checked.

A case is one call (or the few calls that belong together) of a public entry point: the multiply at
batch 1, at small, ordinary and large batch, over several layers at once and inside an LSTM cell; the
multiply with tables shared by several matrices; and the encoding of weights.  Shapes are the library's own
configurations (workloads.py, bench.py) or generic ones.
"""
import math

import torch

import paper_2005_09904_amd as biq

DEV = "cuda"


def listed():
    return [
        # -- batch 1: a token (or a frame) at a time, nothing to batch with ------------------------------
        # the smallest fully connected layer: launch latency and little else
        dict(name="fc512_b1", kind="gemm", m=512, n=512, q=1, batch=1, mu=8, values="fp32"),
        # an ordinary layer of a decoder step
        dict(name="gemv2048_q2_b1", kind="gemm", m=2048, n=2048, q=2, batch=1, mu=8, values="fp32"),
        # the wide projection of a feed-forward block in a decoder step, activations out of bf16 arithmetic
        dict(name="ffn_up_q2_b1", kind="gemm", m=16384, n=4096, q=2, batch=1, mu=8, values="bf16"),
        # a very large output layer: the key stream from memory bounds it
        dict(name="gemv_rows1m_q2_b1", kind="gemm", m=1 << 20, n=2048, q=2, batch=1, mu=8, values="fp32"),
        # -- a few vectors: small serving batches, recurrent layers ----------------------------------------
        # one step of an LSTM cell, gates stacked
        dict(name="lstm1024_q3_b8", kind="lstm", hidden=1024, n=1024, q=3, batch=8, mu=8, values="fp32"),
        # the sub-layers of a block that do not depend on each other, in one call
        dict(name="grouped8_2048_q2_b1", kind="grouped", count=8, m=2048, n=2048, q=2, batch=1, mu=8, values="fp32"),
        # an odd layer with another key width and a ragged batch
        dict(name="ragged_mu6_q3_b7", kind="gemm", m=5003, n=3001, q=3, batch=7, mu=6, values="fp32"),
        # three projections of the same input: the tables are built once and queried by each matrix
        dict(name="tables_shared3_b8", kind="tables", count=3, m=1024, n=1024, q=2, batch=8, mu=8, values="fp32"),
        # a square layer with a decoding batch
        dict(name="sq4096_q3_b32", kind="gemm", m=4096, n=4096, q=3, batch=32, mu=8, values="fp32"),
        # -- many vectors: prefill, large serving batches -----------------------------------------------
        dict(name="ffn_up_q2_b128", kind="gemm", m=16384, n=4096, q=2, batch=128, mu=8, values="fp32"),
        dict(name="ffn_down_q2_b128_bf16", kind="gemm", m=4096, n=16384, q=2, batch=128, mu=8, values="bf16"),
        # -- weights: fp32 matrix -> packed signs and scales (once per checkpoint) ---------------------
        dict(name="quantize4096_q3", kind="quantize", m=4096, n=4096, q=3),
    ]


def _log_int(rng, lo, hi):
    """Spread over the logarithm of [lo, hi], odd values among them."""
    v = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    if rng.random() < 0.4 and v >= 64:
        v = v // 64 * 64                      # layer widths are often multiples of 64
    return max(lo, min(hi, v))


def draw(rng):
    kind = rng.choice(["gemm"] * 8 + ["lstm", "grouped", "tables", "quantize", "pack"])
    values = rng.choice(["fp32", "fp32", "bf16", "fp16"])
    q = rng.choice([1, 2, 2, 3, 4])
    if kind == "gemm":
        mu = rng.choice([8] * 6 + [4, 6, 7])
        if rng.random() < 0.35:
            batch = 1
            m, n = _log_int(rng, 128, 1 << 19), _log_int(rng, 128, 16384)
            while q * m * n > 1 << 31:        # at most 256 MiB of keys
                m = (m + 1) // 2
        else:
            batch = _log_int(rng, 2, 256)
            m, n = _log_int(rng, 128, 32768), _log_int(rng, 128, 16384)
            while q * m * n * max(batch, 32) > 16e9:
                m = (m + 1) // 2
        return dict(kind=kind, m=m, n=n, q=q, batch=batch, mu=mu, values=values)
    if kind == "lstm":
        batch = rng.choice([1, _log_int(rng, 2, 32)])
        n = _log_int(rng, 96, 2048 if batch == 1 else 1024)
        return dict(kind=kind, hidden=_log_int(rng, 32, n - 32), n=n, q=q, batch=batch, mu=8, values=values)
    if kind == "grouped":
        batch = rng.choice([1, 1, _log_int(rng, 2, 16)])
        return dict(kind=kind, count=rng.randint(2, 12), m=_log_int(rng, 128, 4096),
                    n=_log_int(rng, 128, 2048 if batch == 1 else 1024), q=q, batch=batch, mu=8, values=values)
    if kind == "tables":
        return dict(kind=kind, count=rng.randint(2, 4), m=_log_int(rng, 128, 4096), n=_log_int(rng, 128, 4096), q=q,
                    batch=_log_int(rng, 1, 16), mu=rng.choice([8, 8, 4, 6]), values=values)
    m, n = _log_int(rng, 128, 16384), _log_int(rng, 128, 16384)
    while m * n > 4096 * 8192:
        m = (m + 1) // 2
    return dict(kind=kind, m=m, n=n, q=q)


# ---- inputs, from the seed alone ---------------------------------------------------------------------

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _vectors(g, batch, n, values):
    x = torch.randn((batch, n), device=DEV, generator=g)
    if values == "bf16":
        x = x.bfloat16().float()
    elif values == "fp16":
        x = x.half().float()
    return x


def _keys(g, q, m, n):
    """Packed random signs: iid bytes are iid signs; the padding of a row is zero."""
    stride = -(-n // 128) * 16
    K = torch.randint(0, 256, (q, m, stride), dtype=torch.uint8, device=DEV, generator=g)
    full = n // 8
    if n % 8:
        K[:, :, full] &= (1 << (n % 8)) - 1
        full += 1
    if full < stride:
        K[:, :, full:] = 0
    return K


def _alpha(g, q, m):
    """Scales of the planes fall off, as a quantiser's do."""
    a = torch.rand((q, m), device=DEV, generator=g) * 0.95 + 0.05
    return a.sort(dim=0, descending=True).values.contiguous()


def _inputs(case, seed):
    g = _gen(seed)
    kind = case["kind"]
    if kind == "quantize":
        return dict(W=torch.randn((case["m"], case["n"]), device=DEV, generator=g))
    if kind == "pack":
        b = torch.randint(0, 2, (case["q"], case["m"], case["n"]), dtype=torch.int8, device=DEV, generator=g)
        return dict(B=b * 2 - 1)
    n, q, batch = case["n"], case["q"], case["batch"]
    if kind == "lstm":
        h = case["hidden"]
        return dict(X=_vectors(g, batch, n, case["values"]), K=_keys(g, q, 4 * h, n),
                    alpha=_alpha(g, q, 4 * h) * (1.5 / math.sqrt(n)),
                    bias=torch.randn(4 * h, device=DEV, generator=g) * 0.1,
                    C=torch.randn((batch, h), device=DEV, generator=g))
    count = case.get("count", 1)
    shared = _vectors(g, batch, n, case["values"])
    one = [dict(X=shared if kind == "tables" or i == 0 else _vectors(g, batch, n, case["values"]),
                K=_keys(g, q, case["m"], n), alpha=_alpha(g, q, case["m"])) for i in range(count)]
    return one[0] if kind == "gemm" else dict(layers=one)


# ---- what a program holds before the call, and the call ------------------------------------------------

def _workspace(nbytes):
    return torch.empty(max(nbytes, 16), dtype=torch.uint8, device=DEV)


def prepare(case, seed):
    s = _inputs(case, seed)
    kind, q, mu = case["kind"], case["q"], case.get("mu", 8)
    m, n = case.get("m", 0), case["n"]
    s["case"] = dict(case)
    if kind in ("quantize", "pack"):
        s["K"] = torch.empty((q, m, biq.biq_key_row_stride(n)), dtype=torch.uint8, device=DEV)
        s["alpha"] = torch.empty((q, m), device=DEV)
        return s
    batch = case["batch"]
    if kind == "gemm":
        s["Y"] = torch.empty((batch, m), device=DEV)
        ws = _workspace(biq.biq_workspace_bytes(m, n, q, batch, mu))
        s["call"] = biq.PreparedGemm(s["K"], s["alpha"], s["X"], s["Y"], m, n, q, batch, mu, workspace=ws)
    elif kind == "lstm":
        h = case["hidden"]
        s["H"], s["C_out"] = torch.empty((batch, h), device=DEV), torch.empty((batch, h), device=DEV)
        s["call"] = biq.PreparedLstmCell(s["K"], s["alpha"], s["bias"], s["X"], s["C"], s["H"], s["C_out"], h, n, q,
                                         batch, mu)
    else:
        for layer in s["layers"]:
            layer["Y"] = torch.empty((batch, m), device=DEV)
        if kind == "grouped":
            s["call"] = biq.PreparedGroup([(l["K"], l["alpha"], l["X"], l["Y"], m, n, q, batch) for l in s["layers"]], mu)
        else:
            s["LUT"] = torch.empty((biq.biq_num_chunks(n, mu), 1 << mu, batch), device=DEV)
            s["ws"] = _workspace(biq.biq_workspace_bytes(m, n, q, batch, mu))
    return s


def run(state):
    c = state["case"]
    kind = c["kind"]
    if kind == "gemm":
        state["call"]()
        return state["Y"]
    if kind == "lstm":
        state["call"]()
        return [state["H"], state["C_out"]]
    if kind == "grouped":
        state["call"]()
        return [l["Y"] for l in state["layers"]]
    if kind == "tables":
        m, n, q, batch, mu = c["m"], c["n"], c["q"], c["batch"], c["mu"]
        biq.biq_build_lut(state["layers"][0]["X"], state["LUT"], n, batch, mu)
        for l in state["layers"]:
            biq.biq_query(l["K"], l["alpha"], state["LUT"], l["Y"], m, n, q, batch, mu, workspace=state["ws"])
        return [state["LUT"]] + [l["Y"] for l in state["layers"]]
    if kind == "quantize":
        biq.biq_quantize(state["W"], state["K"], state["alpha"], c["m"], c["n"], c["q"])
        return [state["K"], state["alpha"]]
    biq.biq_pack(state["B"], state["K"], c["m"], c["n"], c["q"], 8)
    return state["K"]


def work(case):
    """Bytes: packed signs, scales, inputs and results once each.  Operations: one signed addition
    (two operations) per weight, plane and input vector."""
    kind, n, q = case["kind"], case["n"], case["q"]
    m = 4 * case["hidden"] if kind == "lstm" else case["m"]
    keys, scales = q * m * -(-n // 8), 4 * q * m
    if kind == "quantize":
        return dict(bytes=4 * m * n + keys + scales, flops=4 * q * m * n)
    if kind == "pack":
        return dict(bytes=q * m * n + keys, flops=0)
    batch, count = case["batch"], case.get("count", 1)
    x, y = 4 * n * batch, 4 * m * batch
    flops = 2 * q * m * n * batch * count
    if kind == "lstm":
        return dict(bytes=keys + scales + x + 4 * m + 3 * y // 4, flops=flops)
    if kind == "tables":
        return dict(bytes=count * (keys + scales + y) + x + -(-n // case["mu"]) * (1 << case["mu"]) * batch * 4, flops=flops)
    return dict(bytes=count * (keys + scales + x + y), flops=flops)


def tolerance(case):
    kind = case["kind"]
    if kind == "pack":
        return "exact"
    if kind == "quantize":
        # a sign may differ where the residual is within rounding of zero
        return {"rel": 2e-6, "max": 2e-5, "differ": 2e-4}
    return {"rel": 2e-6, "max": 2e-5}


# ---- the same in 64 bits, plain torch ------------------------------------------------------------------

def _multiply64(K, alpha, X, n):
    """X W^T with W = sum_i alpha_i B_i, rows in blocks."""
    q, m, _ = K.shape
    X = X.double()
    bits = torch.arange(8, device=DEV, dtype=torch.uint8)
    rows = max(1, (1 << 26) // n)
    Y = torch.empty((X.shape[0], m), dtype=torch.float64, device=DEV)
    for r in range(0, m, rows):
        W = 0
        for i in range(q):
            b = ((K[i, r:r + rows, :, None] >> bits) & 1).reshape(-1, K.shape[2] * 8)[:, :n]
            W = W + (b.double() * 2 - 1) * alpha[i, r:r + rows, None].double()
        Y[:, r:r + rows] = X @ W.t()
    return Y


def exact(case, seed):
    s = _inputs(case, seed)
    kind, n, q = case["kind"], case["n"], case["q"]
    if kind == "gemm":
        return _multiply64(s["K"], s["alpha"], s["X"], n)
    if kind == "lstm":
        z = _multiply64(s["K"], s["alpha"], s["X"], n) + s["bias"].double()
        i, f, g, o = z.chunk(4, dim=1)
        c = torch.sigmoid(f) * s["C"].double() + torch.sigmoid(i) * torch.tanh(g)
        return [torch.sigmoid(o) * torch.tanh(c), c]
    if kind in ("grouped", "tables"):
        Y = [_multiply64(l["K"], l["alpha"], l["X"], n) for l in s["layers"]]
        if kind == "grouped":
            return Y
        mu, batch = case["mu"], case["batch"]
        chunks = -(-n // mu)
        X = torch.zeros((batch, chunks * mu), dtype=torch.float64, device=DEV)
        X[:, :n] = s["layers"][0]["X"]
        k = torch.arange(1 << mu, device=DEV)
        signs = ((k[:, None] >> torch.arange(mu, device=DEV)) & 1).double() * 2 - 1
        LUT = torch.stack([X[a].reshape(chunks, mu) @ signs.t() for a in range(batch)], dim=2)
        return [LUT] + Y
    stride = -(-n // 128) * 16
    weights = torch.tensor([1, 2, 4, 8, 16, 32, 64, 128], device=DEV, dtype=torch.int32)

    def packed(positive):
        b = torch.zeros((positive.shape[0], stride * 8), dtype=torch.int32, device=DEV)
        b[:, :n] = positive
        return (b.reshape(-1, stride, 8) * weights).sum(dim=2).to(torch.uint8)

    if kind == "pack":
        return torch.stack([packed(s["B"][i] > 0) for i in range(q)])
    r = s["W"].double()
    K, alpha = [], []
    for _ in range(q):
        positive = r >= 0
        a = r.abs().mean(dim=1)
        K.append(packed(positive))
        alpha.append(a)
        r = r - torch.where(positive, a[:, None], -a[:, None])
    return [torch.stack(K), torch.stack(alpha)]
