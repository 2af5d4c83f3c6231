"""The calls whose speed matters to a user of this framework, as measurable cases.

A user steps token tables: the LM head and the input embedding of a language
model (or one tied table), once per training step, in the middle of a run
(r and c hold the statistics of earlier steps).  The cases go through the
Python entry points such a training loop calls: ``EmberTable.step``,
``step_sparse_rows``, ``step_tokens``, ``step_lmhead`` and ``step_tables``.

A case is a dict of plain values: ``kind`` (the entry point), the table
``V`` x ``D``, the storage types ``w`` and ``g`` of weights and gradients,
``tokens`` (sparse kinds: batch positions, LM head: rows of the logits
gradient), ``row_only`` (the row-only variant) and ``maximize``.
"""
from __future__ import annotations

import math

import torch

DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16}
LR, BETA2, EPS = 1e-3, 0.999, 1e-8
STEPS_BEFORE = 200       # the step that is measured first is number 201
ZIPF_EXPONENT = 1.1      # token frequencies
W_STD, G_STD = 0.02, 1e-3
CHUNK_ELEMS = 1 << 26    # elements made or checked at a time


def _case(kind, V, D, w="bf16", g="bf16", tokens=0, row_only=False, maximize=False, name=None):
    c = {"kind": kind, "V": V, "D": D, "w": w, "g": g, "tokens": tokens, "row_only": row_only,
         "maximize": maximize}
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # The smallest table anyone steps: a toy model's head.  Launches and latency.
        _case("dense", 1024, 64, "f32", "f32", name="dense_tiny_f32"),
        # A small model's table with ragged sizes, fp32 main gradients on bf16 weights, and the
        # ascent form (a reward is maximised).
        _case("dense", 8191, 1000, "bf16", "f32", maximize=True, name="dense_8k_ragged_mixed"),
        # An fp32 LM head of a 32k vocabulary.
        _case("dense", 32000, 4096, "f32", "f32", name="dense_lmhead32k_f32"),
        # A tall, narrow tied table in fp32.
        _case("dense", 151936, 896, "f32", "f32", name="dense_tied152k_f32"),
        # Both untied tables of a large-vocabulary model in one call: a dense LM head and the
        # embedding rows of an 8 x 2048-token batch.
        _case("multi", 128256, 4096, tokens=16384, name="multi_head_embed128k"),
        # The embedding step of one short sequence.
        _case("sparse", 128256, 4096, tokens=2048, name="sparse_embed128k_2k"),
        # The embedding step of a large batch: too many distinct rows to stay on chip.
        _case("sparse", 128256, 4096, tokens=65536, name="sparse_embed128k_64k"),
        # Token ids and per-position gradients of an 8 x 2048 batch -> summed rows -> step.
        _case("tokens", 128256, 4096, tokens=16384, name="tokens_embed128k_16k"),
        # The same for a small fp32 model with an odd width and a short batch.
        _case("tokens", 32000, 1023, "f32", "f32", tokens=1000, name="tokens_32k_odd_f32"),
        # Row-only variant of the two-table step.
        _case("multi", 128256, 4096, tokens=16384, row_only=True, name="rowonly_head_embed128k"),
        # LM-head step from logits gradient and hidden states, a short batch of a 32k fp32 head.
        _case("lmhead", 32000, 4096, "f32", "f32", tokens=2048, name="lmhead32k_2k_f32"),
        # The same at 8 x 2048 tokens and a 128k vocabulary: the largest call.
        _case("lmhead", 128256, 4096, tokens=16384, name="lmhead128k_16k"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["dense", "dense", "sparse", "tokens", "lmhead", "multi"])
    w, g = rng.choice([("bf16", "bf16"), ("bf16", "bf16"), ("f32", "f32"), ("bf16", "f32")])
    row_only = kind != "lmhead" and rng.random() < 0.25
    while True:
        V = _log_int(rng, 1000, 262144)
        D = _log_int(rng, 64, 4096 if kind == "lmhead" else 8192)
        shape = rng.random()
        if shape < 0.6:      # most widths are multiples of 64
            D = max(64, D // 64 * 64)
        elif shape < 0.85:   # others whole 16-byte chunks
            D = max(64, D // 8 * 8)
        tokens = 0
        if kind == "lmhead":
            tokens = _log_int(rng, 256, 16384)
            # at most the largest listed case's work
            if tokens * V * D > 16384 * 128256 * 4096:
                continue
        elif kind != "dense":
            tokens = _log_int(rng, 256, 65536)
            if kind == "tokens" and tokens > V:   # a device-count step takes at most V rows
                continue
        return _case(kind, V, D, w, g, tokens, row_only, rng.random() < 0.25)


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _gen(device, seed, part):
    g = torch.Generator(device=device)
    g.manual_seed((int(seed) * 1000003 + part) % (2 ** 63 - 1))
    return g


def _padded(rows, D, dtype, device):
    """A rows x D tensor whose rows start on 16-byte boundaries."""
    q = 16 // torch.empty(0, dtype=dtype).element_size()
    return torch.empty(max(rows, 1), (D + q - 1) // q * q, dtype=dtype, device=device)[:rows, :D]


def _normal(rows, D, std, dtype, device, gen, row_scale=None):
    out = _padded(rows, D, dtype, device)
    step = max(1, CHUNK_ELEMS // D)
    for r0 in range(0, rows, step):
        r1 = min(rows, r0 + step)
        x = torch.randn(r1 - r0, D, generator=gen, device=device) * std
        if row_scale is not None:
            x *= row_scale[r0:r1, None]
        out[r0:r1] = x.to(dtype)
    return out


def _zipf(V):
    p = torch.arange(1, V + 1, dtype=torch.float64).pow(-ZIPF_EXPONENT)
    return p / p.sum()


def _ids(V, tokens, seed, part):
    return torch.multinomial(_zipf(V).float(), tokens, replacement=True, generator=_gen("cpu", seed, part))


def _history(V, D, row_rms, device, gen):
    """r and c after STEPS_BEFORE steps of gradients with these row scales."""
    seen = 1.0 - BETA2 ** STEPS_BEFORE
    e = row_rms.double().square()
    r = (e * seen * (0.5 + torch.rand(V, generator=gen, device=device, dtype=torch.float64))).float()
    c = (e.mean() * seen * (0.5 + torch.rand(D, generator=gen, device=device, dtype=torch.float64))).float()
    return r, c


def _dense_table(case, seed, device):
    V, D = case["V"], case["D"]
    scale = (_zipf(V) * V).float().to(device)   # row norm follows token frequency
    gen = _gen(device, seed, 1)
    x = {"W": _normal(V, D, W_STD, DTYPES[case["w"]], device, gen),
         "G": _normal(V, D, G_STD, DTYPES[case["g"]], device, gen, scale)}
    x["r"], x["c"] = _history(V, D, scale * G_STD, device, gen)
    return x


def _sparse_table(case, seed, device, coalesced):
    V, D, dt = case["V"], case["D"], DTYPES[case["g"]]
    tok = _ids(V, case["tokens"], seed, 2)
    idx, counts = torch.unique(tok, sorted=True, return_counts=True)
    gen = _gen(device, seed, 3)
    x = {"W": _normal(V, D, W_STD, DTYPES[case["w"]], device, gen)}
    if coalesced:   # a row that occurs k times: the sum of k independent signals
        x["idx"] = idx.to(device)
        x["G"] = _normal(idx.numel(), D, G_STD, dt, device, gen, counts.to(device).float().sqrt())
    else:
        x["tok"] = tok.to(device)
        x["U"] = _normal(case["tokens"], D, G_STD, dt, device, gen)
    often = (_zipf(V) * case["tokens"]).float().sqrt().to(device)
    x["r"], x["c"] = _history(V, D, often * G_STD, device, gen)
    return x


def _lmhead_table(case, seed, device):
    V, D, T = case["V"], case["D"], case["tokens"]
    gen = _gen(device, seed, 4)
    p = _zipf(V)
    y = _ids(V, T, seed, 5).to(device)
    logp = p.log().float().to(device)
    H = _normal(T, D, 1.0, torch.bfloat16, device, gen)
    dY = _padded(T, V, torch.bfloat16, device)
    step = max(1, CHUNK_ELEMS // V)
    for m0 in range(0, T, step):   # softmax that follows the token frequencies, minus the targets
        m1 = min(T, m0 + step)
        q = torch.softmax(torch.randn(m1 - m0, V, generator=gen, device=device) + logp, dim=1)
        q[torch.arange(m1 - m0, device=device), y[m0:m1]] -= 1.0
        dY[m0:m1] = (q / T).to(torch.bfloat16)
    x = {"W": _normal(V, D, W_STD, DTYPES[case["w"]], device, gen), "dY": dY, "H": H,
         "G": _padded(V, D, DTYPES[case["g"]], device)}
    x["r"], x["c"] = _history(V, D, (p / T).float().sqrt().to(device), device, gen)
    return x


def _inputs(case, seed, device):
    """The tables of a case: one, or the dense head and the sparse embedding."""
    kind = case["kind"]
    if kind == "dense":
        return [_dense_table(case, seed, device)]
    if kind == "sparse":
        return [_sparse_table(case, seed, device, True)]
    if kind == "tokens":
        return [_sparse_table(case, seed, device, False)]
    if kind == "lmhead":
        return [_lmhead_table(case, seed, device)]
    return [_dense_table(case, seed, device), _sparse_table(case, seed + 7919, device, True)]


def prepare(case, seed):
    from paper_2607_01455_amd import ember

    device = torch.device("cuda")
    s = {"ember": ember, "case": case, "tables": []}
    for x in _inputs(case, seed, device):
        tab = ember.EmberTable(case["V"], case["D"], device=device, lr=LR, beta2=BETA2, eps=EPS,
                               maximize=case["maximize"], row_only=case["row_only"])
        tab.r.copy_(x["r"])
        if not case["row_only"]:
            tab.c.copy_(x["c"])
        tab.t = STEPS_BEFORE
        x["table"] = tab
        s["tables"].append(x)
    if case["kind"] == "tokens":
        s["coalescer"] = ember.Coalescer(case["tokens"], case["V"], case["D"], dtype=DTYPES[case["g"]],
                                         device=device)
        s["coalescer"].idx.zero_()      # rows past the batch's distinct ids are not written
        s["coalescer"].G_rows.zero_()
    return s


def _state(x):
    tab = x["table"]
    return [x["W"], tab.r] if tab.c is None else [x["W"], tab.r, tab.c]


def run(state):
    kind, tables = state["case"]["kind"], state["tables"]
    x = tables[0]
    if kind == "dense":
        x["table"].step(x["W"], x["G"])
        return _state(x)
    if kind == "sparse":
        x["table"].step_sparse_rows(x["W"], x["G"], x["idx"])
        return _state(x)
    if kind == "tokens":
        co = state["coalescer"]
        x["table"].step_tokens(x["W"], x["tok"], x["U"], co)
        return _state(x) + [co.n_out, co.idx, co.G_rows]
    if kind == "lmhead":
        x["table"].step_lmhead(x["W"], x["dY"], x["H"], x["G"])
        return _state(x) + [x["G"]]
    e = tables[1]
    state["ember"].step_tables([(x["table"], x["W"], x["G"]), (e["table"], e["W"], e["G"], e["idx"])])
    return _state(x) + _state(e)


# ---------------------------------------------------------------------------
# work, tolerance, and the same results in 64 bits
# ---------------------------------------------------------------------------

def _expected_rows(case):
    """Expected distinct ids of a batch: a number every seed comes close to."""
    return float((1.0 - torch.exp(case["tokens"] * torch.log1p(-_zipf(case["V"])))).sum())


def work(case):
    """Each input read once, each output written once.  The canonical dense
    step needs every gradient before the first weight changes, and still counts
    the gradient once."""
    V, D, kind, T = case["V"], case["D"], case["kind"], case["tokens"]
    w, g = (2 if case[k] == "bf16" else 4 for k in ("w", "g"))
    state = 8 * V + (0 if case["row_only"] else 8 * D)
    dense = V * D * (g + 2 * w) + state
    flops = 0
    if kind == "dense":
        return {"bytes": dense, "flops": flops}
    if kind == "lmhead":
        return {"bytes": 2 * T * (V + D) + V * D * (g + 2 * w) + state, "flops": 2 * T * V * D}
    n = _expected_rows(case)
    sparse = n * D * (g + 2 * w) + 8 * n + state
    if kind == "sparse":
        return {"bytes": sparse, "flops": flops}
    if kind == "tokens":   # ids and signals in, ids and summed rows out, weights in and out
        return {"bytes": 8 * T + T * D * g + n * (8 + D * g) + 2 * n * D * w + state, "flops": flops}
    return {"bytes": dense + sparse, "flops": flops}


def tolerance(case):
    """About four times the distance from the correctly rounded float64 result,
    measured over the listed cases and a few drawn ones: the fp32 state is
    within 4e-8, fp32 weights within 2e-8 (4e-7 per element), fp32 G of the LM
    head within 3e-7 (3e-5 per element); bf16 weights and G differ by one ulp
    (at most 2^-7 of an element) in a few of 1e6 elements (5e-6 in all; G of the
    LM head: 6 of 1e4, 5e-5)."""
    lmhead = case["kind"] == "lmhead"
    if "bf16" in (case["w"], case["g"]):
        return {"rel": 2e-4 if lmhead else 2e-5, "max": 0.016}
    return {"rel": 1.2e-6 if lmhead else 2e-7, "max": 1.3e-4 if lmhead else 2e-6}


def _step64(x, G, idx, case):
    """One step in float64: the new (W, r, c)."""
    dev = x["W"].device
    V, D = case["V"], case["D"]
    b2 = float(torch.tensor(BETA2, dtype=torch.float32))
    lr = float(torch.tensor(LR, dtype=torch.float32))
    eps = float(torch.tensor(EPS, dtype=torch.float32))
    n = G.shape[0]
    step = max(1, CHUNK_ELEMS // D)
    row = torch.zeros(V, dtype=torch.float64, device=dev)
    col = torch.zeros(D, dtype=torch.float64, device=dev)
    for r0 in range(0, n, step):
        q = G[r0:r0 + step].double().square()
        at = slice(r0, r0 + q.shape[0]) if idx is None else idx[r0:r0 + step]
        row[at] = q.mean(dim=1)
        col += q.sum(dim=0)
    bias = 1.0 - b2 ** (STEPS_BEFORE + 1)
    r = b2 * x["r"].double() + (1.0 - b2) * row
    c = b2 * x["c"].double() + (1.0 - b2) * col / V
    s = torch.sqrt((r / bias).mean() * (c / bias).mean())
    W = x["W"].double()
    sign = lr if case["maximize"] else -lr
    for r0 in range(0, n, step):
        g = G[r0:r0 + step].double()
        at = slice(r0, r0 + g.shape[0]) if idx is None else idx[r0:r0 + step]
        if case["row_only"]:
            v = (r[at] / bias)[:, None]
        else:
            v = (r[at] / bias)[:, None] * (c / bias)[None, :] / s
        W[at] += sign * g / (v.sqrt() + eps)
    return [W, r] if case["row_only"] else [W, r, c]


def exact(case, seed):
    device = torch.device("cuda")
    kind, out = case["kind"], []
    for x in _inputs(case, seed, device):
        idx, extra, G = x.get("idx"), [], x.get("G")
        if kind == "tokens":
            idx, inv = torch.unique(x["tok"], sorted=True, return_inverse=True)
            G64 = torch.zeros(case["tokens"], case["D"], dtype=torch.float64, device=device)
            G64.index_add_(0, inv, x["U"].double())
            n = idx.numel()
            all_idx = torch.zeros(case["tokens"], dtype=torch.int64, device=device)
            all_idx[:n] = idx
            extra = [torch.tensor([n], device=device), all_idx, G64]
            G = G64[:n].to(DTYPES[case["g"]])     # the step takes the stored rows
        elif kind == "lmhead":
            G64 = torch.empty(case["V"], case["D"], dtype=torch.float64, device=device)
            H64 = x["H"].double()
            for v0 in range(0, case["V"], 8192):
                G64[v0:v0 + 8192] = x["dY"][:, v0:v0 + 8192].double().t().contiguous() @ H64
            extra = [G64]
            G = G64.to(DTYPES[case["g"]])
        out += _step64(x, G, idx, case) + extra
    return out
