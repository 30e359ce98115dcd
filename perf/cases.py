"""The workloads this framework is timed on.

Each case is one call of a public entry point of paper_2608_12573_amd, made
the way a serving or training loop makes it: the plan, the workspace and the
output buffers are kept from call to call, the input is new.

  vec        topk         one fp32 or bf16 vector
  rows       topk_rows    the k largest of every row of a [B, D] matrix
  batch      batchtopk    the B*k_row largest of a [B, D] matrix
  sae        sae_encode_topk   BatchTopK inside the SAE encoder
  sae_decode sae_decode        the SAE decoder on the selected latents

listed() holds the sizes of this repository's own configurations, tests and
benchmark and generic ones between them; draw() gives others of the same
ranges.
"""

import math

import torch

import paper_2608_12573_amd as pk

DEV = "cuda:0"
TORCH_DTYPE = {"f32": torch.float32, "bf16": torch.bfloat16}
CODE = {"f32": pk.F32, "bf16": pk.BF16}
MAX_BYTES = 1 << 30      # the largest listed inputs


def _vec(name, N, k, dtype="f32", dist="normal", lex=0, recall=1.0):
    return dict(name=name, kind="vec", N=N, k=k, dtype=dtype, dist=dist, lex=lex, recall=recall)


def _rows(name, B, D, k, dtype, dist, lex=0):
    return dict(name=name, kind="rows", B=B, D=D, k=k, dtype=dtype, dist=dist, lex=lex)


def listed():
    return [
        # A small vector, sorted exactly without sampling: re-ranking a
        # candidate list, a shortlist in a search.  Latency only.
        _vec("vec_f32_50000_k100", 50_000, 100),
        # The smallest sampled vector of the configurations: one 4 MiB
        # vector, where launches and latency count.
        _vec("vec_f32_2p20_k64", 1 << 20, 64, dist="uniform"),
        # Scores with a wide plateau of equal values across rank k (many
        # items of the same score): the refinement's tie handling.
        _vec("vec_f32_2p26_k512_plateau", 1 << 26, 512, dist="plateau"),
        # The headline: the 1024 largest of 2^28 values (gradient or
        # activation sparsification, large retrieval scores).
        _vec("vec_f32_2p28_k1024", 1 << 28, 1024),
        # Few long rows of odd width: sampling from the logits of a decode
        # batch (about 1e5 candidates per sequence, 64 sequences).
        _rows("rows_f32_64x100003_k50", 64, 100_003, 50, "f32", "normal"),
        # Many short rows: row-wise TopK activations of a wide layer, or
        # per-query selection among a few thousand keys.
        _rows("rows_f32_8192x4096_k64", 8192, 4096, 64, "f32", "normal"),
        # The per-row configuration: ReLU activations, one GiB of them.
        _rows("rows_bf16_4096x131072_k32", 4096, 131072, 32, "bf16", "relu"),
        # A large k per row: keeping 1/32 of each row (row-wise pruning).
        _rows("rows_bf16_16x65536_k2048", 16, 65536, 2048, "bf16", "relu"),
        # A few very long rows: top hits per query over a 4M-item index.
        _rows("rows_f32_8x2p22_k32", 8, 1 << 22, 32, "f32", "normal"),
        # BatchTopK over a GiB of SAE pre-activations, 64 kept per row.
        dict(name="batch_f32_4096x65536_k64", kind="batch", B=4096, D=65536, k_row=64, dtype="f32", recall=1.0),
        # The BatchTopK SAE layer at the paper's shape: encoder and decoder.
        dict(name="sae_4096x512x12288_k32", kind="sae", B=4096, d_model=512, d_dict=12288, k_row=32),
        dict(name="sae_decode_4096x512x12288_k32", kind="sae_decode", B=4096, d_model=512, d_dict=12288, k_row=32),
    ]


# ------------------------------------------------------------------ draws ---

def _log(rng, lo, hi):
    """An integer between lo and hi, spread over its logarithm."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    u = rng.random()
    if u < 0.35:
        dtype = "bf16" if rng.random() < 0.4 else "f32"
        N = _log(rng, 1 << 12, (1 << 28) if dtype == "f32" else (1 << 29))
        k = _log(rng, 1, min(N // 8, 16384))
        dists = ["normal", "relu"] if dtype == "bf16" else ["normal", "uniform", "pareto", "zeros90", "ramp", "plateau"]
        lex = 1 if rng.random() < 0.15 else 0
        return dict(kind="vec", N=N, k=k, dtype=dtype, dist=rng.choice(dists), lex=lex,
                    recall=0.95 if not lex and rng.random() < 0.1 else 1.0)
    if u < 0.70:
        dtype = "bf16" if rng.random() < 0.5 else "f32"
        es = 2 if dtype == "bf16" else 4
        D = _log(rng, 256, 1 << 22)
        k = _log(rng, 1, min(2048, D // 8))
        # rows that are very wide or keep very many come in small batches
        most = min(MAX_BYTES // (D * es), 16384)
        if k > 1024 or D > (1 << 18):
            most = min(most, 64)
        B = _log(rng, 1, most)
        return dict(kind="rows", B=B, D=D, k=k, dtype=dtype, dist="relu" if dtype == "bf16" else "normal",
                    lex=1 if rng.random() < 0.1 else 0)
    if u < 0.82:
        dtype = "bf16" if rng.random() < 0.3 else "f32"
        B = _log(rng, 64, 4096)
        D = _log(rng, 2048, 65536)
        return dict(kind="batch", B=B, D=D, k_row=_log(rng, 8, min(64, D // 32)), dtype=dtype,
                    recall=rng.choice([1.0, 0.95]))
    B = _log(rng, 256, 4096)
    d_model = 64 * rng.randint(2, 12 if u < 0.92 else 8)
    d_dict = _log(rng, 2048, 12288 * 512 // max(d_model, 512))
    k_row = _log(rng, 8, 32)
    return dict(kind="sae" if u < 0.92 else "sae_decode", B=B, d_model=d_model, d_dict=d_dict, k_row=k_row)


# ----------------------------------------------------------------- inputs ---

def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(seed)


def _values(n, dist, dtype, k, seed):
    """n values on the GPU.  normal, uniform: i.i.d.; pareto: shape 1.1, heavy
    tail; zeros90: nine in ten are +0; ramp: ascending; plateau: about 1e4
    equal values across rank k; relu: half are +0 (activations)."""
    g = _gen(seed)
    if dist in ("normal", "relu"):
        x = torch.randn(n, generator=g, device=DEV, dtype=torch.float32)
        if dist == "relu":
            x.clamp_(min=0.0)
    elif dist == "ramp":
        shift = torch.rand(1, generator=g, device=DEV) * 100.0
        x = torch.arange(n, device=DEV, dtype=torch.float32).add_(shift)
    else:
        x = torch.rand(n, generator=g, device=DEV, dtype=torch.float32)
        if dist == "pareto":
            x = (1.0 - x).pow_(-1.0 / 1.1)
        elif dist == "zeros90":
            keep = torch.rand(n, generator=g, device=DEV) >= 0.9
            x = x * keep
        elif dist == "plateau":
            hi, lo = 1.0 - 0.5 * k / n, 1.0 - (k + 1.0e4) / n
            if lo > 0.0:
                x[(x >= lo) & (x < hi)] = hi
    return x.to(TORCH_DTYPE[dtype])


def _preacts(B, D, dtype, seed):
    """SAE pre-activations N(-0.5, 1), one column in a hundred 3 higher."""
    x = torch.randn((B, D), generator=_gen(seed), device=DEV, dtype=torch.float32).sub_(0.5)
    x[:, ::100] += 3.0
    return x.to(TORCH_DTYPE[dtype])


def _sae_layer(case, seed):
    B, d, D = case["B"], case["d_model"], case["d_dict"]
    g = _gen(seed)
    x = torch.randn((B, d), generator=g, device=DEV).to(torch.bfloat16)
    w_enc = (torch.randn((D, d), generator=g, device=DEV) / math.sqrt(d)).to(torch.bfloat16)
    b_enc = torch.full((D,), -0.5, device=DEV)
    b_enc[::100] = 1.5
    w_dec = torch.randn((D, d), generator=g, device=DEV)
    w_dec = (w_dec / w_dec.norm(dim=1, keepdim=True)).to(torch.bfloat16)
    b_dec = torch.randn(d, generator=g, device=DEV) * 0.1
    return x, w_enc, b_enc, w_dec, b_dec


def _sae_selection(case, x, w_enc, b_enc):
    """The layer's B*k_row largest latents (what the decoder is given)."""
    z = torch.relu(x.float() @ w_enc.float().t() + b_enc).view(-1)
    vals, idx = torch.topk(z, case["B"] * case["k_row"])
    return vals, idx


def _info(n=1):
    return torch.zeros(n * pk.INFO_BYTES, dtype=torch.uint8, device=DEV)


def _outs(n, dtype):
    return torch.empty(n, dtype=TORCH_DTYPE[dtype], device=DEV), torch.empty(n, dtype=torch.int64, device=DEV)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "vec":
        x = _values(case["N"], case["dist"], case["dtype"], case["k"], seed)
        p = pk.plan(case["N"], case["k"], recall=case["recall"], lexicographic=case["lex"])
        return dict(kind=kind, x=x, k=case["k"], p=p, ws=pk.workspace(p, CODE[case["dtype"]]),
                    out=_outs(case["k"], case["dtype"]), info=_info())
    if kind == "rows":
        B, D, k = case["B"], case["D"], case["k"]
        x = _values(B * D, case["dist"], case["dtype"], k, seed).view(B, D)
        p = pk.plan_rows(D, k, lexicographic=case["lex"])
        return dict(kind=kind, x=x, k=k, p=p, ws=pk.workspace(p, CODE[case["dtype"]], B),
                    out=_outs(B * k, case["dtype"]), info=_info(B))
    if kind == "batch":
        B, D, k_row = case["B"], case["D"], case["k_row"]
        p = pk.plan(B * D, B * k_row, recall=case["recall"])
        return dict(kind=kind, x=_preacts(B, D, case["dtype"], seed), k=k_row, p=p,
                    ws=pk.workspace(p, CODE[case["dtype"]]), out=_outs(B * k_row, case["dtype"]), info=_info())
    B, d, D, k_row = case["B"], case["d_model"], case["d_dict"], case["k_row"]
    x, w_enc, b_enc, w_dec, b_dec = _sae_layer(case, seed)
    if kind == "sae":
        p = pk.plan_sae(B, D, k_row)
        return dict(kind=kind, x=x, w=w_enc, b=b_enc, k=k_row, p=p, ws=pk.sae_workspace(p, B, D),
                    out=_outs(B * k_row, "f32"), info=_info())
    vals, idx = _sae_selection(case, x, w_enc, b_enc)
    ws = torch.empty(pk.lib().profk_sae_decode_workspace_size(B, B * k_row), dtype=torch.uint8, device=DEV)
    return dict(kind=kind, vals=vals, idx=idx, w=w_dec, b=b_dec, B=B, ws=ws,
                out=torch.empty((B, d), dtype=torch.float32, device=DEV))


def run(s):
    kind = s["kind"]
    if kind == "vec":
        return pk.topk(s["x"], s["k"], p=s["p"], ws=s["ws"], out=s["out"], info=s["info"])
    if kind == "rows":
        return pk.topk_rows(s["x"], s["k"], p=s["p"], ws=s["ws"], out=s["out"], info=s["info"])
    if kind == "batch":
        return pk.batchtopk(s["x"], s["k"], p=s["p"], ws=s["ws"], out=s["out"], info=s["info"])
    if kind == "sae":
        return pk.sae_encode_topk(s["x"], s["w"], s["b"], s["k"], p=s["p"], ws=s["ws"], out=s["out"], info=s["info"])
    return pk.sae_decode(s["vals"], s["idx"], s["w"], s["b"], s["B"], out=s["out"], ws=s["ws"])


def work(case):
    kind = case["kind"]
    if kind in ("vec", "rows", "batch"):
        es = 2 if case["dtype"] == "bf16" else 4
        if kind == "vec":
            n, k, calls = case["N"], case["k"], 1
        elif kind == "rows":
            n, k, calls = case["B"] * case["D"], case["B"] * case["k"], case["B"]
        else:
            n, k, calls = case["B"] * case["D"], case["B"] * case["k_row"], 1
        return {"bytes": n * es + k * (es + 8) + calls * pk.INFO_BYTES, "flops": 0}
    B, d, D, K = case["B"], case["d_model"], case["d_dict"], case["B"] * case["k_row"]
    if kind == "sae":
        return {"bytes": 2 * d * (B + D) + 4 * D + 12 * K + pk.INFO_BYTES, "flops": 2 * B * d * D}
    return {"bytes": 12 * K + 2 * d * min(D, K) + 4 * d + 4 * B * d, "flops": 2 * K * d}


def tolerance(case):
    # Selections are integer work: the same keys, indices and counts.  So are
    # the SAE encoder's, of the fp32 latents that its encoder GEMM gives; its
    # sums in another order move a latent by about 1e-7 of its size, which
    # swaps neighbours in the sorted list of 1e5 latents.
    if case["kind"] == "sae":
        return {"rel": 4e-7, "max": 1e-5, "differ": 0.01}   # measured: 9.5e-8 from 64 bits
    if case["kind"] == "sae_decode":   # fp32 sums of about 32 products
        return {"rel": 5e-7, "max": 1e-5}   # measured: 1.1e-7 from 64 bits
    return "exact"


# ------------------------------------------------------------- in 64 bits ---

def _ordered(x):
    """An integer per value that orders as the value does (the repository's
    total order: by bit pattern, so that -0 lies below +0)."""
    if x.dtype == torch.float32:
        b = x.view(torch.int32).to(torch.int64)
        return torch.where(b < 0, -(b & 0x7FFFFFFF) - 1, b)
    b = x.view(torch.int16).to(torch.int64)
    return torch.where(b < 0, -(b & 0x7FFF) - 1, b)


def _exact_rows(x, k):
    """Largest first, equal values by smaller index: one 64-bit integer per
    element holds both."""
    B, D = x.shape
    vals, idx = [], []
    step = max(1, (1 << 28) // D)
    low = (1 << 32) - 1 - torch.arange(D, device=x.device, dtype=torch.int64)
    for r in range(0, B, step):
        part = x[r:r + step]
        c = _ordered(part.contiguous().view(-1)).view(part.shape) * (1 << 32) + low
        if part.shape[0] == 1:
            top = torch.sort(c.view(-1), descending=True).values[:k].view(1, k)
        else:
            top = torch.topk(c, k, dim=1).values
        i = (1 << 32) - 1 - (top & ((1 << 32) - 1))
        idx.append(i)
        vals.append(torch.gather(part, 1, i))
    return torch.cat(vals), torch.cat(idx)


def exact(case, seed):
    kind = case["kind"]
    if kind in ("vec", "batch") and case["recall"] < 1.0:
        return None    # a relaxed call may return a shorter exact prefix
    if kind == "vec":
        x = _values(case["N"], case["dist"], case["dtype"], case["k"], seed)
        v, i = _exact_rows(x.view(1, -1), case["k"])
        return v.view(-1).double(), i.view(-1), None
    if kind == "rows":
        x = _values(case["B"] * case["D"], case["dist"], case["dtype"], case["k"], seed)
        v, i = _exact_rows(x.view(case["B"], case["D"]), case["k"])
        return v.double(), i, None
    if kind == "batch":
        x = _preacts(case["B"], case["D"], case["dtype"], seed)
        v, i = _exact_rows(x.view(1, -1), case["B"] * case["k_row"])
        return v.view(-1).double(), i.view(-1), None
    x, w_enc, b_enc, w_dec, b_dec = _sae_layer(case, seed)
    K = case["B"] * case["k_row"]
    if kind == "sae":
        z = torch.relu(x.double() @ w_enc.double().t() + b_enc.double()).view(-1)
        # (which of two latents closer than the 32-bit rounding comes first
        # is not determined, so their order has no value in 64 bits)
        return torch.sort(z, descending=True).values[:K], None, None
    vals, idx = _sae_selection(case, x, w_enc, b_enc)
    D = case["d_dict"]
    out = b_dec.double().expand(case["B"], -1).clone()
    for e in range(0, K, 1 << 16):
        r, j = idx[e:e + (1 << 16)] // D, idx[e:e + (1 << 16)] % D
        out.index_add_(0, r, vals[e:e + (1 << 16), None].double() * w_dec[j].double())
    return out
