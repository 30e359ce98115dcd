"""GPU parity of the BatchTopK SAE layer (encoder GEMM with the fused
filter, selection, sparse decode) against the fp64 oracle (oracle.sae).

The GPU sums bf16 products in fp32 on the matrix cores, one rounding per
16-product step (and its accumulator) plus one for the bias, so a latent
may differ from the exact value by at most
    tol = (2 * d_model / 16 + 2) * 2^-24 * (sum_m |x w| + |b|).
Selections are compared modulo that: every selected latent equals the exact
value within tol, and the selected and exact sets differ only by latents
within 2 tol_max of the K-th exact value (near-ties under rounding)."""

import numpy as np
import pytest

import paper_2608_12573_amd as pk
import workloads
from oracle import sae as osae
from gpu_util import gpu_bf16, note, torch

pytestmark = pytest.mark.gpu

U = 2.0 ** -24


def _dev(m):
    t = torch()
    bf = lambda a: t.from_numpy(np.ascontiguousarray(a).view(np.int16)).cuda().view(t.bfloat16)
    return dict(x=bf(m["x"]), w_enc=bf(m["w_enc"]), b_enc=t.from_numpy(m["b_enc"]).cuda(),
                w_dec=bf(m["w_dec"]), b_dec=t.from_numpy(m["b_dec"]).cuda())


def _tol(m):
    d_model = m["x"].shape[1]
    return (2 * d_model / 16 + 2) * U * osae.encode_scale(m["x"], m["w_enc"], m["b_enc"])


def _check_selection(vals, idx, z, tol, K):
    """vals/idx: the GPU's selection; z, tol: exact latents and bounds."""
    zf, tf = z.reshape(-1), tol.reshape(-1)
    n_valid = int((idx >= 0).sum())
    assert n_valid == K
    assert np.unique(idx).size == K
    assert np.all(np.abs(vals - zf[idx]) <= tf[idx]), "a selected latent differs from its exact value"
    # sorted under the total order
    assert np.all(vals[:-1] >= vals[1:])
    same = vals[:-1] == vals[1:]
    assert np.all(idx[:-1][same] < idx[1:][same])
    ev, ei = osae.batchtopk(z, K)
    kth, tmax = ev[-1], tf.max()
    gpu_only = np.setdiff1d(idx, ei)
    exact_only = np.setdiff1d(ei, idx)
    assert gpu_only.size == exact_only.size
    assert np.all(zf[gpu_only] >= kth - 2 * tmax)
    assert np.all(zf[exact_only] <= kth + 2 * tmax)
    return gpu_only.size


@pytest.mark.parametrize("B,d_model,d_dict", [(200, 128, 300), (256, 512, 1024), (1, 64, 129), (300, 192, 700)])
def test_sae_dense_latents(B, d_model, d_dict):
    m = workloads.sae_model(B=B, d_model=d_model, d_dict=d_dict, seed=B + d_dict)
    note(f"sae dense B={B} d_model={d_model} d_dict={d_dict}")
    g = _dev(m)
    z_gpu = pk.sae_encode_dense(g["x"], g["w_enc"], g["b_enc"]).cpu().numpy().astype(np.float64)
    z = osae.encode(m["x"], m["w_enc"], m["b_enc"])
    assert np.all(np.abs(z_gpu - z) <= _tol(m))
    assert np.all(z_gpu >= 0) and not np.any(np.signbit(z_gpu))   # +0.0 for inactive latents


def test_sae_sampled_latents_are_the_gemm_values():
    # internal consistency: stage 1 computes each draw's latent with the GEMM's
    # own MFMA sequence, so its key equals the dense latent's key bit for bit
    t = torch()
    B, d_model, d_dict = 256, 512, 2048
    m = workloads.sae_model(B=B, d_model=d_model, d_dict=d_dict, seed=7)
    g = _dev(m)
    p = pk.plan(B * d_dict, B * 16, 1e-6, 1.0, S_min=4096, S_max=4096, force_mode=pk.FORCE_FILTER)
    note(f"sae sample S={p.S}")
    keys = pk.debug_sae_sample(g["x"], g["w_enc"], g["b_enc"], p, seed=3).cpu().numpy()
    idx = pk.debug_sample_indices(3, 0, p.S, B * d_dict).cpu().numpy()
    dense = pk.sae_encode_dense(g["x"], g["w_enc"], g["b_enc"]).reshape(-1)
    bits = dense.view(t.int32).cpu().numpy().astype(np.int64) & 0xFFFFFFFF
    assert np.array_equal(keys, bits[idx] ^ 0x80000000)     # latents are >= +0: key = bits with the sign set


@pytest.mark.parametrize("B,d_model,d_dict,k_row", [(256, 512, 2048, 32), (300, 128, 1000, 8), (128, 256, 4096, 4),
                                                   (200, 192, 700, 8), (64, 64, 513, 4)])
def test_sae_encode_topk(B, d_model, d_dict, k_row):
    m = workloads.sae_model(B=B, d_model=d_model, d_dict=d_dict, seed=11)
    g = _dev(m)
    K = B * k_row
    p = pk.plan(B * d_dict, K)
    note(f"sae topk B={B} d_model={d_model} d_dict={d_dict} K={K} S={p.S} t={p.t} M={p.M} mode={p.mode}")
    vals, idx, info = pk.sae_encode_topk(g["x"], g["w_enc"], g["b_enc"], k_row, seed=5, p=p)
    rec = pk.read_info(info)[0]
    assert int(rec["status"]) in (0, 3)   # filtered (or the plan's exact path)
    z = osae.encode(m["x"], m["w_enc"], m["b_enc"])
    _check_selection(vals.cpu().numpy().astype(np.float64), idx.cpu().numpy(), z, _tol(m), K)
    # internal consistency: the exact top-K of the GPU's own latents, bit for bit
    t = torch()
    dense = pk.sae_encode_dense(g["x"], g["w_enc"], g["b_enc"]).reshape(-1).cpu().numpy()
    order = np.lexsort((np.arange(dense.size), -dense.astype(np.float64)))[:K]
    assert np.array_equal(idx.cpu().numpy(), order)
    assert np.array_equal(vals.cpu().numpy().view(np.uint32), dense[order].view(np.uint32))


def _exact_topk_of(dense, K):
    """Indices of the K largest of a flat fp32 array under the total order
    (value descending, then index ascending), and their values."""
    d64 = dense.astype(np.float64)
    kth = np.partition(-d64, K - 1)[K - 1]            # minus the K-th largest value
    cand = np.nonzero(-d64 <= kth)[0]                  # every index with a value >= it
    order = cand[np.lexsort((cand, -d64[cand]))][:K]
    return order, dense[order]


@pytest.mark.parametrize("B,d_model,d_dict,k_row", [(4096, 128, 8192, 8), (4000, 192, 8000, 8), (4096, 64, 8192, 8)])
def test_sae_encode_topk_several_tiles_per_workgroup(B, d_model, d_dict, k_row):
    # more 256 x 256 filter tiles than workgroups: the next tile's loads
    # overlap an epilogue, and a tile's survivors are appended during the
    # next tile (an even d_model / 64), or each tile loads behind its own
    # barrier (odd: 3 chunks, and 1); the last row and column tiles are
    # partial in the second
    m = workloads.sae_model(B=B, d_model=d_model, d_dict=d_dict, seed=23)
    g = _dev(m)
    K = B * k_row
    p = pk.plan_sae(B, d_dict, k_row)
    note(f"sae topk tiles B={B} d_model={d_model} d_dict={d_dict} K={K} S={p.S} t={p.t} M={p.M} mode={p.mode}")
    vals, idx, info = pk.sae_encode_topk(g["x"], g["w_enc"], g["b_enc"], k_row, seed=3, p=p)
    assert int(pk.read_info(info)[0]["status"]) == 0
    dense = pk.sae_encode_dense(g["x"], g["w_enc"], g["b_enc"]).reshape(-1).cpu().numpy()
    order, ov = _exact_topk_of(dense, K)
    assert np.array_equal(idx.cpu().numpy(), order)
    assert np.array_equal(vals.cpu().numpy().view(np.uint32), ov.view(np.uint32))


def test_sae_encode_topk_default_plan():
    # the binding's default plan (profk_default_sae_opts: the sample floor)
    B, d_model, d_dict, k_row = 512, 256, 4096, 16
    m = workloads.sae_model(B=B, d_model=d_model, d_dict=d_dict, seed=19)
    g = _dev(m)
    p = pk.plan_sae(B, d_dict, k_row)
    note(f"sae default plan S={p.S} t={p.t} M={p.M} mode={p.mode}")
    vals, idx, info = pk.sae_encode_topk(g["x"], g["w_enc"], g["b_enc"], k_row, seed=1)
    assert int(pk.read_info(info)[0]["status"]) in (0, 3)
    z = osae.encode(m["x"], m["w_enc"], m["b_enc"])
    _check_selection(vals.cpu().numpy().astype(np.float64), idx.cpu().numpy(), z, _tol(m), B * k_row)


def test_sae_encode_topk_fallback():
    # a 64-draw sample with a small buffer overflows: the dense latents are
    # written to the workspace and selected exactly
    B, d_model, d_dict, k_row = 128, 128, 512, 8
    m = workloads.sae_model(B=B, d_model=d_model, d_dict=d_dict, seed=13)
    g = _dev(m)
    K = B * k_row
    p = pk.plan(B * d_dict, K, 1e-6, 1.0, S_min=64, S_max=64, force_mode=pk.FORCE_FILTER)
    p.M = K   # too small for the survivors of a 64-draw threshold
    note(f"sae fallback K={K} S={p.S} t={p.t} M={p.M}")
    vals, idx, info = pk.sae_encode_topk(g["x"], g["w_enc"], g["b_enc"], k_row, seed=2, p=p)
    rec = pk.read_info(info)[0]
    assert int(rec["status"]) in (1, 2)
    z = osae.encode(m["x"], m["w_enc"], m["b_enc"])
    _check_selection(vals.cpu().numpy().astype(np.float64), idx.cpu().numpy(), z, _tol(m), K)


@pytest.mark.parametrize("B,d_model,d_dict,k_row", [(64, 512, 2048, 32), (37, 96, 300, 5)])
def test_sae_decode(B, d_model, d_dict, k_row):
    t = torch()
    m = workloads.sae_model(B=B, d_model=d_model, d_dict=d_dict, seed=17)
    z = osae.encode(m["x"], m["w_enc"], m["b_enc"])
    K = B * k_row
    v64, i64 = osae.batchtopk(z, K)
    v32 = v64.astype(np.float32)
    # padding and a shuffled order must not change the result
    perm = np.random.default_rng(0).permutation(K)
    vals = np.r_[v32[perm], np.float32(-np.inf), np.float32(5.0)]
    idx = np.r_[i64[perm], -1, B * d_dict + 3].astype(np.int64)
    note(f"sae decode B={B} d_model={d_model} d_dict={d_dict} K={K}")
    g = _dev(m)
    out = pk.sae_decode(t.from_numpy(vals).cuda(), t.from_numpy(idx).cuda(), g["w_dec"], g["b_dec"], B)
    ref = osae.decode(v32, i64, m["w_dec"], m["b_dec"], B)
    scale = osae.decode_scale(v32, i64, m["w_dec"], m["b_dec"], B)
    per_row = np.bincount(i64 // d_dict, minlength=B)
    tol = ((per_row + 2) * U)[:, None] * scale
    got = out.cpu().numpy().astype(np.float64)
    assert np.all(np.abs(got - ref) <= tol)
    # the same entries in the oracle's order give the same bits
    out2 = pk.sae_decode(t.from_numpy(v32).cuda(), t.from_numpy(i64).cuda(), g["w_dec"], g["b_dec"], B)
    assert t.equal(out.view(t.int32), out2.view(t.int32))


@pytest.mark.parametrize("B,d_model,d_dict,kind", [
    (1, 64, 100, "spread"),           # one row, one wave's columns only in part
    (300, 72, 1000, "spread"),        # two rows a workgroup, columns past a wave's in part
    (4099, 40, 70, "spread"),         # sixteen rows a workgroup, more workgroups than CUs
    (20000, 8, 200, "dense"),         # several workgroups a group, many chunks
    (2, 64, 16384, "full"),           # a single group
    (4096, 33, 96, "spread"),         # columns not a multiple of eight
    (520, 64, 16384, "hot"),          # one row with more entries than are held at once
    (600, 64, 9000, "full"),          # three neighbouring rows, too many together
    (256, 16, 2048, "half"),          # one row a workgroup, long chunks
    (4096, 8, 512, "half"),           # sixteen rows a workgroup, more entries than it holds, long chunks
    (4100, 24, 600, "half"),          # the same, the last workgroup and chunk in part
    (24, 16, 16384, "half"),          # the largest count held at once, few workgroups
    (3, 512, 3000, "half"),           # one row's columns over the waves
    (250, 1024, 40, "half"),          # 16 pieces of 64 columns: a column a lane
    (250, 1032, 40, "half"),          # 17 pieces: eight columns a lane
    (250, 1984, 150, "half"),         # 31 pieces and more than 64 entries a row: a column a lane
    (250, 1992, 150, "half"),         # 32 pieces: eight columns a lane
    (1000, 512, 4500, "some"),        # a few dense rows, taken in runs, eight columns a lane
])
def test_decode_layouts(B, d_model, d_dict, kind):
    """Rows per workgroup, column remainders, workgroups per group, and rows
    with too many entries, against fp64: each output is a sum of its
    terms in fp32, so it is within (terms + 2) * 2^-24 of the sum of their
    magnitudes.  Padding and out-of-range entries are skipped."""
    t = torch()
    g = np.random.default_rng(B + d_model)
    if kind == "spread":
        idx = g.choice(B * d_dict, min(B * d_dict // 3, 20 * B), replace=False)
    elif kind == "dense":
        idx = g.choice(B * d_dict, B * d_dict // 4, replace=False)
    elif kind == "hot":
        idx = np.concatenate([5 * d_dict + np.arange(d_dict), 400 * d_dict + np.arange(0, d_dict, 7)])
    elif kind == "half":
        idx = np.flatnonzero(g.random(B * d_dict) < 0.5)
    elif kind == "some":
        idx = np.concatenate([r * d_dict + g.permutation(d_dict)[:d_dict // 2 if r in (4, 5, 6, 7, 500, 501, 502) else 1]
                              for r in range(B)])
    else:
        idx = np.concatenate([r * d_dict + np.arange(d_dict - 2) for r in {0, 1, B // 2, B - 1}])
    idx = g.permutation(idx).astype(np.int64)
    idx = np.concatenate([idx, [-1, B * d_dict, -5]])
    vals = g.standard_normal(idx.size).astype(np.float32)
    wb = workloads.f32_to_bf16_bits(g.standard_normal((d_dict, d_model)).astype(np.float32))
    bias = g.standard_normal(d_model).astype(np.float32)
    note(f"decode B={B} d_model={d_model} d_dict={d_dict} K={idx.size} {kind}")
    out = pk.sae_decode(t.from_numpy(vals).cuda(), t.from_numpy(idx).cuda(), gpu_bf16(wb).view(d_dict, d_model),
                        t.from_numpy(bias).cuda(), B).cpu().numpy()
    w = (wb.astype(np.uint32) << 16).view(np.float32).astype(np.float64)
    ok = (idx >= 0) & (idx < B * d_dict)
    r, j, v = idx[ok] // d_dict, idx[ok] % d_dict, vals[ok].astype(np.float64)
    ref = np.tile(bias.astype(np.float64), (B, 1))
    mag = np.abs(ref)
    np.add.at(ref, r, v[:, None] * w[j])
    np.add.at(mag, r, np.abs(v[:, None] * w[j]))
    terms = np.bincount(r, minlength=B)[:, None]
    assert np.all(np.abs(out - ref) <= (terms + 2) * 2.0**-24 * mag)


@pytest.mark.parametrize("B,d_model,d_dict,share", [
    (1000, 512, 2200, 0.5),     # four rows a workgroup, held at once, eight columns a lane
    (1000, 512, 4500, 0.5),     # runs of two rows, a column a lane
    (258, 1024, 9000, 0.5),     # two rows a workgroup, runs of one
    (4096, 192, 1200, 0.5),     # sixteen rows a workgroup, runs of eight
    (4096, 256, 1100, 0.5),     # the same, eight columns a lane
    (300, 512, 16384, 0.9),     # rows that are not held at once
])
def test_decode_dense_rows(B, d_model, d_dict, share):
    """Long rows in every workgroup, against a matrix product in fp64, with the
    bound of test_decode_layouts."""
    t = torch()
    g = np.random.default_rng(B + d_dict)
    z = np.where(g.random((B, d_dict)) < share, g.standard_normal((B, d_dict)), 0).astype(np.float32)
    idx = g.permutation(np.flatnonzero(z))
    wb = workloads.f32_to_bf16_bits(g.standard_normal((d_dict, d_model)).astype(np.float32))
    bias = g.standard_normal(d_model).astype(np.float32)
    note(f"decode dense B={B} d_model={d_model} d_dict={d_dict} K={idx.size}")
    out = pk.sae_decode(t.from_numpy(z.reshape(-1)[idx]).cuda(), t.from_numpy(idx).cuda(),
                        gpu_bf16(wb).view(d_dict, d_model), t.from_numpy(bias).cuda(), B).cpu().numpy()
    w, z = (wb.astype(np.uint32) << 16).view(np.float32).reshape(d_dict, d_model).astype(np.float64), z.astype(np.float64)
    terms = (z != 0).sum(axis=1)[:, None]
    assert np.all(np.abs(out - (z @ w + bias)) <= (terms + 2) * 2.0**-24 * (np.abs(z) @ np.abs(w) + np.abs(bias)))


def _decode_us(B, d_model, d_dict, k_row):
    """Best of three decodes of k_row latents in each row, listed in random
    order, by events."""
    t = torch()
    g = t.Generator(device="cuda").manual_seed(k_row)
    j = (t.randint(0, d_dict, (B, 1), generator=g, device="cuda") + t.arange(k_row, device="cuda") * 4097) % d_dict
    idx = (t.arange(B, device="cuda")[:, None] * d_dict + j).view(-1)
    idx = idx[t.randperm(idx.numel(), generator=g, device="cuda")].contiguous()
    vals = t.rand(idx.numel(), generator=g, device="cuda")
    w = t.randn((d_dict, d_model), generator=g, device="cuda").to(t.bfloat16)
    b = t.zeros(d_model, device="cuda")
    note(f"decode time B={B} d_model={d_model} d_dict={d_dict} k_row={k_row}")
    ev = [t.cuda.Event(enable_timing=True) for _ in range(2)]
    best = float("inf")
    for _ in range(4):
        ev[0].record()
        pk.sae_decode(vals, idx, w, b, B)
        ev[1].record()
        t.cuda.synchronize()
        best = min(best, ev[0].elapsed_time(ev[1]) * 1e3)
    return best


def test_decode_time_follows_the_list():
    """A dense list (a quarter of every row) costs in proportion to its
    length: every workgroup reads its own rows' share of it, not the list.
    Eight times the entries per row, of rows of eight columns, take about 36
    times as long (rows that no longer fit a workgroup together are taken in
    runs, each a pass over the share); with half the list read by every
    workgroup it was 121 times."""
    few, many = _decode_us(4096, 8, 16384, 512), _decode_us(4096, 8, 16384, 4096)
    assert many < 80 * few, (few, many)


def test_decode_time_of_a_few_rows():
    """Columns that a lane could read eight at a time are not left to one wave
    (2.9 times the time of 510 columns, which are read one at a time)."""
    wide, narrow = _decode_us(8, 512, 16384, 4096), _decode_us(8, 510, 16384, 4096)
    assert wide < 2 * narrow, (wide, narrow)
