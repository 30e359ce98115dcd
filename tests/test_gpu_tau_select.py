"""GPU parity of the threshold select: tau, count and status of whole calls
against the oracle, bit-exact, on inputs that drive the select's cases: a
bin of rank t that is one key wide (ties), one that holds few keys, one that
holds more than a counted list and is split again (values packed in a few
adjacent bit patterns beside an outlier), keys over the whole range, t = 1
and t at the union's end; in the filter (small unions, and capped lists with
and without the cut check failing), in the select launch (large unions) and
in the row kernel."""

import dataclasses

import numpy as np
import pytest

import paper_2608_12573_amd as pk
import workloads
from oracle import keys as okeys, plan as oplan, profk as oprofk
from gpu_util import check_rows, compare, gpu_f32, note, oracle_plan_of, plan_from_lib, torch

pytestmark = pytest.mark.gpu


def _values(kind, n, seed):
    g = np.random.default_rng(seed)
    if kind == "normal":
        return g.standard_normal(n, dtype=np.float32)
    if kind == "zeros":        # nearly every sampled key is the same
        x = np.zeros(n, dtype=np.float32)
        x[g.choice(n, n // 50, replace=False)] = g.random(n // 50, dtype=np.float32)
        return x
    if kind == "packed":       # 4096 adjacent patterns, one huge value and one of each infinity
        u = (np.uint32(0x3F800000) + g.integers(0, 4096, n).astype(np.uint32)).view(np.float32).copy()
        u[g.integers(0, n, 3)] = [1e38, np.inf, -np.inf]
        return u
    if kind == "wide":         # every exponent and sign
        u = g.integers(0, 2**32, n, dtype=np.uint64).astype(np.uint32)
        return u.view(np.float32).copy()
    raise ValueError(kind)


def _check(x, k, seed, **kw):
    p = pk.plan(x.size, k, **kw)
    q = oracle_plan_of(p, **kw)
    note(f"vec N={x.size} k={k} S={p.S} t={p.t} M={p.M}")
    vals, idx, info = pk.topk(gpu_f32(x), k, seed=seed, p=p)
    compare(vals, idx, info, oprofk.run(okeys.f32_bits(x), "f32", k, q, seed), "f32")


@pytest.mark.parametrize("kind", ["normal", "zeros", "packed", "wide"])
@pytest.mark.parametrize("N,k", [(70001, 1), (2**18 + 3, 40), (2**20, 2000), (2**20, 9000), (2**18, 16384)])
def test_vector_tau(kind, N, k):
    """t from 3 to about 2000: unions in the filter's registers, capped lists,
    and unions that take the select launch."""
    _check(_values(kind, N, N % 1009 + k), k, 3)


@pytest.mark.parametrize("kind", ["normal", "zeros", "packed", "wide"])
@pytest.mark.parametrize("N,k,t", [(2**20, 1, 1), (2**20 + 5, 2, 4), (1374554, 3, 4), (300001, 2, 5), (300001, 4, 7),
                                   (65983, 2, 8)])
def test_vector_tau_few_ranks(kind, N, k, t):
    """Unions of 32 lists of t keys, which one wave selects from, with the
    candidate that has t keys found early, late or (ties) never."""
    p = pk.plan(N, k)
    assert (p.t, p.S) == (t, 32768)
    _check(_values(kind, N, k), k, 6)


@pytest.mark.parametrize("S,k", [(33, 1), (256, 3), (257, 8), (1025, 60), (2049, 200)])
def test_vector_tau_small_samples(S, k):
    """Partial sample blocks down to one key above a block's size."""
    _check(_values("normal", 50001, S), k, 1, S_min=S, S_max=S, force_mode=pk.FORCE_FILTER)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("D,k,S", [(3001, 1, 64), (3001, 64, 300), (9001, 200, 2048), (9001, 200, 2049), (20001, 900, 4000),
                                   (3001, 96, 366), (3001, 96, 378), (2001, 250, 257), (2001, 250, 500)])
def test_row_tau(dtype, D, k, S):
    """Samples in registers (up to 2048 draws on 256 threads), with t on both
    sides of 32, and in LDS."""
    x = np.concatenate([_values(kind, D, D + k) for kind in ("normal", "zeros", "packed")]).reshape(3, D)
    bits = okeys.f32_bits(x) if dtype == "f32" else workloads.f32_to_bf16_bits(
        np.where(np.isfinite(x), x, np.float32(0)))
    kw = dict(S_min=S, S_max=S, force_mode=pk.FORCE_FILTER)
    p = pk.plan_rows(D, k, **kw)
    q = oracle_plan_of(p, opts=dataclasses.replace(oplan.ROW_OPTS, S_min=S, S_max=S, force_mode=pk.FORCE_FILTER))
    check_rows(bits.reshape(3, D), dtype, k, p, q, 2)


def _capped_union(p):
    """Keys in the union of the plan's capped sample lists (blocks of 1024
    draws, each list at most 16 or 32 long, the draws of a block in the top t
    plus eight standard deviations), 0 when its lists are not capped."""
    if p.t <= 32 or p.S < 2 * 1024 or p.lexicographic:
        return 0
    mu = 1024 * p.t / p.S
    need = mu + 8 * mu**0.5 + 2
    cap = 16 if need <= 16 else 32 if need <= 32 else 0
    whole, last = divmod(p.S - 1, 1024)
    return whole * cap + min(cap, last + 1) if cap else 0


@pytest.mark.parametrize("dtype,B,D,k,kw", [
    ("f32", 1, 393216, 1000, {}), ("f32", 16, 370727, 1024, {}), ("f32", 3, 524288, 1500, {}),
    ("bf16", 4, 370727, 1024, {}), ("f32", 4, 393216, 1000, dict(recall=0.9)), ("f32", 2, 524288, 1100, {}),
])
def test_row_tau_small_capped_union(dtype, B, D, k, kw):
    """Capped lists whose union has at most 256 keys, which one wave could
    hold: default row plans on the vector path, all filtered."""
    p = pk.plan_rows(D, k, **kw)
    code = pk.F32 if dtype == "f32" else pk.BF16
    assert p.t > 32 and 0 < _capped_union(p) <= 256
    assert pk.rows_workspace_size(p, code, B) == B * pk.workspace_size(p, code, 1)
    x = _values("normal", B * D, B + k).reshape(B, D)
    bits = okeys.f32_bits(x) if dtype == "f32" else workloads.f32_to_bf16_bits(x).reshape(B, D)
    st = check_rows(bits, dtype, k, p, oracle_plan_of(p, rows=True), 5)
    assert st == [oprofk.STATUS_FILTERED] * B


@pytest.mark.parametrize("S,k,N,union", [(5000, 1000, 400000, 160), (5121, 1100, 400000, 161), (7169, 1250, 400000, 225),
                                         (8192, 1100, 300000, 256), (8193, 1100, 300000, 257),
                                         (16384, 740, 1000000, 256), (16385, 740, 1000000, 257)])
def test_vector_tau_small_capped_union(S, k, N, union):
    """Both sides of 256 keys, lists of 16 and 32 and a last list of one."""
    p = pk.plan(N, k, S_min=S, S_max=S, force_mode=pk.FORCE_FILTER)
    assert _capped_union(p) == union, (p.t, _capped_union(p))
    _check(_values("normal", N, S), k, 4, S_min=S, S_max=S, force_mode=pk.FORCE_FILTER)


def _tied_top(N, share, seed):
    """Uniform values, the largest `share` of them all 1."""
    x = np.random.default_rng(seed).random(N, dtype=np.float32) * np.float32(0.5)
    x[np.random.default_rng(seed + 1).random(N) < share] = 1.0
    return x


@pytest.mark.parametrize("N,k,S,share,M,union", [
    (2**20, 458, 32768, 0.05, None, 512),        # every list full of ties: cut keys and tau all 1, an overflow
    (2**20, 458, 32768, 0.05, 2**17, 512),       # ... in a buffer that holds them
    (2**20, 458, 32768, 0.016, 2**17, 512),      # some lists full, others not
    (2**22, 9000, 131072, 0.05, 2**18, 4096),    # the select launch, in registers
    (2**22, 9000, 400000, 0.05, 2**18, 12512),   # ... by digit passes
    (2**22, 9000, 400000, 0.0, 2**18, 12512),    # ... no ties, cut keys below tau
])
def test_vector_tau_equal_to_the_cut(N, k, S, share, M, union):
    """Capped lists whose dropped keys only equal tau."""
    p = pk.plan(N, k, S_min=S, S_max=S)
    assert _capped_union(p) == union
    if M:
        p.M = M
    x = _tied_top(N, share, N + k)
    note(f"vec N={N} k={k} S={p.S} t={p.t} M={p.M} share={share}")
    vals, idx, info = pk.topk(gpu_f32(x), k, seed=3, p=p)
    ref = oprofk.run(okeys.f32_bits(x), "f32", k, plan_from_lib(p), 3)
    assert (ref.tau_key == okeys.keys_of(np.array([0x3F800000], dtype=np.uint32), "f32")[0]) == (share > 0)
    assert (ref.status == oprofk.STATUS_FILTERED) == bool(M)
    compare(vals, idx, info, ref, "f32")


def test_time_of_tau_equal_to_the_cut():
    """Such a call selects from its lists: it takes a few us more than the
    call that is given tau (with another select over the whole sample in
    every filter workgroup it took about 75 us more)."""
    t = torch()
    N, k = 2**20, 458
    p = pk.plan(N, k)
    p.M = 2**17
    x = gpu_f32(_tied_top(N, 0.05, 5))
    ws = pk.workspace(p, pk.F32)
    tau = int(okeys.keys_of(np.array([0x3F800000], dtype=np.uint32), "f32")[0])
    note("time of topk and topk_tau on ties")
    ev = [t.cuda.Event(enable_timing=True) for _ in range(2)]

    def us(f):
        best = float("inf")
        for _ in range(6):
            ev[0].record()
            f()
            ev[1].record()
            t.cuda.synchronize()
            best = min(best, ev[0].elapsed_time(ev[1]) * 1e3)
        return best

    given, whole = us(lambda: pk.topk_tau(x, k, tau, p, ws=ws)), us(lambda: pk.topk(x, k, seed=3, p=p, ws=ws))
    print(given, whole)
    assert whole < given + 40, (given, whole)
