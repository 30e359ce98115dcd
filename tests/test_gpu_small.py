"""GPU parity of the one-workgroup selection without sampling (k_small):
vectors from one element to the largest it holds and one more (which takes the
chunked path), k from 1 to N and 4096, unaligned bases with elements before
and after the whole vectors, ties that overflow the collected elements (cut
by index), many distinct keys above the bound, special values, and rows."""

import dataclasses

import numpy as np
import pytest

import paper_2608_12573_amd as pk
import workloads
from oracle import keys as okeys, plan as oplan, profk as oprofk
from gpu_util import check_rows, compare, gpu_bf16, gpu_f32, note, oracle_plan_of

pytestmark = pytest.mark.gpu


def _values(kind, n, seed):
    g = np.random.default_rng(seed)
    if kind == "normal":
        return g.standard_normal(n, dtype=np.float32)
    if kind == "constant":
        return np.full(n, -1.5, dtype=np.float32)
    if kind == "relu":
        return np.maximum(g.standard_normal(n, dtype=np.float32), np.float32(0))
    if kind == "two":
        return np.where(g.random(n) < 0.3, np.float32(2), np.float32(-2)).astype(np.float32)
    if kind == "ramp":
        return np.arange(n, dtype=np.float32)
    if kind == "special":
        return workloads.special_f32(n, seed=seed)
    if kind == "plateau":
        x = g.random(n, dtype=np.float32)
        x[x > 0.5] = np.float32(0.75)
        x[g.integers(0, n, 50)] = 0.9
        return x
    raise ValueError(kind)


def _check(x, k, dtype="f32", offset=0):
    p = pk.plan(x.size, k, force_mode=pk.FORCE_DIRECT)
    q = oracle_plan_of(p, force_mode=oplan.FORCE_DIRECT)
    note(f"direct {dtype} N={x.size} k={k} offset={offset}")
    if dtype == "f32":
        b, t = okeys.f32_bits(x), gpu_f32(x, offset)
    else:
        b = workloads.f32_to_bf16_bits(x)
        t = gpu_bf16(b, offset)
    vals, idx, info = pk.topk(t, k, p=p)
    compare(vals, idx, info, oprofk.run(b, dtype, k, q, 0), dtype)


@pytest.mark.parametrize("N", [1, 3, 5, 17, 64, 1000, 4095, 4099, 8192, 20000, 65535, 65536, 65537])
@pytest.mark.parametrize("offset", [0, 1, 3])
def test_small_sizes(N, offset):
    for k in sorted({1, min(N, 7), min(N, 100), min(N, 4096)}):
        _check(_values("normal", N, N), k, offset=offset)


@pytest.mark.parametrize("N,offset", [(5, 1), (9, 7), (8191, 3), (70001, 5), (131072, 0), (131073, 1)])
def test_small_bf16(N, offset):
    for k in sorted({1, min(N, 500), min(N, 4096)}):
        _check(_values("normal", N, N), k, "bf16", offset)
        _check(_values("relu", N, N + 1), k, "bf16", offset)


@pytest.mark.parametrize("kind", ["constant", "relu", "two", "ramp", "special", "plateau"])
@pytest.mark.parametrize("N,k", [(700, 700), (9001, 4000), (40003, 60), (65536, 1200), (65536, 4096)])
def test_small_distributions(kind, N, k):
    _check(_values(kind, N, N + k), k, offset=2)
    if kind != "special":
        _check(_values(kind, N, N + k), k, "bf16", offset=2)


@pytest.mark.parametrize("dtype,B,D,k,stride", [("f32", 3, 5001, 800, 5003), ("bf16", 5, 9000, 4000, 9001),
                                                ("f32", 260, 4100, 600, 4100), ("bf16", 300, 700, 200, 705)])
def test_small_rows(dtype, B, D, k, stride):
    p = pk.plan_rows(D, k)
    assert p.mode == pk.MODE_DIRECT
    x = _values("relu", B * D, B).reshape(B, D)
    b = okeys.f32_bits(x).reshape(B, D) if dtype == "f32" else workloads.f32_to_bf16_bits(x)
    check_rows(b, dtype, k, p, oracle_plan_of(p, rows=True), 0, offset=1, stride=stride)
