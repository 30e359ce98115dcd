"""GPU parity of the row kernel's workgroup sizes (256, 512 and 1024 threads)
where the choice between them changes: batches at and above the number of
compute units, rows around 32 and 128 KiB, k from 1025 to 4096 (which only
the larger workgroups collect), ragged widths shorter than one step of the
largest workgroup, unaligned rows, ties, relaxed recall, the lexicographic
rule, underflow in one row, and plans that select without sampling."""

import dataclasses

import numpy as np
import pytest

import paper_2608_12573_amd as pk
import workloads
from oracle import keys as okeys, plan as oplan, profk as oprofk
from gpu_util import check_rows, oracle_plan_of

pytestmark = pytest.mark.gpu


def _bits(dtype, B, D, seed):
    if dtype == "bf16":
        return workloads.relu_normal_bf16((B, D), seed=seed)
    return okeys.f32_bits(workloads.normal_f32(B * D, seed=seed)).reshape(B, D)


@pytest.mark.parametrize("dtype,B,D,k", [
    ("f32", 1, 8192, 20), ("f32", 256, 8191, 20), ("f32", 257, 8192, 20),      # 32 KiB, around the CU count
    ("bf16", 3, 16384, 20), ("bf16", 258, 65536, 32), ("f32", 260, 32768, 7),  # 128 KiB on 512 threads
    ("f32", 2, 50001, 1024), ("bf16", 259, 65537, 300),
])
def test_row_block_sizes(dtype, B, D, k):
    p = pk.plan_rows(D, k)
    check_rows(_bits(dtype, B, D, seed=B + D % 97), dtype, k, p, oracle_plan_of(p, rows=True), 1)


@pytest.mark.parametrize("dtype,B,D,k", [
    ("f32", 5, 20001, 1025), ("bf16", 3, 40000, 2049), ("f32", 2, 65536, 4096), ("bf16", 258, 16401, 2048),
    ("f32", 4, 9000, 1100),
])
def test_row_block_large_k(dtype, B, D, k):
    p = pk.plan_rows(D, k)
    check_rows(_bits(dtype, B, D, seed=k), dtype, k, p, oracle_plan_of(p, rows=True), 2, offset=1, stride=D + 5)


@pytest.mark.parametrize("k", [40, 2000])
def test_row_block_rules(k):
    """Relaxed recall and the lexicographic rule, on ordinary rows, a constant
    row, a row of two values and one whose sample sees only its spikes."""
    B, D = 6, 40001
    x = workloads.normal_f32(B * D, seed=9).reshape(B, D)
    x[1] = 2.5
    x[2] = np.where(np.arange(D) % 7 == 0, 1.0, -1.0)
    x[3, : D // 2] = 0.0
    b = okeys.f32_bits(x)
    for kw in (dict(recall=0.9), dict(lexicographic=1)):
        p = pk.plan_rows(D, k, **kw)
        opts = dataclasses.replace(oplan.ROW_OPTS, lexicographic=bool(kw.get("lexicographic", 0)))
        st = check_rows(b, "f32", k, p, oracle_plan_of(p, opts=opts), 3)
        assert oprofk.STATUS_FILTERED in st


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_row_block_fallback(dtype):
    """A plan whose buffer is too small for most rows: every row falls back
    on its own, on each workgroup size."""
    for B, D, k in ((3, 33000, 30), (300, 66000, 30), (3, 33000, 1500)):
        p = pk.plan_rows(D, k)
        p.M = p.k + 1
        q = oplan.Plan(N=p.N, k=p.k, eps=p.eps, recall=p.recall, k_req=p.k_req, S=p.S, t=p.t, M=p.M, mode=p.mode,
                       p_underflow=p.p_underflow, p_overflow=p.p_overflow, lexicographic=False)
        st = check_rows(_bits(dtype, B, D, seed=11), dtype, k, p, q, 4)
        assert oprofk.STATUS_OVERFLOW in st


def test_row_block_direct():
    """No sampling (8 k > D) with k above 1024: in a block for a batch."""
    p = pk.plan_rows(9001, 1500)
    assert p.mode == pk.MODE_DIRECT
    check_rows(_bits("f32", 7, 9001, seed=5), "f32", 1500, p, oracle_plan_of(p, rows=True), 0)


@pytest.mark.parametrize("dtype,D,k,offset,extra", [
    ("f32", 4096, 64, 0, 0), ("f32", 4095, 90, 1, 2), ("f32", 1501, 150, 0, 0), ("f32", 700, 1, 3, 1), ("f32", 2051, 30, 0, 5),
    ("bf16", 8192, 64, 0, 0), ("bf16", 8191, 60, 5, 3), ("bf16", 1500, 3, 1, 0),
])
def test_row_block_one_wave(dtype, D, k, offset, extra):
    """A wave per row (large batches of rows up to 16 KiB), full and ragged
    widths, unaligned rows, with rows of ties and of few distinct values,
    whose buckets are large or which overflow the buffer and fall back."""
    B = 1030
    b = _bits(dtype, B, D, seed=D + k)
    one, two = (okeys.f32_bits(np.array([1.5], np.float32))[0], okeys.f32_bits(np.array([2.0], np.float32))[0]) \
        if dtype == "f32" else workloads.f32_to_bf16_bits(np.array([1.5, 2.0], np.float32))
    b[3] = one
    b[5] = np.where(np.arange(D) % 3 == 0, two, one)
    b[7, : D - D // 8] = 0
    p = pk.plan_rows(D, k)
    assert p.mode == pk.MODE_FILTER and p.S <= 512 and p.M <= 1024
    st = check_rows(b, dtype, k, p, oracle_plan_of(p, rows=True), 1, offset=offset, stride=D + extra)
    assert st.count(oprofk.STATUS_FILTERED) >= B - 3 and oprofk.STATUS_OVERFLOW in st


@pytest.mark.parametrize("B", [512, 513])
def test_row_block_lexicographic_long_rows(B):
    """More than two long rows per compute unit go to the smaller workgroup."""
    D, k = 65543, 20
    p = pk.plan_rows(D, k, lexicographic=1)
    opts = dataclasses.replace(oplan.ROW_OPTS, lexicographic=True)
    st = check_rows(_bits("bf16", B, D, seed=B), "bf16", k, p, oracle_plan_of(p, opts=opts), 4, offset=1)
    assert st == [oprofk.STATUS_FILTERED] * B
