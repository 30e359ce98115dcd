"""GPU parity of profk_topk_rows on the batched vector path: every launch
takes as many rows as the workspace holds (all of them, some, or one), on
contiguous, odd-stride and unaligned rows, with ties, the lexicographic rule
(whose threshold takes launches of its own), relaxed recall, unions that need
the select launch, rows that fall back beside rows that do not, and rows
selected without sampling.  Every workspace size gives the same result."""

import dataclasses

import numpy as np
import pytest

import paper_2608_12573_amd as pk
import workloads
from oracle import keys as okeys, plan as oplan, profk as oprofk
from gpu_util import check_rows, gpu_f32, host_bits, note, oracle_plan_of, torch

pytestmark = pytest.mark.gpu


def _bits(dtype, B, D, seed):
    if dtype == "bf16":
        return workloads.relu_normal_bf16((B, D), seed=seed)
    return okeys.f32_bits(workloads.normal_f32(B * D, seed=seed)).reshape(B, D)


def _batched(p, dtype, B):
    code = pk.F32 if dtype == "f32" else pk.BF16
    return pk.rows_workspace_size(p, code, B) == min(B, 64) * pk.workspace_size(p, code, 1)


@pytest.mark.parametrize("dtype,B,D,k,offset,extra", [
    ("f32", 3, 2**20 + 3, 16, 1, 5), ("bf16", 5, 2**21 + 1, 40, 3, 2), ("f32", 2, 2**20, 4000, 0, 0),
    ("bf16", 67, 2**19 + 7, 1, 0, 1),
])
def test_batched_rows(dtype, B, D, k, offset, extra):
    p = pk.plan_rows(D, k)
    assert _batched(p, dtype, B)
    check_rows(_bits(dtype, B, D, seed=B + k), dtype, k, p, oracle_plan_of(p, rows=True), 3, offset=offset,
               stride=D + extra)


@pytest.mark.parametrize("kw", [dict(recall=0.9), dict(lexicographic=1), dict(S_min=60000, S_max=60000)])
def test_batched_rows_rules(kw):
    """(60000 draws of k = 2000: t in the hundreds, unions above 2048 keys)"""
    B, D, k = 4, 2**20 + 9, 2000
    x = workloads.normal_f32(B * D, seed=9).reshape(B, D)
    x[1] = 2.5
    x[2] = np.where(np.arange(D) % 7 == 0, 1.0, -1.0)
    p = pk.plan_rows(D, k, **kw)
    assert _batched(p, "f32", B)
    opt = {a: b for a, b in kw.items() if a != "recall"}
    if "lexicographic" in opt:
        opt["lexicographic"] = True
    st = check_rows(okeys.f32_bits(x), "f32", k, p, oracle_plan_of(p, opts=dataclasses.replace(oplan.ROW_OPTS, **opt)), 1)
    assert oprofk.STATUS_FILTERED in st
    if kw.get("lexicographic"):
        assert st == [oprofk.STATUS_FILTERED] * B
    elif kw.get("recall") is None:
        assert oprofk.STATUS_OVERFLOW in st


def test_batched_rows_direct():
    """Rows selected without sampling that no row block holds."""
    p = pk.plan_rows(30001, 3900, force_mode=pk.FORCE_DIRECT)
    b = _bits("f32", 3, 30001, seed=4)
    check_rows(b, "f32", 3900, p, oracle_plan_of(p, opts=dataclasses.replace(oplan.ROW_OPTS, force_mode=oplan.FORCE_DIRECT)), 0)


@pytest.mark.parametrize("D,k", [(2**22, 32), (2**20, 64)])
def test_workspace_sizes_agree(D, k):
    """One, two and all rows at a time; the smaller plan also without a
    workspace (one workgroup per row) and with the least that is accepted."""
    t = torch()
    B = 5
    p = pk.plan_rows(D, k)
    x = gpu_f32(workloads.normal_f32(B * D, seed=12)).view(B, D)
    one, least = pk.workspace_size(p, pk.F32, 1), pk.workspace_size(p, pk.F32, B)
    ref = None
    for n in sorted({least, one, 2 * one + 17, B * one, 64 * one}):
        note(f"rows D={D} k={k} workspace {n}")
        ws = t.empty(n, dtype=t.uint8, device="cuda")
        vals, idx, info = pk.topk_rows(x, k, p=p, ws=ws, seed=2)
        got = (host_bits(vals), idx.cpu().numpy(), info.cpu().numpy())
        if ref is None:
            ref = got
        assert all(np.array_equal(a, b) for a, b in zip(ref, got)), n


@pytest.mark.parametrize("shift", [0, 1, 4, 8, 16])
def test_unaligned_workspace(shift):
    """A plan that needs no workspace accepts one at any address: the vector
    path takes it where it is 16-byte aligned, else it is left as it is."""
    t = torch()
    B, D, k = 4, 2**20, 64
    p = pk.plan_rows(D, k)
    assert _batched(p, "f32", B) and pk.workspace_size(p, pk.F32, B) == 256
    x = gpu_f32(workloads.normal_f32(B * D, seed=13)).view(B, D)
    n = pk.rows_workspace_size(p, pk.F32, B)
    buf = t.full((n + 64,), 0xA5, dtype=t.uint8, device="cuda")
    assert buf.data_ptr() % 256 == 0
    note(f"rows B={B} D={D} k={k} workspace at {shift}")
    got = [a.view(-1) for a in pk.topk_rows(x, k, p=p, ws=buf[shift:shift + n], seed=2)]
    ref = [a.view(-1) for a in pk.topk_rows(x, k, p=p, seed=2)]
    assert all(t.equal(a, b) for a, b in zip(got, ref))
    assert bool((buf == 0xA5).all()) == (shift % 16 != 0)
    assert bool((buf[:shift] == 0xA5).all()) and bool((buf[shift + n:] == 0xA5).all())
