"""Contractions planned once and run many times: handles, tunings, eviction, graphs, threads."""
import ctypes
import threading

import pytest
import torch

import paper_2007_08056_amd as P
from paper_2007_08056_amd import _lib as L
from paper_2007_08056_amd import symtensor as S

DEV = "cuda:0"
SUB = "abkl,klij->abij"


def _operands(G=3, b=5, dtype=torch.float64, device=DEV):
    g = torch.Generator().manual_seed(G * 100 + b)
    make = lambda signs: P.SymTensor(torch.randn(G, G, G, b, b + 1, b, b + 1, dtype=dtype, generator=g).to(device),
                                     signs, 1, (G,))
    return make("++--"), make("++--")


def test_null_handles_are_refused_without_a_device():
    out = ctypes.c_void_p(1)
    assert L.LIB.symtensor_prepare(None, b"ab,bc->ac", None, None, None, None, 0, ctypes.byref(out)) == -1
    assert L.LIB.symtensor_contract_prepared(None, None, None, None, None, 0, None) == -1
    assert L.LIB.symtensor_release(None) == L.SYMT_OK


def test_wrapped_results_carry_the_validated_fields():
    # einsum builds its output without a second validation: the fields must be what validation would make of them
    u = P.SymTensor(torch.zeros(2, 4, 4, 2, 2, 2, 2, dtype=torch.float64), "++--", 1, 4, None, (2, 4, 4, 4))
    v = P.SymTensor(torch.zeros(4, 4, 4, 2, 2, 2, 2, dtype=torch.float64), "++--", 2, (4,))
    call = S._Einsum(SUB, u, v, "f64")
    w = S._wrap(torch.empty(call.shape, dtype=torch.float64), *call.meta_w)
    ref = P.SymTensor(torch.empty(call.shape, dtype=torch.float64), *call.meta_w)
    assert [(f, getattr(w, f)) for f in ("signs", "charge", "group", "mode_charges", "sectors")] == \
        [(f, getattr(ref, f)) for f in ("signs", "charge", "group", "mode_charges", "sectors")]
    assert w.sectors == (2, 4, 4, 4) and w.key() == ref.key()


@pytest.mark.gpu
@pytest.mark.parametrize("steps", [False, True])
def test_prepared_runs_match_the_one_call_entry_point(steps):
    u, v = _operands()
    w = P.output_like(SUB, u, v)
    P.contract_into(SUB, u, v, w, steps=steps)
    one = torch.full_like(w.data, 7.0)
    ws = torch.empty(max(1, P.plan(SUB, u, v, w=w, steps=steps).workspace_bytes), dtype=torch.uint8, device=DEV)
    ctx, g = L.context(0), L.make_group((3,))
    du, dv, dw = u.desc(), v.desc(), w.desc(one)
    L.check(L.LIB.symtensor_contract(ctx, SUB.encode(), ctypes.byref(g), du.ref, dv.ref, dw.ref,
                                     S._code("f64", steps), ctypes.c_void_p(ws.data_ptr()), ws.numel(),
                                     ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)), ctx)
    assert torch.equal(w.data, one)


@pytest.mark.gpu
def test_prepared_checks_stay_and_name_their_error():
    u, v = _operands()
    w = P.output_like(SUB, u, v)
    with pytest.raises(L.SymtError, match="overlaps"):
        P.contract_into(SUB, u, v, P.SymTensor(u.data, w.signs, w.charge, w.group))
    with pytest.raises(ValueError, match="contiguous"):
        P.einsum(SUB, P.SymTensor(u.data.transpose(0, 1), u.signs, u.charge, u.group), v)
    with pytest.raises(ValueError):
        P.einsum(SUB, u, v, "f16")


@pytest.mark.gpu
def test_eviction_gives_tables_back_and_results_stay(monkeypatch):
    monkeypatch.setattr(S, "_MAX_PLANS", 3)
    want = {}
    for turn in range(2):
        for b in (1, 2, 3, 4, 5, 6):
            u, v = _operands(b=b)
            got = P.einsum(SUB, u, v).data
            assert torch.equal(want.setdefault(b, got), got)
            assert len(S._PLANS) <= 3 and len(S._EINSUMS) <= 3


@pytest.mark.gpu
def test_prepared_under_capture_streams_and_threads():
    u, v = _operands(b=7)
    w = P.output_like(SUB, u, v)
    ws = torch.empty(max(1, P.plan(SUB, u, v, w=w).workspace_bytes), dtype=torch.uint8, device=DEV)
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):                   # the first call of this contraction
        P.contract_into(SUB, u, v, w, "f64", ws)
    for k in (1.0, 2.0, -3.0):
        u.data.mul_(k)
        want = P.einsum(SUB, u, v).data
        w.data.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(w.data, want)
    got = [None] * 4

    def work(i):
        s = torch.cuda.Stream()
        s.wait_stream(torch.cuda.default_stream())
        with torch.cuda.stream(s):
            for _ in range(8):
                got[i] = P.einsum(SUB, u, v).data
        s.synchronize()

    threads = [threading.Thread(target=work, args=(i,)) for i in range(4)]
    [t.start() for t in threads]
    [t.join() for t in threads]
    assert all(torch.equal(g, want) for g in got)
