"""Contractions to time: one list of named cases, and a draw of more from the same ranges.

A case is a dict of plain values.  ``kind`` says what one pass is:

* ``contract``  one contraction of two symmetric tensors, through
  ``contract_into`` with the output and the workspace kept between calls
  (a solver's inner loop) or through ``einsum`` (``call``);
* ``chain``     the tensor-network environment update E' = E A W A, three
  contractions through ``einsum``;
* ``grad``      that chain, L = <E', R>, and its backward: the gradients with
  respect to E, A and W.

Shapes are those of this repository's workloads, of the paper's contractions
(Table 1, Table 2, the (s, t, v) sweep and the G sweeps) and of their
neighbours; values follow the workloads' laws (uniform in [-1, 1), or N(0, 1)
integrals and 1e-2 N(0, 1) amplitudes for the ladders).
"""
import itertools
import math

import numpy as np
import torch

import paper_2007_08056_amd as P

DEVICE = "cuda:0"
DTYPES = {"f64": torch.float64, "f32": torch.float32, "c128": torch.complex128, "c64": torch.complex64}

# einsum, signs of u and of v: every contracted pair carries opposite signs
FORMS = {
    "ladder": ("abcd,cdij->abij", "++--", "++--"),
    "mm": ("ij,jk->ik", "+-", "+-"),
    "cc1": ("ijkl,mnkl->ijmn", "++--", "--++"),
    "cc2": ("opij,opkm->ijmk", "++--", "--++"),
    "cc3": ("opmn,opij->ijmn", "++--", "--++"),
    "mps": ("ijk,klm->ijlm", "++-", "++-"),
    "peps": ("ijkl,klmn->ijmn", "++--", "++--"),
}
CHAIN = (("abc,asA->bcsA", "E", "A", "T1"), ("bcsA,bsSB->cASB", "T1", "W", "T2"), ("cASB,cSC->ABC", "T2", "A", "Ep"))
CHAIN_SIGNS = {"E": "---", "A": "++-", "W": "+---", "R": "---"}
STV = ((1, 1, 1), (2, 1, 1), (1, 2, 1), (1, 1, 2), (2, 2, 1), (2, 1, 2), (1, 2, 2), (2, 2, 2), (3, 1, 1), (1, 3, 1),
       (1, 1, 3))


def _stv_form(s, t, v):
    letters = "abcdefgh"
    i, k, j = letters[:s], letters[s:s + v], letters[s + v:s + v + t]
    return f"{i}{k},{k}{j}->{i}{j}", "+" * s + "-" * v, "+" * v + "-" * t


def _contract(form, group, dims, storage, compute, law="uniform", call="into", sectors="", shift=0):
    """``dims``: one block dimension per letter, in order of first appearance."""
    sub, su, sv = _stv_form(*map(int, form[3:])) if form.startswith("stv") else FORMS[form]
    return {"kind": "contract", "form": form, "sub": sub, "su": su, "sv": sv, "group": group,
            "dims": ",".join(map(str, dims)), "storage": storage, "compute": compute, "law": law, "call": call,
            "sectors": sectors, "shift": shift}


def _chain(kind, group, bond, mpo, phys, storage, compute):
    return {"kind": kind, "group": group, "bond": bond, "mpo": mpo, "phys": phys, "storage": storage,
            "compute": compute}


def listed():
    cases = [
        # The smallest call: the plain Z_4 contraction of the worked example, 2 MFLOP.  Host path and launches.
        dict(_contract("ladder", "4", (4,) * 6, "f64", "f64", call="einsum"), name="plain_z4_f64"),
        # A sweep's local update at an ordinary bond: three products of 0.3 to 1 GFLOP, in real arithmetic ...
        dict(_chain("chain", "2x3", 64, 4, 2, "f64", "f64"), name="mps_env_f64"),
        # ... and for complex states (time evolution).
        dict(_chain("chain", "2x3", 64, 4, 2, "c128", "f64"), name="mps_env_c128"),
        # Block-diagonal matrix product of the G sweep: blocks of 500, no multiple of a tile or of a K-step.
        dict(_contract("mm", "9", (500, 500, 500), "f64", "f64"), name="mm_z9_f64"),
        # Coupled-cluster contraction whose contracted modes lead in both operands (Table 2, CC2 at Z_16).
        dict(_contract("cc2", "16", (8, 8, 16, 16, 16, 8), "f32", "f32"), name="cc2_z16_f32"),
        # Unbalanced patterns of the (s, t, v) sweep at its odd block dimension: two large operands into a small
        # output (an energy or overlap) ...
        dict(_contract("stv113", "4", (57,) * 5, "f64", "f64"), name="stv113_f64"),
        # ... and a small matrix applied to one mode of a large tensor (a change of basis).
        dict(_contract("stv131", "4", (57,) * 5, "f32", "f32"), name="stv131_f32"),
        # The particle-particle ladder of CCD, Z_8, in split-bf16 (binary32 tensors).
        dict(_contract("ladder", "8", (24, 24, 24, 24, 6, 6), "f32", "bf16x3", "ladder"), name="ladder_z8_bf16x3"),
        # The same ladder with a and b in the Z_4 subgroup.
        dict(_contract("ladder", "8", (24, 24, 24, 24, 6, 6), "f64", "f64", "ladder", sectors="4,4,8,8,8,8"),
             name="ladder_z8_sub_f64"),
        # A variational step: the chain at bond 128, forward and backward.
        dict(_chain("grad", "2x3", 128, 4, 2, "f32", "f32"), name="mps_grad_f32"),
        dict(_chain("grad", "2x3", 128, 4, 2, "f64", "f64"), name="mps_grad_f64"),
        # The largest: the Z_16 ladder in binary64, 8.8 TFLOP.
        dict(_contract("ladder", "16", (32, 32, 32, 32, 8, 8), "f64", "f64", "ladder"), name="ladder_z16_f64"),
    ]
    return cases


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    while True:
        c = _draw(rng)
        w = work(c)
        if w["flops"] <= 1e12 and w["bytes"] <= 6e9:
            return c


def _draw(rng):
    real = rng.choice((("f64", "f64"), ("f64", "f64"), ("f32", "f32"), ("f32", "f32"), ("f32", "bf16x3")))
    any_ = rng.choice((real, real, real, ("c128", "f64"), ("c64", "f32")))
    what = rng.choice(("small", "mm", "cc", "cc", "peps", "stv", "stv", "ladder", "ladder", "chain", "chain", "grad",
                       "grad"))
    G = rng.choice((2, 3, 4, 5, 6, 7, 8, 9, 10, 12))
    group = rng.choice((str(G), str(G), "2x2", "2x3", "2x4"))
    size = math.prod(map(int, group.split("x")))
    shift = rng.choice((0, 0, 0, 1))          # U(1)-like charge tables: label l carries charge l + offset
    if what == "small":
        return _contract(rng.choice(("ladder", "cc1", "cc2", "peps")), group, [rng.randint(2, 8) for _ in range(6)],
                         *any_, call="einsum")
    if what == "mm":
        n = _log_int(rng, 60, 1200)
        return _contract("mm", group, [max(8, int(n * rng.uniform(0.6, 1.4))) for _ in range(3)], *any_, shift=shift)
    if what in ("cc", "peps"):
        n = _log_int(rng, 4, 20)
        dims = [max(2, int(n * rng.uniform(0.5, 1.5))) for _ in range(6)]
        form = "peps" if what == "peps" else rng.choice(("cc1", "cc2", "cc3"))
        if form == "peps":
            dims[:2] = [rng.randint(12, 48) for _ in range(2)]
            dims[2:] = [rng.randint(3, 10) for _ in range(4)]
        return _contract(form, group, dims, *any_, shift=shift)
    if what == "stv":
        s, t, v = rng.choice(STV)
        flops = math.exp(rng.uniform(math.log(1e8), math.log(8e10)))
        n = (flops / 2 / size ** (s + t + v - 2)) ** (1.0 / (s + t + v))
        dims = [max(2, int(round(n * rng.uniform(0.8, 1.2)))) for _ in range(s + t + v)]
        return _contract(f"stv{s}{t}{v}", group, dims, *real, shift=shift)
    if what == "ladder":
        nv, no = _log_int(rng, 8, 28), rng.randint(2, 8)
        sectors = ""
        if group == str(size) and size % 2 == 0 and rng.random() < 0.3:
            h = size // 2
            sectors, shift = f"{h},{h},{size},{size},{size},{size}", 0
        return _contract("ladder", group, (nv,) * 4 + (no,) * 2, *any_, law="ladder", sectors=sectors, shift=shift)
    group = rng.choice(("2", "3", "4", "2x2", "2x3"))
    return _chain(what, group, _log_int(rng, 16, 160), rng.randint(3, 6), rng.randint(2, 3),
                  *(any_ if what == "chain" else rng.choice((("f64", "f64"), ("f32", "f32")))))


# ---------------------------------------------------------------------------
def _orders(case):
    return tuple(int(x) for x in case["group"].split("x"))


def _terms(sub):
    tu, rest = sub.split(",")
    tv, tw = rest.split("->")
    return tu, tv, tw


def _letters(case):
    """letter -> (block dimension, sectors, charge offset) of a contraction."""
    tu, tv, _ = _terms(case["sub"])
    letters = list(dict.fromkeys(tu + tv))
    dims = [int(x) for x in case["dims"].split(",")]
    G = math.prod(_orders(case))
    hs = [int(x) for x in case["sectors"].split(",")] if case["sectors"] else [G] * len(letters)
    off = [(2 * i + 1) % G if case["shift"] else 0 for i in range(len(letters))]
    return {m: (d, h, o) for m, d, h, o in zip(letters, dims, hs, off)}


def _tables(group, modes, letters):
    G = math.prod(group)
    if not any(letters[m][2] for m in modes):
        return None
    return tuple(tuple((l + letters[m][2]) % G for l in range(G)) for m in modes)


def _shape(modes, letters):
    return [letters[m][1] for m in modes[:-1]] + [letters[m][0] for m in modes]


def _chain_letters(case):
    G = math.prod(_orders(case))
    d = {"a": case["bond"], "A": case["bond"], "c": case["bond"], "C": case["bond"], "b": case["mpo"],
         "B": case["mpo"], "s": case["phys"], "S": case["phys"]}
    return {m: (n, G, 0) for m, n in d.items()}


CHAIN_MODES = {"E": "abc", "A": "asA", "W": "bsSB", "R": "ABC"}


def _fill(shape, dtype, gen, law, scale=1.0):
    x = torch.empty(shape, dtype=dtype, device=DEVICE)
    parts = torch.view_as_real(x) if dtype.is_complex else x
    if law == "normal":
        parts.normal_(0.0, scale, generator=gen)
    else:
        parts.uniform_(-1.0, 1.0, generator=gen)
    return x


def _inputs(case, seed):
    """The case's input tensors, from the seed alone."""
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(1000003 * int(seed) + 17)
    dtype = DTYPES[case["storage"]]
    if case["kind"] == "contract":
        tu, tv, _ = _terms(case["sub"])
        letters = _letters(case)
        ladder = case["law"] == "ladder"
        u = _fill(_shape(tu, letters), dtype, gen, "normal" if ladder else "uniform")
        v = _fill(_shape(tv, letters), dtype, gen, "normal" if ladder else "uniform", 1e-2)
        return {"u": u, "v": v}
    letters = _chain_letters(case)
    out = {k: _fill(_shape(CHAIN_MODES[k], letters), dtype, gen, "uniform") for k in ("E", "A", "W")}
    if case["kind"] == "grad":
        out["R"] = _fill(_shape("ABC", letters), dtype, gen, "normal")
    return out


def prepare(case, seed):
    x = _inputs(case, seed)
    group = _orders(case)
    if case["kind"] == "contract":
        tu, tv, _ = _terms(case["sub"])
        letters = _letters(case)
        ops = [P.SymTensor(x[k], case["s" + k], 0, group, _tables(group, modes, letters),
                           tuple(letters[m][1] for m in modes)) for k, modes in (("u", tu), ("v", tv))]
        state = {"case": case, "u": ops[0], "v": ops[1]}
        if case["call"] == "into":
            w = P.output_like(case["sub"], *ops)
            need = P.plan(case["sub"], *ops, case["compute"], w).workspace_bytes
            state.update(w=w, ws=torch.empty(max(1, need), dtype=torch.uint8, device=DEVICE))
        return state
    if case["kind"] == "grad":
        for k in ("E", "A", "W"):
            x[k].requires_grad_(True)
    return {"case": case, **{k: P.SymTensor(t, CHAIN_SIGNS[k], 0, group) for k, t in x.items()}}


def run(state):
    case = state["case"]
    compute = case["compute"]
    if case["kind"] == "contract":
        if case["call"] == "into":
            return P.contract_into(case["sub"], state["u"], state["v"], state["w"], compute, state["ws"]).data
        return P.einsum(case["sub"], state["u"], state["v"], compute).data
    cur = {k: state[k] for k in ("E", "A", "W")}
    if case["kind"] == "grad":
        for t in cur.values():
            t.data.grad = None
    for sub, u, v, w in CHAIN:
        cur[w] = P.einsum(sub, cur[u], cur[v], compute)
    ep = cur["Ep"].data
    if case["kind"] == "chain":
        return ep
    torch.dot(ep.reshape(-1), state["R"].data.reshape(-1)).backward()
    return [ep.detach()] + [state[k].data.grad for k in ("E", "A", "W")]


# ---------------------------------------------------------------------------
# Work: every input read once, every output written once, allowed blocks only.
# ---------------------------------------------------------------------------
def _add(group, a, b, sign=1):
    r, mul = 0, 1
    for o in reversed(group):
        r += ((a % o + sign * (b % o)) % o) * mul
        a, b, mul = a // o, b // o, mul * o
    return r


def _charge(group, letters, mode, label):
    G = math.prod(group)
    _, h, off = letters[mode]
    return (label + off) % G if off else label * (G // h)


def _tuples(group, letters, modes, signs):
    """Sector tuples of some modes by their total charge."""
    by = {}
    for t in itertools.product(*[range(letters[m][1]) for m in modes]):
        q = 0
        for m, s, l in zip(modes, signs, t):
            q = _add(group, q, _charge(group, letters, m, l), 1 if s == "+" else -1)
        by.setdefault(q, []).append(t)
    return by


def _slices(case_group, letters, sub, su, sv):
    """(I, K, J) sector tuples of each nonzero slice of a contraction (total charges 0)."""
    tu, tv, _ = _terms(sub)
    k = [m for m in tu if m in tv]
    i = [m for m in tu if m not in k]
    j = [m for m in tv if m not in k]
    sgn_u, sgn_v = dict(zip(tu, su)), dict(zip(tv, sv))
    by_i = _tuples(case_group, letters, i, [sgn_u[m] for m in i])
    by_j = _tuples(case_group, letters, j, [sgn_v[m] for m in j])
    for q, ks in _tuples(case_group, letters, k, [sgn_u[m] for m in k]).items():
        qv = 0
        for m, l in zip(k, ks[0]):
            qv = _add(case_group, qv, _charge(case_group, letters, m, l), 1 if sgn_v[m] == "+" else -1)
        ni, nj = _add(case_group, 0, q, -1), _add(case_group, 0, qv, -1)
        if ni in by_i and nj in by_j:
            yield (i, by_i[ni]), (k, ks), (j, by_j[nj])


def _elems(modes, letters):
    return math.prod(_shape(modes, letters))


def _one(group, letters, sub, su, sv):
    """(bytes of one element times elements of u, v, w; real multiply-add flops) of a contraction."""
    tu, tv, tw = _terms(sub)
    blk = math.prod(letters[m][0] for m in set(tu + tv))
    G = math.prod(group)
    if all(letters[m][1] == G for m in set(tu + tv)):
        flops = 2.0 * blk * float(G) ** (len(set(tu + tv)) - 2)
    else:
        flops = 2.0 * blk * sum(len(a[1]) * len(b[1]) * len(c[1]) for a, b, c in _slices(group, letters, sub, su, sv))
    return (_elems(tu, letters), _elems(tv, letters), _elems(tw, letters)), flops


def work(case):
    group = _orders(case)
    dtype = DTYPES[case["storage"]]
    size = torch.empty((), dtype=dtype).element_size()
    mul = 4.0 if dtype.is_complex else 1.0
    if case["kind"] == "contract":
        n, flops = _one(group, _letters(case), case["sub"], case["su"], case["sv"])
        return {"bytes": float(size * sum(n)), "flops": mul * flops}
    letters = _chain_letters(case)
    io = [_elems(CHAIN_MODES[k], letters) for k in ("E", "A", "W")]
    flops = sum(_one(group, letters, sub, "", "")[1] for sub, *_ in CHAIN)
    if case["kind"] == "chain":
        return {"bytes": float(size * (sum(io) + io[0])), "flops": mul * flops}
    # forward and, for each contraction, two of the same size backward; R and E' beside the gradients
    return {"bytes": float(size * (2 * sum(io) + 2 * io[0])), "flops": 3.0 * flops}


# ---------------------------------------------------------------------------
# The same results in 64 bits from plain torch.
# ---------------------------------------------------------------------------
def _plain(group, letters, sub, su, sv, u, v):
    tu, tv, tw = _terms(sub)

    def stored(modes, *parts):
        """Index of the stored block of every combination of the parts' sector tuples."""
        idx = np.zeros([len(t) for _, t in parts], dtype=np.int64)
        for m in modes[:-1]:
            for axis, (names, tuples) in enumerate(parts):
                if m in names:
                    col = np.array([t[names.index(m)] for t in tuples], dtype=np.int64)
                    shape = [1] * len(parts)
                    shape[axis] = -1
                    idx = idx * letters[m][1] + col.reshape(shape)
        return torch.from_numpy(idx).to(u.device)

    def dims(modes):
        return [letters[m][0] for m in modes]
    ub, vb = u.reshape([-1] + dims(tu)), v.reshape([-1] + dims(tv))
    wb = torch.zeros([math.prod(_shape(tw, letters)[:len(tw) - 1])] + dims(tw), dtype=u.dtype, device=u.device)
    for I, K, J in _slices(group, letters, sub, su, sv):
        (i, it), (k, kt), (j, jt) = I, K, J
        a = ub[stored(tu, I, K)].permute([0] + [2 + tu.index(m) for m in i] + [1] + [2 + tu.index(m) for m in k])
        b = vb[stored(tv, K, J)].permute([0] + [2 + tv.index(m) for m in k] + [1] + [2 + tv.index(m) for m in j])
        nk = len(kt) * math.prod(dims(k))
        c = torch.matmul(a.reshape(-1, nk), b.reshape(nk, -1))
        c = c.reshape([len(it)] + dims(i) + [len(jt)] + dims(j))
        at = {m: 1 + x for x, m in enumerate(i)}
        at.update({m: 2 + len(i) + x for x, m in enumerate(j)})
        c = c.permute([0, 1 + len(i)] + [at[m] for m in tw]).reshape([-1] + dims(tw))
        wb[stored(tw, I, J).reshape(-1)] = c
    return wb.reshape(_shape(tw, letters))


def exact(case, seed):
    group = _orders(case)
    x = {k: t.to(torch.complex128 if t.is_complex() else torch.float64) for k, t in _inputs(case, seed).items()}
    if case["kind"] == "contract":
        return _plain(group, _letters(case), case["sub"], case["su"], case["sv"], x["u"], x["v"])
    grad = case["kind"] == "grad"
    letters = _chain_letters(case)
    signs = dict(CHAIN_SIGNS, T1="--+-", T2="----")
    if grad:
        for k in ("E", "A", "W"):
            x[k].requires_grad_(True)
    for sub, u, v, w in CHAIN:
        x[w] = _plain(group, letters, sub, signs[u], signs[v], x[u], x[v])
    if not grad:
        return x["Ep"]
    torch.sum(x["Ep"] * x["R"]).backward()
    return [x["Ep"].detach()] + [x[k].grad for k in ("E", "A", "W")]
