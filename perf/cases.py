"""What the speed of this library is measured on: the provers and verifiers a program calls, over the sizes it calls them with.

A case is one call of a public entry point on device-resident inputs.  Every result is a proof (or a verdict with its
claims), which is exact: the same bytes on every run and every implementation.
"""
import math

import numpy as np
import torch

import paper_2404_16109_amd as zk
from paper_2404_16109_amd import synth


# ---- the cases ---------------------------------------------------------------------------------------------------

def listed():
    return [
        # The smallest range check of the test workloads (bytes against 0..255): a proof whose time is launches and
        # round trips to the transcript.
        {"name": "lookup_u8_tiny", "kind": "lookup", "logD": 10, "logN": 8, "real": 1000, "table": "unsigned",
         "dist": "uniform", "how": "hints"},
        # 8-bit quantisation of a layer of 2^20 activations: few rows, every row hot.
        {"name": "lookup_i8_quant", "kind": "lookup", "logD": 20, "logN": 8, "real": 1 << 20, "table": "signed",
         "dist": "uniform", "how": "hints"},
        # The activation of a 7B feed-forward layer, 2048 tokens x 11008, in a pair table of 2^16 rows; the tail up to
        # the power of two repeats row 0.  The headline of the benchmark.
        {"name": "lookup_activation_7b", "kind": "lookup", "logD": 25, "logN": 16, "real": 2048 * 11008, "table": "pair",
         "dist": "normal", "how": "hints"},
        # A shorter prompt through the same table from a caller that keeps no row numbers: 333 tokens x 11008.
        {"name": "lookup_activation_no_hints", "kind": "lookup", "logD": 22, "logN": 16, "real": 333 * 11008,
         "table": "pair", "dist": "normal", "how": "none"},
        # The activation of a small model (2048 tokens x 3072) handed over as its two integer columns.
        {"name": "lookup_activation_ints", "kind": "lookup_ints", "logD": 23, "logN": 16, "real": 2048 * 3072,
         "table": "pair", "dist": "normal"},
        # The two 16-bit digits of the attention scores of 20 heads x 2048 x 2048 under one sumcheck: the low digit is
        # spread over its table, the high one sits in a few rows.
        {"name": "attention_digits_batch", "kind": "batch", "logD": 27, "logN": 16, "real": 20 * 2048 * 2048, "K": 2},
        # LayerNorm of 2048 rows (the remainder of the downscaling, then 1/sqrt) together with the activation that
        # follows in a small layer: three lookups of three shapes.
        {"name": "layernorm_multi", "kind": "multi", "K": 3, "logD0": 11, "logN0": 10, "real0": 2048, "logD1": 12,
         "logN1": 12, "real1": 2048, "logD2": 18, "logN2": 16, "real2": 200000},
        # Y = X W at the 13B layer's shape, from field vectors.
        {"name": "matmul_13b", "kind": "matmul", "D0": 2048, "D1": 5120, "D2": 5120},
        # The same proof from 16-bit matrices, at a ragged shape of a small model: 333 tokens, 3000 in, 777 out.
        {"name": "matmul_i16_ragged", "kind": "matmul_i16", "D0": 333, "D1": 3000, "D2": 777},
        # The sumcheck that closes an attention layer, from field vectors: 4 heads x 2048 rows of 2048 scores.
        {"name": "attention_link_4heads", "kind": "link", "log_rows": 13, "log_cols": 11, "real_rows": 4 * 2048, "K": 2},
        # The same from the integer tensors for the whole layer of 40 heads: the largest proof.
        {"name": "attention_link_ints_40heads", "kind": "link_ints", "log_rows": 17, "log_cols": 11,
         "real_rows": 40 * 2048, "K": 2},
        # The other side: a lookup proof verified against its witness tensors, 2048 x 1376 activations.
        {"name": "verify_lookup", "kind": "verify", "logD": 22, "logN": 16, "real": 2048 * 1376, "table": "pair",
         "dist": "normal"},
    ]


def _real(rng, logD):
    """How many of 2^logD entries are the tensor's own: anything above half, the power of two itself included."""
    D = 1 << logD
    return D if rng.random() < 0.25 else rng.randint(D // 2 + 1, D)


def _each(case, field):
    return [case["%s%d" % (field, i)] for i in range(case["K"])]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["lookup", "lookup", "lookup", "lookup_ints", "batch", "multi", "matmul", "matmul", "matmul_i16",
                       "link", "link_ints", "verify"])
    if kind in ("lookup", "lookup_ints", "verify"):
        logD = rng.randint(10, 25)
        logN = rng.randint(4, min(logD, 16))
        case = {"kind": kind, "logD": logD, "logN": logN, "real": _real(rng, logD), "table": rng.choice(["unsigned", "signed", "pair", "pair"]),
                "dist": rng.choice(["uniform", "normal"])}
        if kind == "lookup":
            case["how"] = rng.choice(["hints", "hints", "none", "checked", "rows"])
        return case
    if kind == "batch":
        logD = rng.randint(11, 25)
        return {"kind": kind, "logD": logD, "logN": rng.randint(6, min(logD, 16)), "real": _real(rng, logD),
                "K": rng.randint(2, 4)}
    if kind == "multi":
        case = {"kind": kind, "K": rng.randint(2, 4)}
        for i in range(case["K"]):
            logD = rng.randint(10, 23)
            case.update({"logD%d" % i: logD, "logN%d" % i: rng.randint(6, min(logD, 16)), "real%d" % i: _real(rng, logD)})
        return case
    if kind in ("matmul", "matmul_i16"):
        return {"kind": kind, "D0": _log_uniform(rng, 1, 4096), "D1": _log_uniform(rng, 64, 8192),
                "D2": _log_uniform(rng, 16, 8192)}
    log_cols = rng.randint(5, 11)
    log_rows = rng.randint(2, 13 if kind == "link" else 16)
    rows = 1 << log_rows
    return {"kind": kind, "log_rows": log_rows, "log_cols": log_cols,
            "real_rows": rows if rng.random() < 0.25 else rng.randint(rows // 2 + 1, rows), "K": rng.randint(1, 3)}


# ---- inputs ------------------------------------------------------------------------------------------------------

_CHUNK = 1 << 24


def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) & 0x7FFFFFFFFFFFFFFF)
    return g


def _seed_bytes(seed):
    return np.array([(int(seed) * 0x9E3779B97F4A7C15 + i) & 0xFFFFFFFFFFFFFFFF for i in range(4)], dtype="<u8").tobytes()


def _rows_looked_up(g, D, real, N, dist):
    """Table rows of a tensor of D entries as int32: `real` of them drawn, the rest row 0."""
    idx = torch.zeros(D, dtype=torch.int32, device="cuda")
    for s in range(0, real, _CHUNK):
        e = min(real, s + _CHUNK)
        if dist == "uniform":
            idx[s:e] = torch.randint(0, N, (e - s,), generator=g, device="cuda", dtype=torch.int32)
        else:
            x = torch.randn(e - s, generator=g, device="cuda")
            idx[s:e] = (x * (N / 16.0)).round_().clamp_(-(N // 2), N // 2 - 1).to(torch.int32) + N // 2
    return idx


def _embedded(values):
    v = zk.Vec(values.numel())
    assert zk.fr_from_i32(v, values.contiguous()) == 0
    return v


def _gathered(T, idx):
    S = zk.Vec(idx.numel())
    for s in range(0, idx.numel(), _CHUNK):
        S.data[:, s:s + _CHUNK] = T.data[:, :T.n].index_select(1, idx[s:s + _CHUNK].long())
    return S


def _table(g, N, kind, sb):
    """A table of N rows: the integers from 0 or from -N/2 by themselves, or paired with an output column under the
    combiner rho."""
    tx = torch.arange(N, dtype=torch.int32, device="cuda") - (0 if kind == "unsigned" else N // 2)
    T = _embedded(tx)
    if kind != "pair":
        return {"T": T, "tx": tx, "ty": None, "rho": None}
    ty = torch.randint(-(1 << 15), 1 << 15, (N,), generator=g, device="cuda", dtype=torch.int32)
    rho = synth.pair_combiner(sb)
    assert zk.fr_axpy(T, T, rho, _embedded(ty)) == 0
    return {"T": T, "tx": tx, "ty": ty, "rho": rho}


def _workspace(nbytes):
    return torch.empty(max(int(nbytes), 256), dtype=torch.uint8, device="cuda")


def _digits(g, real, D, sigma=65536.0, cols=2048):
    """Attention scores below their row's maximum, negated, as two 16-bit digits; padded with the digit 0."""
    lo = torch.zeros(D, dtype=torch.int32, device="cuda")
    hi = torch.zeros(D, dtype=torch.int32, device="cuda")
    step = _CHUNK // cols * cols
    for s in range(0, real, step):
        e = min(real, s + step)
        n = (e - s + cols - 1) // cols * cols
        z = (torch.randn(n, generator=g, device="cuda", dtype=torch.float32) * sigma).round_().to(torch.int32).reshape(-1, cols)
        z = (z.max(dim=1, keepdim=True).values - z).reshape(-1)[:e - s]
        lo[s:e] = z & 0xFFFF
        hi[s:e] = z >> 16
    return lo, hi


def _link_tensors(case, g):
    """The integer tensors of an attention layer's closing sumcheck: K digits of the shifted scores, their table
    outputs, the product of these and its row sums."""
    K, rows, cols = case["K"], 1 << case["log_rows"], 1 << case["log_cols"]
    D, real = rows * cols, case["real_rows"] * cols
    lo, hi = _digits(g, real, D, cols=cols)
    if K == 1:
        X, bases = [lo], [1]
        del hi
    elif K == 2:
        X, bases = [lo, hi], [1, 1 << 16]
    else:
        X, bases = [lo & 0xFF, lo >> 8, hi], [1, 1 << 8, 1 << 16]
    out_hi = 1 << 16 if K < 3 else 1 << 12
    Yk, Zp, Y = [], torch.zeros(D, dtype=torch.int64, device="cuda"), None
    for k in range(K):
        ty = torch.randint(0, out_hi, (1 << 16,), generator=g, device="cuda", dtype=torch.int32)
        yk = torch.empty(D, dtype=torch.int32, device="cuda")
        for s in range(0, D, _CHUNK):
            part = slice(s, min(D, s + _CHUNK))
            yk[part] = ty[X[k][part].long()]
            Zp[part] -= bases[k] * X[k][part].long()
        Yk.append(yk)
        if Y is None:
            Y = yk.long()
        else:
            Y *= yk
    sums = Y.reshape(rows, cols).sum(dim=1)
    canon = torch.zeros((rows, 4), dtype=torch.int64, device="cuda")
    canon[:, 0] = sums
    yhat = zk.Vec(rows)
    assert zk.fr_from_canonical(yhat, canon) == 0
    return {"rows": rows, "cols": cols, "X": X, "Yk": Yk, "Y": Y, "Zp": Zp, "yhat": yhat, "bases": bases}


def prepare(case, seed):
    g, sb, kind = _generator(seed), _seed_bytes(seed), case["kind"]
    st = {"case": case, "seed": sb}
    if kind in ("lookup", "lookup_ints", "verify"):
        D, N = 1 << case["logD"], 1 << case["logN"]
        st.update(_table(g, N, case["table"], sb))
        st["idx"] = _rows_looked_up(g, D, case["real"], N, case["dist"])
        if kind == "lookup_ints":
            rows = st["idx"].long()
            st["X"] = st["tx"][rows].contiguous()
            st["Y"] = st["ty"][rows].contiguous() if st["ty"] is not None else None
            st["ws"] = _workspace(zk.tlookup_small_workspace_bytes(D, N))
            return st
        st["S"] = _gathered(st["T"], st["idx"])
        st["ws"] = _workspace(zk.tlookup_workspace_bytes(D, N))
        if kind == "verify":
            rc, proof, info = zk.tlookup_prove(sb, st["S"], st["idx"], st["T"], ws=st["ws"])
            assert rc == 0, rc
            st["proof"] = proof
            rc, st["m"], _ = zk.tlookup_multiplicities(st["S"], st["idx"], st["T"], ws=st["ws"])
            assert rc == 0, rc
            for name, src in (("A", st["S"]), ("B", st["T"])):
                shifted, st[name] = zk.Vec(src.n), zk.Vec(src.n)
                assert zk.fr_add_scalar(shifted, src, info["beta"]) == 0
                assert zk.fr_batch_inverse(st[name], shifted) == 0
            st["ws"] = _workspace(zk.raw().tlookup_verify_workspace_bytes(D, N))
        return st
    if kind == "batch":
        D, N, K = 1 << case["logD"], 1 << case["logN"], case["K"]
        tables = [_table(g, N, "pair", sb) for _ in range(K)]
        lo, hi = _digits(g, case["real"], D)
        rows = [lo, hi] + [lo >> 8, lo & 0xFF][:max(0, K - 2)]
        st["idx"] = [(r & (N - 1)).contiguous() for r in rows]
        st["T"] = [t["T"] for t in tables]
        st["S"] = [_gathered(t, i) for t, i in zip(st["T"], st["idx"])]
        st["ws"] = _workspace(zk.tlookup_batch_workspace_bytes(D, N, K))
        return st
    if kind == "multi":
        Ds, Ns = [1 << d for d in _each(case, "logD")], [1 << n for n in _each(case, "logN")]
        st["T"] = [_table(g, N, "pair" if i % 2 else "signed", sb)["T"] for i, N in enumerate(Ns)]
        st["idx"] = [_rows_looked_up(g, D, real, N, "normal") for D, N, real in zip(Ds, Ns, _each(case, "real"))]
        st["S"] = [_gathered(t, i) for t, i in zip(st["T"], st["idx"])]
        st["ws"] = _workspace(zk.tlookup_multi_workspace_bytes(Ds, Ns))
        return st
    if kind in ("matmul", "matmul_i16"):
        D0, D1, D2 = case["D0"], case["D1"], case["D2"]
        st["X"] = (torch.randn(D0, D1, generator=g, device="cuda") * 256.0).round_().to(torch.int16)
        st["W"] = (torch.randn(D1, D2, generator=g, device="cuda") * 64.0).round_().to(torch.int16)
        if kind == "matmul":
            st["X"] = _embedded(st["X"].reshape(-1).to(torch.int32))
            st["W"] = _embedded(st["W"].reshape(-1).to(torch.int32))
        st["ws"] = _workspace(zk.matmul_workspace_bytes(D0, D1, D2))
        return st
    st.update(_link_tensors(case, g))
    if kind == "link":
        mul = zk.Vec(st["Y"].numel())                       # Y = prod_k Y^(k), Z' = -sum_k B^(k) X^(k) as field vectors
        st["X"] = [_embedded(x) for x in st["X"]]
        st["Yk"] = [_embedded(y) for y in st["Yk"]]
        st["Zp"], st["Y"] = zk.Vec(mul.n), zk.Vec(mul.n)
        assert zk.fr_mul_scalar(st["Zp"], st["X"][0], synth.BLS12_381_R - st["bases"][0]) == 0
        assert zk.fr_mul_scalar(st["Y"], st["Yk"][0], 1) == 0
        for k in range(1, case["K"]):
            assert zk.fr_axpy(st["Zp"], st["Zp"], synth.BLS12_381_R - st["bases"][k], st["X"][k]) == 0
            assert zk.fr_mul(mul, st["Y"], st["Yk"][k]) == 0
            st["Y"], mul = mul, st["Y"]
    st["ws"] = _workspace(zk.zkattn_link_workspace_bytes(st["rows"], st["cols"], case["K"]))
    return st


# ---- one pass ----------------------------------------------------------------------------------------------------

def _bytes(b):
    return np.frombuffer(b, dtype=np.uint8)


def _proof(rc, proof):
    assert rc == 0, rc
    return {"rc": rc, "proof": _bytes(proof)}


def run(st):
    case, kind, seed = st["case"], st["case"]["kind"], st["seed"]
    if kind == "lookup":
        how = case["how"]
        call = {"checked": zk.tlookup_prove_checked, "rows": zk.tlookup_prove_by_rows}.get(how, zk.tlookup_prove)
        rc, proof, info = call(seed, st["S"], None if how == "none" else st["idx"], st["T"], ws=st["ws"])
        out = _proof(rc, proof)
        out["sums"] = _bytes(b"".join(info[k].to_bytes(32, "little") for k in ("sum_A", "sum_mB")))
        return out
    if kind == "lookup_ints":
        rc, proof, info = zk.tlookup_prove_small(seed, st["X"], st["Y"], st["rho"], st["idx"], st["T"], ws=st["ws"])
        out = _proof(rc, proof)
        out["sums"] = _bytes(b"".join(info[k].to_bytes(32, "little") for k in ("sum_A", "sum_mB")))
        return out
    if kind == "batch":
        return _proof(*zk.tlookup_prove_batch(seed, st["S"], st["idx"], st["T"], ws=st["ws"])[:2])
    if kind == "multi":
        return _proof(*zk.tlookup_prove_multi(seed, st["S"], st["idx"], st["T"], ws=st["ws"])[:2])
    if kind == "matmul":
        return _proof(*zk.matmul_sumcheck_prove(seed, st["X"], case["D0"], case["D1"], st["W"], case["D2"], ws=st["ws"]))
    if kind == "matmul_i16":
        return _proof(*zk.matmul_sumcheck_prove_i16(seed, st["X"], st["W"], ws=st["ws"]))
    if kind == "link":
        return _proof(*zk.zkattn_link_prove(seed, st["Zp"], st["X"], st["Y"], st["Yk"], st["yhat"], st["bases"], st["rows"],
                                            st["cols"], ws=st["ws"]))
    if kind == "link_ints":
        return _proof(*zk.zkattn_link_prove_small(seed, st["Zp"], st["X"], st["Y"], st["Yk"], st["yhat"], st["bases"],
                                                  st["rows"], st["cols"], ws=st["ws"]))
    rc, claims = zk.tlookup_verify(seed, st["proof"], st["T"], 1 << case["logD"], S=st["S"], A=st["A"], B=st["B"], m=st["m"],
                                   ws=st["ws"])
    assert rc == 0, rc
    values = [claims[k] for k in ("A_v", "S_v", "B_vp", "m_vp", "T_vp")] + claims["v"]
    return {"rc": rc, "claims": _bytes(b"".join(v.to_bytes(32, "little") for v in values))}


# ---- what a pass cannot do without -------------------------------------------------------------------------------

_MUL = 2 * 64               # a product of two 256-bit integers: 64 multiply-adds of 32-bit words


def work(case):
    """Inputs read once (the outputs are a few kilobytes).  A sumcheck over D entries binds them one variable at a time:
    one product for a round's sum and one to fold per pair, D multiplications in all per array that is folded."""
    kind = case["kind"]
    if kind == "lookup":
        D, N = 1 << case["logD"], 1 << case["logN"]
        return {"bytes": (32 if case["how"] == "none" else 36) * D + 32 * N, "flops": 3 * D * _MUL}
    if kind == "lookup_ints":
        D, N = 1 << case["logD"], 1 << case["logN"]
        return {"bytes": (12 if case["table"] == "pair" else 8) * D + 32 * N, "flops": 3 * D * _MUL}
    if kind == "batch":
        D, N, K = 1 << case["logD"], 1 << case["logN"], case["K"]
        return {"bytes": K * (36 * D + 32 * N), "flops": K * 3 * D * _MUL}
    if kind == "multi":
        D, N = sum(1 << d for d in _each(case, "logD")), sum(1 << n for n in _each(case, "logN"))
        return {"bytes": 36 * D + 32 * N, "flops": 3 * D * _MUL}
    if kind in ("matmul", "matmul_i16"):
        entries = case["D0"] * case["D1"] + case["D1"] * case["D2"]
        wide = kind == "matmul"                             # a 16-bit entry times a 256-bit weight: 8 multiply-adds
        return {"bytes": (32 if wide else 2) * entries, "flops": entries * (_MUL if wide else 16)}
    if kind in ("link", "link_ints"):
        D, K = 1 << (case["log_rows"] + case["log_cols"]), case["K"]
        per = 32 * (2 + 2 * K) if kind == "link" else 16 + 8 * K
        return {"bytes": per * D + (32 << case["log_rows"]), "flops": (2 + K) * D * _MUL}
    D, N = 1 << case["logD"], 1 << case["logN"]             # verify: S and A evaluated at a point
    return {"bytes": 64 * D + 68 * N, "flops": 2 * D * _MUL}


def tolerance(case):
    """Whole numbers: a proof has one right value for every byte."""
    return "exact"
