"""Performance cases of the prover: what a program that proves fixed-point
networks has it do, each through the public binding (paper_2505_17623_amd.ra).

A case is one of
  prove   a dense network (prove_network / prove_network_fp2): every layer's
          exact product, witness and sum-checks.  field "fp": challenges in
          F_p; "fp2": in F_{p^2}; "fs": non-interactive, the challenges
          hashed on the device.  planned: the program proves one network
          over and over, so it knows each layer's range parameter t, keeps
          its output buffers and (fp) defers its outputs to one wait per
          proof; else t is derived from the data and every call waits.
  cnn     the convolutional network with its gather links proven.
  commit  Pedersen commitments to a layer's witness tables or to one weight
          matrix.
  bind    one multilinear binding of a matrix (ra_mle_bind).
Dimensions are the real ones; programs pad them with zeros to powers of two,
and so does prepare().  Every output is an integer or a field element and is
the same, bit for bit, in any correct implementation.
"""
from __future__ import annotations

import hashlib
import math

import numpy as np
import torch

from paper_2505_17623_amd import inputs, ra

DEV = "cuda"
TABLES = ("C", "R", "Rm", "Y", "Z", "bits")
SCALARS = ("c0", "a_star", "b_star", "r_claim", "rm_claim", "y_claim", "z_claim", "range_sum", "bits_claim", "r_at",
           "y_at")


def _prove(name, field, batch, widths, s, values="normal", relu_last=False, floor=False, planned=True):
    c = dict(op="prove", field=field, batch=batch, widths=widths, s=s, values=values, relu_last=relu_last,
             floor=floor, planned=planned)
    return dict(name=name, **c) if name else c


def listed():
    return [
        # the smallest call: one 64 x 64 layer, a matrix product with rounding, proven once (t from the data)
        _prove("fp-64", "fp", 64, "64-64", 8, "uniform10", True, planned=False),
        # an MNIST-sized network: three small layers, ragged widths, one wait per proof
        _prove("fp-mnist", "fp", 64, "784-256-128-10", 8),
        # a single inference: a batch of one through two ragged layers
        _prove("fp-batch1", "fp", 1, "3000-1000-100", 10, planned=False),
        # one square layer over the full int16 range (62 of 64 bit planes in use)
        _prove("fp-1024", "fp", 1024, "1024-1024", 12, "uniform15", True),
        # a transformer block's MLP at batch 512, the throughput workload
        _prove("fp-mlp4096", "fp", 512, "4096-4096-4096", 12),
        # the largest table: 2^23 outputs, t from the data, literal floor rounding
        _prove("fp-2048x4096", "fp", 2048, "2048-4096", 12, relu_last=True, floor=True, planned=False),
        # a small CNN (im2col layers) with the links between its layers proven
        dict(name="cnn-links", op="cnn", batch=32, side=32),
        # the same MLP with challenges in F_{p^2} (the soundness a deployment asks for)
        _prove("fp2-mlp4096", "fp2", 512, "4096-4096-4096", 12),
        # non-interactive proofs: the small network, proven once, and the large one, over and over
        _prove("fs-mnist", "fs", 64, "784-256-128-10", 8, planned=False),
        _prove("fs-mlp4096", "fs", 512, "4096-4096-4096", 12),
        # commitments to the five witness tables of one 512 x 4096 layer
        dict(name="commit-witness", op="commit", what="witness", rows=512, cols=4096, s=12),
        # one binding of a weight matrix's columns
        dict(name="bind-4096", op="bind", rows=4096, cols=4096, dtype="int16", bind_rows=False),
    ]


def _log(rng, lo, hi):
    return max(lo, min(hi, round(math.exp(rng.uniform(math.log(lo), math.log(hi))))))


def draw(rng):
    op = rng.choice(["fp", "fp", "fp", "fp2", "fs", "cnn", "commit", "bind"])
    if op == "cnn":
        return dict(op="cnn", batch=rng.choice([1, 2, 4, 8, 16, 32]), side=rng.choice([8, 16, 32]))
    if op == "commit":
        what = rng.choice(["witness", "weights"])
        rows, cols = _log(rng, 16, 512), _log(rng, 16, 4096)
        return dict(op="commit", what=what, rows=rows, cols=cols, s=rng.choice([8, 10, 12]))
    if op == "bind":
        rows = inputs.next_pow2(_log(rng, 16, 8192))
        cols = inputs.next_pow2(_log(rng, 16, min(8192, (1 << 24) // rows)))
        return dict(op="bind", rows=rows, cols=cols, dtype=rng.choice(["int16", "int32", "int64", "field"]),
                    bind_rows=rng.random() < 0.5)
    s = rng.choice([8, 10, 12])
    planned = rng.random() < 0.5
    floor = rng.random() < 0.25
    if op == "fp" and rng.random() < 0.25:  # uniform entries: one layer
        values = rng.choice(["uniform10", "uniform15"])
        return _prove("", "fp", _log(rng, 16, 2048), f"{_log(rng, 16, 2048)}-{_log(rng, 16, 2048)}",
                      12 if values == "uniform15" else 8, values, True, floor, planned)
    layers = rng.choice([1, 2, 3])
    batch = _log(rng, 1, 2048 if op == "fp" else 512)
    top = 4096 if batch <= 512 else 2048
    widths = [_log(rng, 10, top) for _ in range(layers + 1)]
    return _prove("", op, batch, "-".join(map(str, widths)), s, "normal", layers == 1 and rng.random() < 0.5,
                  floor, planned)


# --- inputs ------------------------------------------------------------------
def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed) & 0x7FFFFFFFFFFFFFFF)


def _matrix(g, rows, cols, values, f):
    """An int16 matrix padded with zeros to powers of two: N(0, 0.5^2) with f
    fractional bits, or uniform over 11 or 16 bits."""
    out = torch.zeros((inputs.next_pow2(rows), inputs.next_pow2(cols)), dtype=torch.int16, device=DEV)
    if values == "normal":
        x = torch.randn((rows, cols), generator=g, device=DEV) * (0.5 * (1 << f))
        out[:rows, :cols] = x.round().clamp(-32768, 32767).to(torch.int16)
    else:
        b = int(values[len("uniform"):])
        out[:rows, :cols] = torch.randint(-(1 << b), 1 << b, (rows, cols), generator=g, device=DEV,
                                          dtype=torch.int32).to(torch.int16)
    return out


def _seed64(seed):
    return (0x9E3779B97F4A7C15 * (2 * int(seed) + 1)) & 0xFFFFFFFFFFFFFFFF or 1


def _widths(case):
    return [int(w) for w in case["widths"].split("-")]


def _dense(case, seed):
    g = _gen(seed)
    w = _widths(case)
    X = _matrix(g, case["batch"], w[0], case["values"], case["s"])
    last = len(w) - 2
    layers = [inputs.Layer(_matrix(g, w[i], w[i + 1], case["values"], case["s"]), case["s"],
                           i < last or case["relu_last"]) for i in range(last + 1)]
    return inputs.Workload("dense", X, layers, [None] * len(layers), int(case["floor"]))


def _cnn(case, seed):
    batch, H = case["batch"], case["side"]
    wl = inputs.cfg4(batch=batch, H=H)  # the layer layout; the values below replace its own
    g = _gen(seed)
    img = (torch.rand((batch * H * H, 3), generator=g, device=DEV) * 1024).round().to(torch.int16)
    wl.X = ra.to_device(inputs.Im2col(batch, H, H, 3, 3, 3, 1, 1, 32)(img.cpu().numpy()), DEV)
    real = [(27, 32), (128, 32), (288, 64), (256, 64), ((H // 4) ** 2 * 64, 10)]
    for layer, (r, c) in zip(wl.layers, real):
        B = torch.zeros(layer.B.shape, dtype=torch.int16, device=DEV)
        small = _matrix(g, r, c, "normal", 10)
        B[:r, :c] = small[:r, :c]
        layer.B = B
    return wl


def _witness(C, s, relu, floor, t=None):
    """(R, Rm, Y, Z, bits, t) of the exact product C, as the layouts in include/ra.h state them."""
    off = 0 if floor else 1 << (s - 1)
    R, Rm = (C + off) >> s, (C + off) & ((1 << s) - 1)
    if t is None:
        t = 0
        while int(R.max()) >= 1 << (t + 1) or int(R.min()) < -(1 << (t + 1)):
            t += 1
    Y = R.abs()
    Z = R.clamp(min=0) if relu else R
    bits = Rm | ((R + (1 << (t + 1))) << s)
    if relu:
        bits = bits | (Y << (s + t + 2))
    i32 = torch.int32
    return R.to(i32), Rm.to(torch.int16), Y.to(i32), Z.to(i32), bits.reshape(-1), t


def prepare(case, seed):
    op = case["op"]
    if op == "bind":
        g = _gen(seed)
        shape = (case["rows"], case["cols"])
        if case["dtype"] == "int16":
            T = _matrix(g, *shape, "normal", 12)
        elif case["dtype"] == "int32":  # a previous layer's outputs
            T = (torch.randn(shape, generator=g, device=DEV) * (1 << 16)).to(torch.int32)
        elif case["dtype"] == "int64":  # an exact product
            T = (torch.randn(shape, generator=g, device=DEV) * (1 << 28)).to(torch.int64)
        else:
            T = torch.randint(0, ra.P61, shape, generator=g, device=DEV, dtype=torch.int64)
        n = (case["rows"] if case["bind_rows"] else case["cols"]).bit_length() - 1
        return dict(op=op, ctx=ra.Context(seed=_seed64(seed)), T=T, rows=case["bind_rows"],
                    point=inputs.xorshift64_stream(_seed64(seed), n), field=case["dtype"] == "field")
    if op == "commit":
        g = _gen(seed)
        n = case["rows"] * case["cols"]
        if case["what"] == "weights":
            tables = [(_matrix(g, 1, n, "normal", case["s"])[0, :n].contiguous(), None)]
        else:  # the tables of a product of N(0, 0.5^2) operands with inner dimension 4096
            C = (torch.randn(n, generator=g, device=DEV, dtype=torch.float64) * (16 << (2 * case["s"]))).to(torch.int64)
            R, Rm, Y, Z, bits, _ = _witness(C, case["s"], True, False)
            tables = [(R, None), (Rm, ra.RA_U16), (Y, None), (Z, None), (bits, ra.RA_U64)]
        ctx = ra.Context(seed=_seed64(seed))
        gens = ra.commit_generators(ctx, hashlib.sha256(b"generators of the perf cases").digest(), n)
        return dict(op=op, ctx=ctx, gens=gens, tables=tables)
    wl = _cnn(case, seed) if op == "cnn" else _dense(case, seed)
    field = "fp" if op == "cnn" else case["field"]
    st = dict(op=op, field=field, wl=wl, Bs=[L.B for L in wl.layers], pubs=None, ts=None, bufs=None)
    if field == "fs":
        domain = hashlib.sha256(b"transcript %d" % int(seed)).digest()
        st["pubs"] = [hashlib.sha256(domain + bytes([i])).digest() for i in range(len(wl.layers))]
        st["ctx"] = ra.Context(fs_domain=domain)
    else:
        st["ctx"] = ra.Context(seed=_seed64(seed))
    if op == "cnn" or case["planned"]:  # a first proof fixes each layer's t; later ones are given it
        first = _network(st)
        st["ts"] = [o["transcript"]["t"] for o in first]
        st["bufs"] = []
        if field == "fp":
            st["ctx"].set_deferred(True)
        _network(st)
        st["ctx"].sync()
    return st


def _network(st):
    wl = st["wl"]
    if st["field"] == "fp":
        return ra.prove_network(st["ctx"], wl, DEV, X=wl.X, Bs=st["Bs"], ts=st["ts"], bufs=st["bufs"],
                                links=st["op"] == "cnn")
    return ra.prove_network_fp2(st["ctx"], wl, DEV, X=wl.X, Bs=st["Bs"], ts=st["ts"], bufs=st["bufs"],
                                pubs=st["pubs"])


# --- one pass ----------------------------------------------------------------
def _words(tr, field):
    vals = tr["mm_evals"] + tr["rs_evals"] + tr["zc_evals"] + [tr[k] for k in SCALARS]
    tp = [tr["t"], tr["P"]]
    return np.array(vals + (tp if field == "fp" else [tuple(tp)]), dtype=np.int64)


def run(st):
    if st["op"] == "bind":
        return ra.ra_mle_bind(st["ctx"], st["T"], st["rows"], st["point"], st["field"])
    if st["op"] == "commit":
        if len(st["tables"]) == 1:
            pts = [ra.commit(st["ctx"], st["tables"][0][0], st["gens"], st["tables"][0][1])]
        else:
            pts = ra.commit_batch(st["ctx"], st["tables"], st["gens"])
        return [np.frombuffer(p, dtype=np.uint8) for p in pts]
    res = _network(st)
    if st["ctx"].deferred:
        st["ctx"].sync()  # the proof is written out
    out = []
    for r in res:
        d = {k: r[k] for k in TABLES}
        d["transcript"] = _words(r["transcript"], st["field"])
        if r.get("root"):
            d["root"] = np.frombuffer(r["root"], dtype=np.uint8)
        if "link" in r:
            lk = r["link"]
            d["A"] = r["A"]
            d["link"] = np.array(lk["evals"] + [lk["claim"], lk["z_at"], lk["w_at"]], dtype=np.int64)
        out.append(d)
    return out


# --- accounting --------------------------------------------------------------
def _shapes(case):
    """(n, m, k, bytes per entry of A, relu) per layer, padded."""
    p = inputs.next_pow2
    if case["op"] == "cnn":
        b, H = case["batch"], case["side"]
        return [(b * H * H, 32, 32, 2, True), (b * H * H // 4, 128, 32, 4, True), (b * H * H // 4, 512, 64, 4, True),
                (b * H * H // 16, 256, 64, 4, True), (b, p((H // 4) ** 2 * 64), 16, 4, True)]
    w = _widths(case)
    last = len(w) - 2
    return [(p(case["batch"]), p(w[i]), p(w[i + 1]), 2 if i == 0 else 4, i < last or case["relu_last"])
            for i in range(last + 1)]


FIELD_MUL = 8  # operations of a product in F_p: four 32 x 32 -> 64 bit multiply-adds


def work(case):
    """Bytes: operands read, tables written.  Operations: the products' 2 n m
    k, and the sum-checks' field products (two bindings, 5 per pair of the
    matrix instance, 6 and 7 per pair over x of the range and the ReLU
    instance; three times as many over F_{p^2}); a commitment's additions,
    one per 8-bit digit at 11 products of 64 multiply-adds."""
    if case["op"] == "bind":
        size = {"int16": 2, "int32": 4}.get(case["dtype"], 8)
        e = case["rows"] * case["cols"]
        return {"bytes": e * size + 8 * (case["cols"] if case["bind_rows"] else case["rows"]), "flops": e * FIELD_MUL}
    if case["op"] == "commit":
        n = case["rows"] * case["cols"]
        per = [2] if case["what"] == "weights" else [4, 2, 4, 4, 8]
        return {"bytes": n * (sum(per) + 64), "flops": n * sum(per) * 11 * 128}
    by = ops = 0
    mul = FIELD_MUL * (1 if case["op"] == "cnn" or case["field"] == "fp" else 3)
    shapes = _shapes(case)
    for li, (n, m, k, ab, relu) in enumerate(shapes):
        N = n * k
        by += n * m * ab + m * k * 2 + N * 30
        ops += 2 * N * m + mul * (n * m + m * k + 5 * m + N * (6 + 7 * relu))
        if case["op"] == "cnn" and li:
            nz = shapes[li - 1][0] * shapes[li - 1][2]
            by += n * m * 8 + nz * 4
            ops += mul * (n * m + 5 * nz)
    return {"bytes": by, "flops": ops}


def tolerance(case):
    return "exact"


def exact(case, seed):
    """The integer tables of a dense network's layers: products in float64,
    exact below 2^53.  Transcripts have no floating value."""
    if case["op"] != "prove":
        return None
    wl = _dense(case, seed)
    A, out = wl.X, []
    for layer in wl.layers:
        C = (A.to(torch.float64) @ layer.B.to(torch.float64)).to(torch.int64)
        R, Rm, Y, Z, bits, _ = _witness(C, layer.s, layer.relu, bool(wl.mode))
        out.append(dict(C=C, R=R, Rm=Rm, Y=Y, Z=Z, bits=bits, transcript=None, root=None))
        A = Z
    return out
