"""Pedersen vector commitments on the GPU (ra_commit_generators, ra_commit)
against the oracle (oracle/ec_oracle.py), through the C ABI: the generators
limb for limb, commitments byte for byte for every value type and for sizes
from one value to full-layer tables (the latter on sparse vectors the oracle
computes, and by homomorphism on dense ones), and the tables of a proven
layer."""
import hashlib

import numpy as np
import pytest
import torch

from oracle import ec_oracle as ec
from paper_2505_17623_amd import inputs

pytestmark = pytest.mark.gpu
DOMAIN = hashlib.sha256(b"range-arithmetic commitment tests").digest()


@pytest.fixture(scope="module")
def ra():
    from paper_2505_17623_amd import ra as ra_mod
    ra_mod.lib()
    assert torch.cuda.is_available()
    return ra_mod


@pytest.fixture(scope="module")
def ctx(ra):
    return ra.Context(seed=1)


def test_generators_match_oracle(ra, ctx):
    g = ra.commit_generators(ctx, DOMAIN, 64).cpu().numpy().view(np.uint32)
    assert np.array_equal(g, ra.point_limbs(ec.generators(DOMAIN, 64)))
    first = (1 << 21) - 3
    g2 = ra.commit_generators(ctx, DOMAIN, 6, first=first).cpu().numpy().view(np.uint32)
    assert np.array_equal(g2, ra.point_limbs([ec.generator(DOMAIN, first + i) for i in range(6)]))


@pytest.fixture(scope="module")
def gens_small(ra, ctx):
    return ra.commit_generators(ctx, DOMAIN, 4096), ec.generators(DOMAIN, 4096)


DTYPES = [(np.int16, None), (np.uint16, "RA_U16"), (np.int32, None), (np.uint64, "RA_U64")]


@pytest.mark.parametrize("n", [1, 7, 256, 3001])
@pytest.mark.parametrize("dt,code", DTYPES)
def test_commit_matches_oracle(ra, ctx, gens_small, n, dt, code):
    dev_gens, gens = gens_small
    rng = np.random.default_rng(n + np.dtype(dt).itemsize)
    info = np.iinfo(dt)
    v = rng.integers(info.min, info.max, size=n, dtype=dt, endpoint=True)
    v[: min(n, 3)] = [info.min, info.max, 0][: min(n, 3)]
    if n > 16:
        v[rng.random(n) < 0.3] = 0
    t = torch.from_numpy(v.view(np.int16 if dt == np.uint16 else (np.int64 if dt == np.uint64 else dt))).cuda()
    got = ra.commit(ctx, t, dev_gens, getattr(ra, code) if code else None)
    want = ec.encode(ec.commit([int(x) for x in v], gens[:n]))
    assert got == want
    assert ra.commit_open(v, ra.point_limbs(gens[:n]), got)


def test_commit_zero_and_empty(ra, ctx, gens_small):
    dev_gens, _ = gens_small
    assert ra.commit(ctx, torch.zeros(100, dtype=torch.int32).cuda(), dev_gens) == bytes(64)
    e = torch.zeros(1, dtype=torch.int32).cuda()
    assert ra.commit(ctx, e[:0], dev_gens) == bytes(64)


def test_commit_full_layer(ra, ctx):
    """2^21 values (the tables of one 512 x 4096 output layer): sparse vectors
    against the oracle at their positions, and a + b = (a) + (b) on dense ones."""
    n = 1 << 21
    gens = ra.commit_generators(ctx, DOMAIN, n)
    rng = np.random.default_rng(21)
    pos = np.sort(rng.choice(n, size=40, replace=False))
    v = np.zeros(n, dtype=np.int32)
    v[pos] = rng.integers(-(2 ** 31), 2 ** 31, size=40)
    got = ra.commit(ctx, torch.from_numpy(v).cuda(), gens)
    want = ec.encode(ec.commit([int(v[i]) for i in pos], [ec.generator(DOMAIN, int(i)) for i in pos]))
    assert got == want
    a = rng.integers(-(2 ** 30), 2 ** 30, size=n).astype(np.int32)
    b = rng.integers(-(2 ** 30), 2 ** 30, size=n).astype(np.int32)
    ca = ec.decode(ra.commit(ctx, torch.from_numpy(a).cuda(), gens))
    cb = ec.decode(ra.commit(ctx, torch.from_numpy(b).cuda(), gens))
    cab = ec.decode(ra.commit(ctx, torch.from_numpy(a + b).cuda(), gens))
    assert ec.on_curve(ca) and ec.on_curve(cb)
    assert ec.add(ca, cb) == cab
    # a full-size u64 table of words (the bit table's layout)
    w = rng.integers(0, 2 ** 63, size=n, dtype=np.uint64)
    cw = ec.decode(ra.commit(ctx, torch.from_numpy(w.view(np.int64)).cuda(), gens, ra.RA_U64))
    w2 = w.copy()
    w2[pos[:3]] += np.uint64(1)
    cw2 = ec.decode(ra.commit(ctx, torch.from_numpy(w2.view(np.int64)).cuda(), gens, ra.RA_U64))
    assert ec.add(cw, ec.commit([1, 1, 1], [ec.generator(DOMAIN, int(i)) for i in pos[:3]])) == cw2


def test_commit_layer_tables(ra, ctx):
    """The witness tables of a proven layer, committed on the GPU, against
    the oracle and the host opening."""
    wl = inputs.small(1)
    got = ra.prove_network(ra.Context(wl.challenges), wl)[0]
    N = got["R"].numel()
    dev_gens = ra.commit_generators(ctx, DOMAIN, N)
    gens = ec.generators(DOMAIN, N)
    limbs = ra.point_limbs(gens)
    for name, code in (("R", None), ("Y", None), ("Z", None), ("Rm", "RA_U16"), ("bits", "RA_U64")):
        t = got[name].reshape(-1)
        P = ra.commit(ctx, t, dev_gens, getattr(ra, code) if code else None)
        host = t.cpu().numpy()
        host = host.view(np.uint16) if name == "Rm" else (host.view(np.uint64) if name == "bits" else host)
        assert P == ec.encode(ec.commit([int(x) for x in host], gens)), name
        assert ra.commit_open(host, limbs, P), name


def test_commit_heavy_buckets(ra, ctx):
    """Values whose digits fall in one or two buckets (every run of every
    sorted chunk holds the same digit, so a bucket's partials are summed by the
    segmented tree), against sums of the generators formed on the host."""
    n = 1 << 16
    dev_gens = ra.commit_generators(ctx, DOMAIN, n)
    limbs = dev_gens.cpu().numpy().view(np.uint32).reshape(n, 16).astype(object)
    w = [1 << (32 * k) for k in range(8)]
    pts = [(sum(l[k] * w[k] for k in range(8)), sum(l[8 + k] * w[k] for k in range(8))) for l in limbs]
    even = odd = None
    for i, p in enumerate(pts):
        if i & 1:
            odd = ec.add(odd, p)
        else:
            even = ec.add(even, p)
    total = ec.add(even, odd)
    ones = torch.ones(n, dtype=torch.int32, device="cuda")
    assert ec.decode(ra.commit(ctx, ones, dev_gens)) == total
    assert ec.decode(ra.commit(ctx, ones * 257, dev_gens)) == ec.mul(257, total)
    assert ec.decode(ra.commit(ctx, -ones, dev_gens)) == ec.neg(total)
    v = ones.clone()
    v[1::2] = 3 << 16
    assert ec.decode(ra.commit(ctx, v, dev_gens)) == ec.add(even, ec.mul(3 << 16, odd))
    u = torch.full((n,), 1 << 40, dtype=torch.int64, device="cuda")
    assert ec.decode(ra.commit(ctx, u, dev_gens, ra.RA_U64)) == ec.mul(1 << 40, total)


def test_commit_batch_matches_single_calls(ra, ctx, gens_small):
    """ra_commit_batch over tables of every value type and size (one value to
    3001, an all-zero table, an empty one) in one call: each table's point
    equals its own ra_commit and the oracle's sum.  Then the argument checks:
    no tables, more than 64, an unknown type."""
    dev_gens, gens = gens_small
    rng = np.random.default_rng(77)
    tables, want = [], []
    for i, (n, (dt, code)) in enumerate([(3001, DTYPES[2]), (1, DTYPES[0]), (256, DTYPES[3]), (7, DTYPES[1]),
                                         (3001, DTYPES[3]), (100, DTYPES[2]), (0, DTYPES[2]), (4096, DTYPES[0])]):
        info = np.iinfo(dt)
        v = rng.integers(info.min, info.max, size=n, dtype=dt, endpoint=True)
        if i == 5:
            v[:] = 0
        elif n >= 3:
            v[:3] = [info.min, info.max, 0]
        t = torch.from_numpy(v.view(np.int16 if dt == np.uint16 else (np.int64 if dt == np.uint64 else dt))).cuda()
        tables.append((t, getattr(ra, code) if code else None))
        want.append(ec.encode(ec.commit([int(x) for x in v], gens[:n])))
    got = ra.commit_batch(ctx, tables, dev_gens)
    assert got == want
    assert got == [ra.commit(ctx, t, dev_gens, d) for t, d in tables]
    import ctypes
    L = ra.lib()
    one = (ctypes.c_void_p * 65)(*([tables[0][0].data_ptr()] * 65))
    dts = (ctypes.c_int32 * 65)(*([ra.RA_I32] * 65))
    ns = (ctypes.c_uint64 * 65)(*([8] * 65))
    out = ctypes.create_string_buffer(64 * 65)
    assert L.ra_commit_batch(ctx.h, one, dts, ns, 0, dev_gens.data_ptr(), None, 0, out) == -1  # RA_E_INVAL
    assert L.ra_commit_batch(ctx.h, one, dts, ns, 65, dev_gens.data_ptr(), None, 0, out) == -9  # RA_E_NOT_IMPLEMENTED
    dts[1] = ra.RA_I64
    assert L.ra_commit_batch(ctx.h, one, dts, ns, 2, dev_gens.data_ptr(), None, 0, out) == -1  # RA_E_INVAL


# values at the edges of the 9-bit signed digits (a digit of -256, 255, 256, a carry into the top digit and out of
# 64 bits), and lengths at the edges of a sort and of a chunk
@pytest.mark.parametrize("n", [511, 1024, 1025, 2049])
@pytest.mark.parametrize("dt,code", DTYPES)
def test_commit_digit_and_sort_edges(ra, ctx, gens_small, n, dt, code):
    dev_gens, gens = gens_small
    info = np.iinfo(dt)
    edges = [(1 << b) + d for b in (0, 8, 9, 17, 18, 26, 27, 62, 63, 64) for d in (-1, 0, 1)]
    edges += [256 * sum(512 ** i for i in range(k)) + d for k in range(1, 8) for d in (-1, 0)]
    edges = [x for e in edges for x in (e, -e) if info.min <= x <= info.max] + [info.min, info.max]
    v = np.zeros(n, dtype=dt)
    pos = np.linspace(0, n - 1, len(edges)).astype(int)
    v[pos] = np.array(edges, dtype=dt)
    t = torch.from_numpy(v.view(np.int16 if dt == np.uint16 else (np.int64 if dt == np.uint64 else dt))).cuda()
    got = ra.commit(ctx, t, dev_gens, getattr(ra, code) if code else None)
    at = [int(i) for i in np.nonzero(v)[0]]
    assert got == ec.encode(ec.commit([int(v[i]) for i in at], [gens[i] for i in at]))


@pytest.mark.parametrize("n", [2, 700, 20000])
def test_commit_equal_and_opposite_points(ra, ctx, gens_small, n):
    """One generator at every position: sums of equal points (doublings), of
    opposite ones (the identity, in the middle of a run too) and of both."""
    dev_gens, gens = gens_small
    same = dev_gens[:1].expand(n, 16).contiguous()
    rng = np.random.default_rng(n)
    mixed = rng.integers(-300, 300, size=n).astype(np.int32)
    pairs = np.where(np.arange(n) & 1, -77, 77).astype(np.int32)
    pairs[n // 2 * 2:] = 0
    for v in (np.full(n, 5, dtype=np.int32), pairs, mixed):
        got = ra.commit(ctx, torch.from_numpy(v).cuda(), same)
        assert got == ec.encode(ec.commit([int(v.sum())], [gens[0]])), int(v.sum())


@pytest.mark.parametrize("n", [2, 1024, 5000])
def test_commit_edge_points(ra, ctx, n):
    """Points with y = q - 1 and y = 6 (x a cube root of y^2 - 7), whose limbs
    are all full or all empty, taken with either sign in every order within a
    thread's run and a bucket: the extremes of the lazy limbs, which hashed
    generators do not reach."""
    pts = []
    for y in (ec.Q - 1, 6):
        x = pow((y * y - 7) % ec.Q, (ec.Q + 2) // 9, ec.Q)  # q = 7 mod 9
        assert ec.on_curve((x, y)) and y % 2 == 0
        pts.append((x, y))
    rng = np.random.default_rng(n)
    which = rng.integers(0, 2, size=n)
    which[:2] = [0, 1]
    limbs = ra.point_limbs(pts)[which].view(np.int32)
    gens = torch.from_numpy(np.ascontiguousarray(limbs)).cuda()
    signs = rng.choice([-1, 1], size=n).astype(np.int32)
    for v in (np.full(n, -1, dtype=np.int32), np.full(n, 1, dtype=np.int32), signs):
        got = ra.commit(ctx, torch.from_numpy(v).cuda(), gens)
        sums = [int(v[which == g].sum()) for g in (0, 1)]
        assert got == ec.encode(ec.commit(sums, pts)), sums
