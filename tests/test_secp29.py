"""The field and point arithmetic of the commitments (csrc/secp29.hpp), built
for the host with traps on signed overflow, against Python's integers and the
oracle's curve: coordinates whose limbs are all near 0 or all near 2^29, which
hashed generators never have, and operands at the stated magnitude bounds."""
import itertools
import os
import random
import subprocess

import pytest

from oracle import ec_oracle as ec

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2505_17623_amd", "csrc")
Q = ec.Q

# The host stand-ins for the attributes, and one command per input line.  "sum": points added one by one the way a
# bucket's run does it (the first taken as it is, y negated by limbs); "full": two such sums by the general addition;
# "dbl": doublings in Jacobian coordinates; "inv"; "mul", "sqr", "msm": products of raw limbs.
STUB = """
#pragma once
#define __host__
#define __device__
#define __forceinline__ inline
#define __noinline__
"""
MAIN = r"""
#include <cinttypes>
#include <cstdio>
#include <cstring>
#include "secp29.hpp"
using namespace secp29;
static F field()
{
    uint32_t w[8];
    for (int i = 0; i < 8; i++)
        if (scanf("%" SCNx32, &w[i]) != 1) w[i] = 0;
    return from_limbs32(w);
}
static F limbs()
{
    F a;
    for (int i = 0; i < 9; i++)
        if (scanf("%" SCNd32, &a.v[i]) != 1) a.v[i] = 0;
    return a;
}
static Pt sum()
{
    int n = 0;
    if (scanf("%d", &n) != 1) return identity();
    Pt acc = identity();
    for (int i = 0; i < n; i++) {
        int s = 0;
        if (scanf("%d", &s) != 1) break;
        const F x = field();
        F y = field();
        if (s) y = neg(y);
        if (is_identity(acc)) acc = Pt{x, y, one(), one()};
        else add_affine(acc, x, y);
    }
    return acc;
}
static void put(F a)
{
    const secp::Fe c = canon(a);
    for (int i = 7; i >= 0; i--) printf("%08x", c.v[i]);
}
static void put(const Pt &p)
{
    if (is_identity(p)) {
        printf("0 0\n");
        return;
    }
    const F iz3 = inverse(p.ZZZ), iz = mul(iz3, p.ZZ);
    put(mul(p.X, sqr(iz)));
    printf(" ");
    put(mul(p.Y, iz3));
    printf("\n");
}
static void put_limbs(const F &a)
{
    for (int i = 0; i < 9; i++) printf("%d ", a.v[i]);
    printf("\n");
}
int main()
{
    char op[8];
    while (scanf("%7s", op) == 1) {
        if (!strcmp(op, "sum")) put(sum());
        else if (!strcmp(op, "full")) {
            const Pt a = sum(), b = sum();
            put(add(a, b));
        } else if (!strcmp(op, "dbl")) {
            int n = 0;
            if (scanf("%d", &n) != 1) return 1;
            Jac j = to_jac(sum());
            for (int i = 0; i < n; i++) j = dbl(j);
            put(from_jac(j));
        } else if (!strcmp(op, "inv")) {
            put(inverse(field()));
            printf("\n");
        } else if (!strcmp(op, "mul")) {
            const F a = limbs(), b = limbs();
            put_limbs(mul(a, b));
        } else if (!strcmp(op, "sqr")) put_limbs(sqr(limbs()));
        else if (!strcmp(op, "msm")) {
            const F a = limbs(), b = limbs(), c = limbs(), d = limbs();
            put_limbs(mul_sub_mul(a, b, c, d));
        } else return 1;
        fflush(stdout);
    }
    return 0;
}
"""


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    d = tmp_path_factory.mktemp("secp29")
    (d / "hip").mkdir()
    (d / "hip" / "hip_runtime.h").write_text(STUB)
    (d / "main.cpp").write_text(MAIN)
    exe = str(d / "secp29")
    subprocess.run(["g++", "-std=c++17", "-O0", "-ftrapv", "-w", f"-I{d}", f"-I{CSRC}", str(d / "main.cpp"), "-o", exe],
                   check=True)

    def go(lines):
        r = subprocess.run([exe], input="\n".join(lines) + "\n", capture_output=True, text=True, timeout=120)
        out = r.stdout.splitlines()
        at = lines[min(len(out), len(lines) - 1)]
        assert r.returncode == 0, f"signed overflow or failure ({r.returncode}) at: {at}"
        assert len(out) == len(lines)
        return out

    return go


def hex_words(a):
    return " ".join(f"{(a >> (32 * i)) & 0xFFFFFFFF:x}" for i in range(8))


def terms(ts):  # (negated, point) ..
    return f"{len(ts)} " + " ".join(f"{int(s)} {hex_words(p[0])} {hex_words(p[1])}" for s, p in ts)


def point(line):
    x, y = (int(v, 16) for v in line.split())
    return None if (x, y) == (0, 0) else (x, y)


def total(ts):
    acc = None
    for s, p in ts:
        acc = ec.add(acc, ec.neg(p) if s else p)
    return acc


def cube_root(a):
    """A cube root of a mod q, or None (q = 7 mod 9: a cube a has the root a^((q + 2) / 9))."""
    assert Q % 9 == 7
    r = pow(a, (Q + 2) // 9, Q)
    return r if pow(r, 3, Q) == a % Q else None


def edge_points():
    """Curve points with y, or x, at either end of [0, q): every limb 0 but the lowest, or every limb full."""
    pts = []
    for ys in (range(1, 60), range(Q - 1, Q - 60, -1)):
        found = [(x, y) for y in ys if y % 2 == 0 and (x := cube_root((y * y - 7) % Q)) is not None]
        pts += found[:3]
    for xs in (range(1, 60), range(Q - 1, Q - 60, -1)):
        for x in xs:
            y = pow((x ** 3 + 7) % Q, (Q + 1) // 4, Q)
            if y * y % Q == (x ** 3 + 7) % Q:
                pts += [(x, y if y % 2 == 0 else Q - y)]
                break
    assert len(pts) == 8 and all(ec.on_curve(p) for p in pts)
    return pts


def test_runs_of_edge_points(run):
    """Every pair, and triples, of edge points with every choice of signs."""
    pts = edge_points()
    cases = [list(zip(sg, ps)) for ps in itertools.product(pts, repeat=2) for sg in itertools.product((0, 1), repeat=2)]
    rng = random.Random(5)
    cases += [[(rng.randrange(2), rng.choice(pts)) for _ in range(n)] for n in (3, 3, 4, 8, 40) for _ in range(40)]
    out = run([f"sum {terms(c)}" for c in cases])
    for c, line in zip(cases, out):
        assert point(line) == total(c), c


def test_general_addition_and_doublings(run):
    pts = edge_points()
    rng = random.Random(6)
    pairs = [([(rng.randrange(2), rng.choice(pts)) for _ in range(rng.randrange(1, 4))],
              [(rng.randrange(2), rng.choice(pts)) for _ in range(rng.randrange(1, 4))]) for _ in range(150)]
    pairs += [([(s, p)], [(t, p)]) for p in pts for s in (0, 1) for t in (0, 1)]
    out = run([f"full {terms(a)} {terms(b)}" for a, b in pairs])
    for (a, b), line in zip(pairs, out):
        assert point(line) == ec.add(total(a), total(b))
    dbls = [(n, [(s, p)]) for p in pts for s in (0, 1) for n in (0, 1, 2, 71)]
    out = run([f"dbl {n} {terms(t)}" for n, t in dbls])
    for (n, t), line in zip(dbls, out):
        assert point(line) == ec.mul(2 ** n, total(t))


def test_inverse(run):
    rng = random.Random(7)
    vals = [0, 1, 2, 3, Q - 1, Q - 2, (Q + 1) // 2, 2 ** 255, 2 ** 29 - 1, Q >> 1] + [rng.randrange(Q) for _ in range(40)]
    for a, line in zip(vals, run([f"inv {hex_words(a)}" for a in vals])):
        assert int(line, 16) == pow(a, Q - 2, Q)


def value(v):
    return sum(x << (29 * i) for i, x in enumerate(v))


def test_products_at_the_magnitude_bound(run):
    """Operands of any signs with magnitudes m1 m2 < 3.5 (a b - c d: the sum of both below 3.5): no overflow, the
    right residue, and a result with limbs in (-2^21, 2^29 + 2^20)."""
    rng = random.Random(8)
    U = 1 << 29

    def operand(m):
        top = int(m * U)
        return rng.choice([[top] * 9, [-top] * 9, [rng.choice((-top, top)) for _ in range(9)],
                           [rng.randrange(-top, top + 1) for _ in range(9)]])

    def fmt(v):
        return " ".join(map(str, v))

    lines, want = [], []
    for m1, m2 in [(1.74, 2.0), (3.48, 1.0), (1.0, 3.48), (1.86, 1.86)] * 30:
        a, b = operand(m1), operand(m2)
        lines.append(f"mul {fmt(a)} {fmt(b)}")
        want.append(value(a) * value(b))
    for _ in range(60):
        a = operand(1.86)
        lines.append(f"sqr {fmt(a)}")
        want.append(value(a) ** 2)
        a, b, c, d = operand(1.7), operand(1.03), operand(1.7), operand(1.0)
        lines.append(f"msm {fmt(a)} {fmt(b)} {fmt(c)} {fmt(d)}")
        want.append(value(a) * value(b) - value(c) * value(d))
    for line, w in zip(run(lines), want):
        r = [int(x) for x in line.split()]
        assert value(r) % Q == w % Q
        assert all(-2 ** 21 < x < U + 2 ** 20 for x in r)
