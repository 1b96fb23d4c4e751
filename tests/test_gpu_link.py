"""The GPU prover of the gather links between layers (ra_link_prove) against
the oracle, through the C ABI: every word of every link and layer
transcript, and the challenge cursor, bit-exact on the small CNN (im2col and
flatten links) and on synthetic gathers; the full-size CNN against the
oracle's stored transcripts (tests/golden/full_links_cfg4.json, written by
make_golden.py --links, which calls only the oracle); the library verifier
on the GPU's proofs; the call's refusals."""
import hashlib
import json
import os

import numpy as np
import pytest
import torch

from helpers import diff_transcripts
from oracle import oracle as orc
from paper_2505_17623_amd import inputs

pytestmark = pytest.mark.gpu
GOLD = os.path.join(os.path.dirname(__file__), "golden")
P61 = (1 << 61) - 1


@pytest.fixture(scope="module")
def ra():
    from paper_2505_17623_amd import ra as ra_mod
    ra_mod.lib()
    assert torch.cuda.is_available()
    return ra_mod


def link_words(lk):
    return [list(lk["evals"]), lk["claim"], lk["z_at"], lk["w_at"]]


@pytest.mark.parametrize("deferred", [False, True])
def test_small_cnn_links_match_oracle(ra, deferred):
    wl = inputs.small(4)
    want = orc.prove_network(wl, links=True)
    ctx = ra.Context(wl.challenges, deferred=deferred)
    got = ra.prove_network(ctx, wl, links=True)
    ctx.sync()
    for li, (g, o) in enumerate(zip(got, want)):
        bad = diff_transcripts(g["transcript"], o)
        assert not bad, f"layer {li}: {bad}"
        assert np.array_equal(g["Z"].cpu().numpy().astype(np.int64), o["Z"])
        assert ("link" in g) == ("link" in o)
        if "link" in o:
            assert link_words(g["link"]) == link_words(o["link"]), f"layer {li} link"
    assert ctx.cursor() == want[-1]["cursor"]


# (|Z| as rows x cols, n x m of the next input, fraction of zero padding)
GATHERS = [(1, 1, 1, 1, 0.0), (2, 4, 4, 4, 0.3), (64, 32, 256, 16, 0.2), (256, 128, 512, 128, 0.5),
           (1024, 256, 2048, 512, 0.1)]


@pytest.mark.parametrize("zr,zc,n,m,pad", GATHERS)
def test_synthetic_gathers_match_oracle(ra, zr, zc, n, m, pad):
    """A layer, then a random gather of its output (repeated sources, padding)
    as the next layer's input, linked: the link words against the oracle's
    for the same stream and point."""
    rng = np.random.default_rng(zr * 7 + m)
    A0 = rng.integers(-3000, 3000, size=(zr, 8)).astype(np.int16)
    B0 = rng.integers(-3000, 3000, size=(8, zc)).astype(np.int16)
    src = rng.integers(0, zr * zc, size=n * m).astype(np.int32)
    src[rng.random(n * m) < pad] = -1
    B1 = rng.integers(-3000, 3000, size=(m, 4)).astype(np.int16)
    chal = inputs.xorshift64_stream(500 + zr + n, 2048)
    o0 = orc.prove_layer(A0, B0, 9, True, 0, chal, 0)
    A1 = np.where(src >= 0, o0["Z"].reshape(-1)[np.maximum(src, 0)], 0).reshape(n, m).astype(np.int32)
    o1 = orc.prove_layer(A1, B1, 9, True, 0, chal, o0["cursor"])
    z = orc.link_point(n, m, 4, chal, o0["cursor"])
    ol = orc.prove_link(o0["Z"], src, z, chal, o1["cursor"])
    ctx = ra.Context(chal)
    g0 = ra.prove_layer(ctx, torch.from_numpy(A0).cuda(), torch.from_numpy(B0).cuda(), 9, True, 0)
    g1 = ra.prove_layer(ctx, torch.from_numpy(A1).cuda(), torch.from_numpy(B1).cuda(), 9, True, 0)
    gl = ra.link_prove(ctx, g0["Z"], torch.from_numpy(src).cuda())
    assert not diff_transcripts(g1["transcript"], o1)
    assert link_words(gl) == link_words(ol)
    assert gl["claim"] == o1["a_star"]
    assert ctx.cursor() == ol["cursor"]


@pytest.mark.parametrize("vz", [1, 6, 10, 11, 12, 13, 14, 15, 17])
def test_link_passes_and_shared_sources(ra, vz):
    """Round counts around the passes' edges (none, one, two or three rounds
    in the last pass; 1 to 2^11 entries left), with maps in which up to 4096
    entries read one source, so that a weight's word wraps many times."""
    rng = np.random.default_rng(900 + vz)
    zr, zc = 1 << ((vz + 1) // 2), 1 << (vz // 2)
    n, m = 64, 64
    A0 = rng.integers(-3000, 3000, size=(zr, 2)).astype(np.int16)
    B0 = rng.integers(-3000, 3000, size=(2, zc)).astype(np.int16)
    B1 = rng.integers(-3000, 3000, size=(m, 2)).astype(np.int16)
    chal = inputs.xorshift64_stream(700 + vz, 2048)
    o0 = orc.prove_layer(A0, B0, 9, True, 0, chal, 0)
    for sources in (1, 3):
        src = rng.choice(rng.integers(0, zr * zc, size=sources), size=n * m).astype(np.int32)
        A1 = o0["Z"].reshape(-1)[src].reshape(n, m).astype(np.int32)
        o1 = orc.prove_layer(A1, B1, 9, True, 0, chal, o0["cursor"])
        ol = orc.prove_link(o0["Z"], src, orc.link_point(n, m, 2, chal, o0["cursor"]), chal, o1["cursor"])
        ctx = ra.Context(chal)
        g0 = ra.prove_layer(ctx, torch.from_numpy(A0).cuda(), torch.from_numpy(B0).cuda(), 9, True, 0)
        ra.prove_layer(ctx, torch.from_numpy(A1).cuda(), torch.from_numpy(B1).cuda(), 9, True, 0)
        gl = ra.link_prove(ctx, g0["Z"], torch.from_numpy(src).cuda())
        assert link_words(gl) == link_words(ol)
        assert ctx.cursor() == ol["cursor"]


def test_link_refusals(ra):
    chal = inputs.xorshift64_stream(31, 1024)
    A = torch.full((4, 4), 100, dtype=torch.int16).cuda()
    B = torch.full((4, 4), 100, dtype=torch.int16).cuda()
    Z = torch.zeros(16, dtype=torch.int32).cuda()
    src = torch.zeros(16, dtype=torch.int32).cuda()
    ctx = ra.Context(chal)
    with pytest.raises(ra.RAError) as e:                      # no layer proven yet
        ra.link_prove(ctx, Z, src)
    assert e.value.code == -7
    ra.prove_layer(ctx, A, B, 4, True, 0)
    with pytest.raises(ra.RAError) as e:                      # a map of the wrong size
        ra.link_prove(ctx, Z, src[:8].contiguous())
    assert e.value.code == -1
    with pytest.raises(ra.RAError) as e:                      # a previous output of 12 entries
        ra.link_prove(ctx, Z[:12].contiguous(), src)
    assert e.value.code == -1
    bad = src.clone()
    bad[5] = 16                                               # outside Z: refused, not followed
    with pytest.raises(ra.RAError) as e:
        ra.link_prove(ctx, Z, bad)
    assert e.value.code == -1
    bad[5] = -2
    with pytest.raises(ra.RAError) as e:
        ra.link_prove(ctx, Z, bad)
    assert e.value.code == -1
    cur = ctx.cursor()
    ra.link_prove(ctx, Z, src)                                # the refusals consumed nothing
    assert ctx.cursor() == cur + 4
    with pytest.raises(ra.RAError) as e:                      # one link per layer
        ra.link_prove(ctx, Z, src)
    assert e.value.code == -7


def test_gpu_link_proofs_verify(ra):
    wl = inputs.small(4)
    ctx = ra.Context(seed=wl.challenge_seed)
    got = ra.prove_network(ctx, wl, links=True)
    layers = []
    for li, g in enumerate(got):
        L = dict(A=g["A"].cpu().numpy(), B=wl.layers[li].B, Z=g["Z"].cpu().numpy(), R=g["R"].cpu().numpy(),
                 Rm=g["Rm"].cpu().numpy(), Y=g["Y"].cpu().numpy(), bits=g["bits"].cpu().numpy(),
                 transcript=g["transcript"], chained=li > 0 and wl.links[li] is None)
        if "link" in g:
            L["link_src"] = g["link_src"].cpu().numpy()
            L["link"] = g["link"]
        layers.append(L)
    assert ra.ra_verify(wl.challenge_seed, layers) == (0, 0)
    lk = layers[3]["link"]
    layers[3]["link"] = dict(lk, w_at=(lk["w_at"] + 1) % P61)
    assert ra.ra_verify(wl.challenge_seed, layers) == (15, 3)


def test_full_cnn_links_match_oracle(ra):
    """Config 4 at full size (32 images of 32x32x3, five layers, four links)."""
    gold = json.load(open(os.path.join(GOLD, "full_links_cfg4.json")))
    wl = inputs.workload(4, "full")
    ctx = ra.Context(seed=wl.challenge_seed, deferred=True)
    got = ra.prove_network(ctx, wl, links=True)
    ctx.sync()
    for li, (g, o) in enumerate(zip(got, gold["layers"])):
        bad = diff_transcripts(g["transcript"], o["transcript"])
        assert not bad, f"layer {li}: {bad}"
        z = hashlib.sha256(np.ascontiguousarray(g["Z"].cpu().numpy().astype("<i8")).tobytes()).hexdigest()
        assert z == o["digests"]["Z"]
        assert ("link" in g) == (o["link"] is not None)
        if o["link"] is not None:
            assert link_words(g["link"]) == link_words(o["link"]), f"layer {li} link"
    assert ctx.cursor() == gold["cursor"]
