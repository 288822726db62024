"""GPU parity of the routed per-expert calibration Grams and the loss table
against them (bitsmoe_gram_routed, bitsmoe_score_routed) vs oracle.routed.

Bars: every H_e within 1e-3 relative Frobenius; L within 1e-3 relative per
entry (1e-4 measured for the shared-H table).
"""
import sys

import numpy as np
import pytest

import oracle
import synth
from conftest import gpu_available
from oracle import routed

pytestmark = pytest.mark.gpu

if not gpu_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

import torch  # noqa: E402

import paper_2606_00079_amd as bm  # noqa: E402

DEV = "cuda:0"
REL = 1e-3


def say(*a):
    print("[gpu-routed]", *a, flush=True)
    sys.stdout.flush()


def dev(a, dtype):
    if dtype == "bf16":
        return torch.from_numpy(np.ascontiguousarray(a).view(np.int16)).view(torch.bfloat16).to(DEV)
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).to(DEV)


def relfro(a, b):
    a = np.asarray(a, np.float64)
    b = np.asarray(b, np.float64)
    return float(np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-300))


@pytest.mark.parametrize("config", ["tiny", "qwen_gate"])
def test_gram_routed(config):
    say("gram_routed", config)
    cfg = synth.CONFIGS[config]
    X = synth.calibration_input(cfg, cfg.projs[0].name)
    off, tok, w = synth.routing(cfg, X)
    Hs = bm.gram_routed(dev(X, cfg.dtype), off, tok, w).cpu().numpy()
    X64 = synth.as_f64(X, cfg.dtype)
    experts = range(cfg.E) if cfg.E <= 8 else [0, 1, 17, 63, 127]
    ref = routed.gram_routed(X64, off, tok, w)
    for e in experts:
        err = relfro(Hs[e], ref[e])
        assert err <= REL, (e, err)
        assert np.array_equal(Hs[e], Hs[e].T)
    # every token's weights sum to 1: the experts' Grams add up to the shared one
    Hsum = Hs.astype(np.float64).sum(axis=0)
    assert relfro(Hsum, oracle.gram(X64)) <= REL
    say("max rel fro", max(relfro(Hs[e], ref[e]) for e in experts))


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("d", [64, 256, 320, 576, 4160])
def test_grams_without_split(d, dt):
    """K loops too short to split, for every Gram of the library: part of a
    tile, a whole one, two and three tiles a side, and enough tiles (17 a
    side) that the GEMM writes them itself.  Bound: the products are exact but for the dropped
    lo x lo term (2^-18) and the rounding of w x to two bf16 terms (2^-17),
    and at most 64 terms are added in fp32 (64 x 2^-24)."""
    say("grams without split", d, dt)
    g = np.random.default_rng(d)
    X = synth.random_rows(50, d, seed=d, scale=1.0, heavy=True)
    Xd = dev(X, "f32") if dt == "f32" else dev(X, "f32").to(torch.bfloat16)
    X64 = Xd.double().cpu().numpy()
    bar = 2.0**-17 + 2.0**-18 + 64 * 2.0**-24
    H = bm.gram(Xd).cpu().numpy()
    assert np.array_equal(H, H.T) and relfro(H, X64.T @ X64 / 50) <= bar
    off = np.array([0, 20, 20, 50, 90], dtype=np.int64)
    tok = g.integers(0, 50, 90).astype(np.int32)
    w = g.random(90).astype(np.float32)
    Hs = bm.gram_routed(Xd, off, tok, w).cpu().numpy()
    ref = routed.gram_routed(X64, off, tok, w)
    for e in range(4):
        assert np.array_equal(Hs[e], Hs[e].T) and relfro(Hs[e], ref[e]) <= bar
    # W of one expert [d][64], M = W W^T in fp64, and the input-space form
    W = dev(synth.random_rows(d, 64, seed=d + 1, scale=1.0), "f32").to(Xd.dtype)
    W64 = W.double().cpu().numpy()
    M = bm.gram_experts(W[None]).cpu().numpy()
    assert M.dtype == np.float64 and np.array_equal(M, M.T) and relfro(M, W64 @ W64.T) <= bar
    Wt = W.t().contiguous()
    Mi = bm.gram_experts_in(Wt[None]).cpu().numpy()
    assert np.array_equal(Mi, Mi.T) and relfro(Mi, W64 @ W64.T) <= bar


@pytest.mark.parametrize("dt", ["f32", "bf16"])
def test_gram_routed_own_token_counts(dt):
    """Enough experts that K is not split: every expert's K ends with its own
    tokens, from none over the edges of a K tile to several tiles."""
    say("gram_routed own counts", dt)
    g = np.random.default_rng(8)
    E, n, d = 128, 300, 576
    cnt = np.r_[0, 1, 31, 32, 33, 63, 64, 65, 200, g.integers(0, 40, E - 9)].astype(np.int64)
    off = np.r_[0, np.cumsum(cnt)].astype(np.int64)
    tok = g.integers(0, n, off[-1]).astype(np.int32)
    w = g.random(off[-1]).astype(np.float32)
    X = dev(synth.random_rows(n, d, seed=8, scale=1.0, heavy=True), "f32")
    X = X if dt == "f32" else X.to(torch.bfloat16)
    Hs = bm.gram_routed(X, off, tok, w).cpu().numpy()
    ref = routed.gram_routed(X.double().cpu().numpy(), off, tok, w)
    for e in range(E):
        assert np.array_equal(Hs[e], Hs[e].T)
        # as for the shared Gram, over up to 200 tokens
        assert relfro(Hs[e], ref[e]) <= 2.0**-17 + 2.0**-18 + max(1, cnt[e]) * 2.0**-24, e
    assert np.all(Hs[0] == 0.0)


def test_gram_routed_empty_expert_and_ragged_rows():
    g = np.random.default_rng(3)
    X = synth.random_rows(150, 192, seed=3, scale=1.0, heavy=True)
    off = np.array([0, 40, 40, 107, 150], dtype=np.int64)
    tok = np.concatenate([np.sort(g.choice(150, 40, replace=False)), np.sort(g.choice(150, 67, replace=False)),
                          np.sort(g.choice(150, 43, replace=False))]).astype(np.int32)
    w = g.random(150).astype(np.float32)
    Hs = bm.gram_routed(dev(X, "f32"), off, tok, w).cpu().numpy()
    ref = routed.gram_routed(X.astype(np.float64), off, tok, w)
    assert np.all(Hs[1] == 0.0)
    for e in (0, 2, 3):
        assert relfro(Hs[e], ref[e]) <= REL


@pytest.mark.parametrize("E,upe,d,bits,group", [
    (4, 64, 256, (1, 2, 3, 4), 64),     # tiny shape: one 256-row tile per expert
    (3, 128, 768, (1, 2, 3, 4), 128),   # two tiles per expert, three row tiles of H
    (2, 256, 320, (1, 2, 4, 8), 64),    # ragged K block
])
def test_score_routed(E, upe, d, bits, group):
    say("score_routed", E, upe, d, bits, group)
    g = np.random.default_rng(E + upe + d)
    C = synth.random_rows(E * upe, d, seed=d, scale=0.05, heavy=True)
    C[0] = 0.0
    X = synth.random_rows(4 * d, d, seed=d + 1, scale=1.0, heavy=True)
    Hs = np.stack([oracle.gram(X[g.choice(4 * d, 2 * d, replace=False)].astype(np.float64)) *
                   (1.0 + e) for e in range(E)]).astype(np.float32)
    L = bm.score_routed(dev(C, "f32"), dev(Hs, "f32"), upe, bits, group).cpu().numpy()
    ref = routed.score_routed(C, Hs.astype(np.float64), upe, bits, group)
    assert np.all(L[0] == 0.0)
    err = float(np.max(np.abs(L[1:] - ref[1:]) / np.maximum(np.abs(ref[1:]), 1e-30)))
    say("max rel", err)
    assert err <= REL
    # the shared-H entry point agrees with the routed one when all H_e are equal
    Lsh = bm.score(dev(C, "f32"), dev(Hs[0], "f32"), bits, group).cpu().numpy()
    Lr = bm.score_routed(dev(C, "f32"), dev(np.stack([Hs[0]] * E), "f32"), upe, bits, group).cpu().numpy()
    assert np.array_equal(Lsh, Lr)


@pytest.mark.parametrize("scale", [1.0, 1e-7, 3e6])
def test_score_scale_of_matrices_without_a_dominant_diagonal(scale):
    """H_off's scale is taken from the diagonal and checked against every
    entry: symmetric matrices whose largest entry is off the diagonal (in the
    first and the last block of the upper triangle), on it, or whose diagonal
    is zero, next to each other.  Bound: fp16 rounding of both operands
    (2^-11 each) relative to the sum of the magnitudes of all terms."""
    say("score scale", scale)
    g = np.random.default_rng(11)
    d, upe, bits, group = 320, 64, (1, 2, 3, 4), 64
    S = g.standard_normal((4, d, d))
    S = (S + S.transpose(0, 2, 1)) / 2
    S[0] = S[0] @ S[0].T / d
    S[1, 0, 9] = S[1, 9, 0] = 70.0
    S[2, 300, 319] = S[2, 319, 300] = -500.0
    S[3][np.arange(d), np.arange(d)] = 0.0
    Hs = (S * scale).astype(np.float32)
    C = synth.random_rows(4 * upe, d, seed=5, scale=0.05, heavy=True)
    L = bm.score_routed(dev(C, "f32"), dev(Hs, "f32"), upe, bits, group).cpu().numpy()
    for e in range(4):
        rows = C[e * upe:(e + 1) * upe]
        H64 = Hs[e].astype(np.float64)
        ref = oracle.score(rows, H64, bits, group)
        mag = oracle.score(rows, np.abs(H64), bits, group)  # not below what cancels ...
        err = np.abs(L[e * upe:(e + 1) * upe] - ref)
        # ... but its own terms cancel too: the spread of the errors decides
        den = np.maximum(np.abs(mag), np.linalg.norm(H64) * _err2(rows, bits, group))
        assert np.all(err <= 2.0**-10 * den), (e, float(np.max(err / den)))
        one = bm.score(dev(rows, "f32"), dev(Hs[e], "f32"), bits, group).cpu().numpy()
        assert np.array_equal(one, L[e * upe:(e + 1) * upe])
    # enough matrices (44 of 320) that the scale comes from the diagonals: the
    # same bits as from the pass over all entries
    n = 11
    many = bm.score_routed(dev(np.tile(C, (n, 1)), "f32"), dev(np.tile(Hs, (n, 1, 1)), "f32"), upe, bits,
                           group).cpu().numpy()
    assert np.array_equal(many, np.tile(L, (n, 1)))


@pytest.mark.parametrize("nh,d", [(9, 1024), (1, 2112)])
def test_score_scale_second_look_takes_several_blocks(nh, d):
    """Matrices that fail the check of H_off's scale and have more blocks than
    the second look has workgroups (80 against 32 for more than eight
    matrices, 306 against 256 for one): every block is converted again.  The
    entries are random, so that a block left at the first scale would be wrong
    by a power of two in every row.  Bound as above."""
    say("second look", nh, d)
    g = np.random.default_rng(nh)
    upe, bits, group = 64, (1, 2, 3, 4), 64
    S = g.standard_normal((nh, d, d)).astype(np.float32)
    S = (S + S.transpose(0, 2, 1)) / 2
    for e in range(nh):  # in a block of its own for every matrix
        i, k = (29 * e) % d, d - 1 - (97 * e) % d
        S[e, i, k] = S[e, k, i] = 300.0
    C = synth.random_rows(nh * upe, d, seed=d, scale=0.05, heavy=True)
    L = bm.score_routed(dev(C, "f32"), dev(S, "f32"), upe, bits, group).cpu().numpy()
    for e in range(nh):
        rows = C[e * upe:(e + 1) * upe]
        H64 = S[e].astype(np.float64)
        ref = oracle.score(rows, H64, bits, group)
        den = np.maximum(np.abs(oracle.score(rows, np.abs(H64), bits, group)),
                         np.linalg.norm(H64) * _err2(rows, bits, group))
        err = np.abs(L[e * upe:(e + 1) * upe] - ref)
        assert np.all(err <= 2.0**-10 * den), (e, float(np.max(err / den)))
        if nh > 1:  # alone it takes the pass over all entries: the same bits (an even
            # number of row tiles: every sum runs in the same order)
            one = bm.score(dev(rows, "f32"), dev(S[e], "f32"), bits, group).cpu().numpy()
            assert np.array_equal(one, L[e * upe:(e + 1) * upe])


def _err2(rows, bits, group):
    """|delta|^2 of every row and width: the loss under H = I."""
    return oracle.score(rows, np.eye(rows.shape[1]), bits, group)


def test_routed_qwen_gate_full_size_sampled():
    """The Qwen3-30B-A3B gate shape: 128 routed Grams of 2048^2, the loss table
    of 49152 units against them, sampled rows checked."""
    cfg = synth.CONFIGS["qwen_gate"]
    X = synth.calibration_input(cfg, "gate")
    off, tok, w = synth.routing(cfg, X)
    Hs = bm.gram_routed(dev(X, cfg.dtype), off, tok, w)
    units, d, upe = 128 * 384, 2048, 384
    gen = torch.Generator(device="cuda").manual_seed(5)
    C = torch.randn(units, d, device="cuda", generator=gen) * 0.05
    L = bm.score_routed(C, Hs, upe, cfg.bits, cfg.group).cpu().numpy()
    rows = np.sort(np.random.default_rng(2).choice(units, 96, replace=False))
    Cs = C[torch.from_numpy(rows).cuda()].cpu().numpy()
    H64 = Hs.cpu().numpy().astype(np.float64)
    for i, u in enumerate(rows):
        ref = oracle.score_rows(Cs[i:i + 1], H64[u // upe], cfg.bits, cfg.group)[0]
        err = float(np.max(np.abs(L[u] - ref) / np.abs(ref)))
        assert err <= REL, (u, err)
