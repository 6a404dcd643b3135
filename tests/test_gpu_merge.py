"""GPU parity: affmae_merge_select / affmae_merge_fwd / affmae_merge_bwd against the CPU oracle.  Anchor indices
bit-exact; floats at max|gpu - ref| / max|ref| <= 1e-5 (fp32 storage) and 2e-2 (bf16 storage); dp, one scalar, is
judged against the sum of the absolute per-anchor contributions (returned by the oracle)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2602_16249_amd as aff
from workloads import CONFIGS, bf16_round, make_workload

pytestmark = pytest.mark.gpu

TOL = {"f32": 1e-5, "bf16": 2e-2}


@pytest.mark.parametrize("B,N,n_keep,kind", [
    (3, 1000, 250, "normal"), (2, 16384, 4096, "normal"), (2, 5000, 1, "ties"), (4, 777, 777, "ties"),
    (2, 4096, 1638, "ties"), (1, 100000, 40000, "ties"), (2, 64, 33, "equal"), (1, 2049, 1024, "normal"),
    # each size class of the selection: keys in registers (4, 16, 32 per thread), sizes that are not whole pieces
    (2, 4097, 1000, "ties"), (2, 16383, 16383, "normal"), (2, 20000, 5000, "ties"), (1, 32768, 1, "normal"),
    (1, 32769, 8192, "ties"), (3, 5, 5, "equal"), (2, 16384, 16384, "equal"),
])
def test_select_matches_oracle(B, N, n_keep, kind):
    print(f"case select B={B} N={N} n_keep={n_keep} {kind}", flush=True)
    rng = np.random.default_rng(N + n_keep)
    if kind == "normal":
        score = rng.normal(size=(B, N)).astype(np.float32)
    elif kind == "ties":  # few distinct values, both zeros, extremes of the fp32 range
        score = rng.choice(np.array([-3e38, -1.5, -0.0, 0.0, 1e-45, 0.25, 3.0, 3e38], dtype=np.float32), size=(B, N))
    else:
        score = np.full((B, N), 0.75, dtype=np.float32)
    coords = rng.uniform(0, 100, size=(B, N, 2)).astype(np.float32)
    idx, xy = aff.affmae_merge_select(torch.from_numpy(score).cuda(), n_keep, torch.from_numpy(coords).cuda())
    torch.cuda.synchronize()
    ref = oracle.merge_select(score, n_keep)
    assert np.array_equal(idx.cpu().numpy(), ref)
    assert np.array_equal(xy.cpu().numpy(), np.take_along_axis(coords, ref[..., None].astype(np.int64), axis=1))


CASES = [
    # dtype, B, N, C, K, S, M, n_keep, p
    ("f32", 2, 512, 64, 16, 32, 4, 128, 0.5),
    ("f32", 1, 256, 20, 7, 32, 2, 100, 1.3),      # rows of whole pieces (5), K odd
    ("f32", 2, 256, 6, 5, 16, 4, 64, 0.0),        # rows that are not whole 16-byte pieces: lanes are channels
    ("bf16", 2, 1024, 64, 48, 64, 8, 256, 0.25),  # the stage-1 shape: 8 pieces per row, 8 rows per trip
    ("bf16", 2, 512, 256, 48, 32, 8, 205, 0.7),   # 32 pieces per row
    ("bf16", 1, 512, 1032, 33, 64, 4, 77, 0.1),   # more than 64 pieces per row: several trips over the pieces
    ("bf16", 3, 300, 6, 64, 50, 6, 299, 2.0),     # K at the limit, odd rows, nearly every token an anchor
    ("bf16", 1, 128, 8, 1, 16, 2, 64, 1.0),       # K = 1: the merged token is the anchor itself
    ("f32", 2, 512, 64, 16, 32, 4, 128, 3.0),     # weights close to saturated on the anchor itself: gradients are small differences
    ("f32", 1, 256, 32, 12, 32, 2, 64, 8.0),
]


@pytest.mark.parametrize("dtype,B,N,C,K,S,M,n_keep,p", CASES)
def test_merge_forward_backward_match_oracle(dtype, B, N, C, K, S, M, n_keep, p):
    print(f"case merge {dtype} B={B} N={N} C={C} K={K} n_keep={n_keep} p={p}", flush=True)
    cfg = CONFIGS["knn_scale"].scaled(B=B, N=N, S=S, M=M, K=K)
    w = make_workload(cfg, features=False)
    coords = w["coords"]
    nbr, _ = oracle.knn(coords, None, S, M, K)
    rng = np.random.default_rng(N + C + K)
    feat = rng.normal(size=(B, N, C)).astype(np.float32)
    dout = rng.normal(size=(B, n_keep, C)).astype(np.float32)
    score = rng.normal(size=(B, N)).astype(np.float32)
    tdt = torch.float32
    if dtype == "bf16":
        feat, dout, tdt = bf16_round(feat), bf16_round(dout), torch.bfloat16
    d_coords, d_score = torch.from_numpy(coords).cuda(), torch.from_numpy(score).cuda()
    d_feat, d_dout = torch.from_numpy(feat).cuda().to(tdt), torch.from_numpy(dout).cuda().to(tdt)
    d_nbr = torch.from_numpy(nbr).cuda()
    anchors, _ = aff.affmae_merge_select(d_score, n_keep)
    out = aff.affmae_merge_fwd(d_feat, d_coords, d_score, d_nbr, anchors, p)
    g = aff.affmae_merge_bwd(d_feat, d_coords, d_score, d_nbr, anchors, d_dout, p)
    torch.cuda.synchronize()
    r_anchors = oracle.merge_select(score, n_keep)
    assert np.array_equal(anchors.cpu().numpy(), r_anchors)
    r_out = oracle.merge_fwd(coords, feat, score, nbr, r_anchors, p)
    rg = oracle.merge_bwd(coords, feat, score, nbr, r_anchors, dout, p)

    def err(a, ref):
        a = a.float().cpu().numpy().astype(np.float64)
        return float(np.abs(a - ref).max() / max(np.abs(ref).max(), 1e-30))

    tol = TOL[dtype]
    assert err(out, r_out) <= tol
    assert err(g["dfeat"], rg["dfeat"]) <= tol
    if K > 1:  # with one neighbour the weight is 1 whatever the score: dscore and dp are exactly 0
        assert err(g["dscore"], rg["dscore"]) <= tol
        assert abs(float(g["dp"].cpu()) - rg["dp"]) <= tol * rg["dp_abs"]
    else:
        assert float(g["dscore"].abs().max().cpu()) == 0.0 and float(g["dp"].cpu()) == 0.0


def test_merge_at_the_stage1_shape():
    """One step of the 1024px fine-tuning configuration going from stage 1 to stage 2 at d_s = 0.25: 8 images of
    16384 tokens, C = 64, K = 48, 4096 anchors each; the first two images against the oracle."""
    cfg = CONFIGS["ft_s1_1024"]
    w = make_workload(cfg, features=False)
    rng = np.random.default_rng(7)
    B, N, C, K, n_keep, p = cfg.B, cfg.N, cfg.C, cfg.K, cfg.N // 4, 0.25
    nbr_d, _ = aff.affmae_knn(torch.from_numpy(w["coords"]).cuda(), None, cfg.S, cfg.M, K)
    feat = bf16_round(rng.normal(size=(B, N, C)).astype(np.float32))
    dout = bf16_round(rng.normal(size=(B, n_keep, C)).astype(np.float32))
    score = rng.normal(size=(B, N)).astype(np.float32)
    d_coords, d_score = torch.from_numpy(w["coords"]).cuda(), torch.from_numpy(score).cuda()
    d_feat, d_dout = torch.from_numpy(feat).cuda().bfloat16(), torch.from_numpy(dout).cuda().bfloat16()
    anchors, _ = aff.affmae_merge_select(d_score, n_keep)
    out = aff.affmae_merge_fwd(d_feat, d_coords, d_score, nbr_d, anchors, p)
    g = aff.affmae_merge_bwd(d_feat, d_coords, d_score, nbr_d, anchors, d_dout, p, want_dp=False)
    torch.cuda.synchronize()
    nb = 2
    nbr = nbr_d[:nb].cpu().numpy()
    r_anchors = oracle.merge_select(score[:nb], n_keep)
    assert np.array_equal(anchors[:nb].cpu().numpy(), r_anchors)
    r_out = oracle.merge_fwd(w["coords"][:nb], feat[:nb], score[:nb], nbr, r_anchors, p)
    rg = oracle.merge_bwd(w["coords"][:nb], feat[:nb], score[:nb], nbr, r_anchors, dout[:nb], p)
    for a, ref in ((out[:nb], r_out), (g["dfeat"][:nb], rg["dfeat"]), (g["dscore"][:nb], rg["dscore"])):
        a = a.float().cpu().numpy().astype(np.float64)
        assert np.abs(a - ref).max() / np.abs(ref).max() <= 2e-2


@pytest.mark.parametrize("dtype,B,N,C,K,S,M,n_keep,p", [
    ("bf16", 2, 256, 32, 16, 32, 4, 100, 0.4),     # 4 pieces per row: 16 neighbours per trip
    ("bf16", 1, 256, 24, 33, 32, 4, 64, 0.4),      # 3 pieces, the fourth lane of each row idle
    ("f32", 1, 256, 44, 7, 32, 4, 60, 0.4),        # 11 pieces in 16 lanes
    ("bf16", 1, 256, 104, 64, 32, 4, 51, 0.4),     # 13 pieces, K at the limit
    ("f32", 1, 192, 132, 17, 32, 4, 50, 0.4),      # 33 pieces: one row per trip
    ("bf16", 1, 192, 512, 9, 32, 4, 50, 0.4),      # 64 pieces exactly
    ("f32", 1, 192, 260, 9, 32, 4, 50, 0.4),       # 65 pieces: two trips over the pieces
    ("f32", 1, 10000, 4, 3, 16, 2, 9000, 0.4),     # more groups per image than a workgroup of the pair lists holds
    ("bf16", 1, 10000, 8, 3, 16, 2, 8192, 0.4),    # exactly as many
])
def test_merge_row_shapes_and_long_group_lists(dtype, B, N, C, K, S, M, n_keep, p):
    test_merge_forward_backward_match_oracle(dtype, B, N, C, K, S, M, n_keep, p)


@pytest.mark.parametrize("dtype,C,K", [
    ("bf16", 512, 9), ("bf16", 256, 3), ("bf16", 64, 8), ("bf16", 64, 24), ("bf16", 64, 5), ("bf16", 32, 48),
    ("f32", 256, 5), ("f32", 64, 4), ("f32", 64, 12), ("f32", 64, 13), ("f32", 8, 16), ("f32", 6, 7), ("f32", 260, 3)])
def test_merge_of_infinite_features(dtype, C, K):
    """One token's features are infinite.  An anchor with that token among its neighbours, in any place (the last one is
    repeated to fill a trip of rows), has an infinite merged feature; every other anchor is what it was."""
    print(f"case merge infinite {dtype} C={C} K={K}", flush=True)
    rng = np.random.default_rng(C + K)
    N, n_keep, hot = 128, 100, 77
    coords = rng.uniform(0, 10, size=(1, N, 2)).astype(np.float32)
    nbr = np.stack([rng.permutation(N)[:K] for _ in range(N)])[None].astype(np.int32)
    nbr[0, :40, K - 1] = hot  # (a row may then hold it twice: its weight counts twice)
    score = rng.normal(size=(1, N)).astype(np.float32)
    feat = rng.normal(size=(1, N, C)).astype(np.float32)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    up = lambda x: torch.from_numpy(x).cuda()
    args = (up(coords), up(score), up(nbr), up(np.arange(n_keep, dtype=np.int32)[None]), 0.1)
    clean = aff.affmae_merge_fwd(up(feat).to(tdt), *args).float().cpu().numpy()
    feat[0, hot] = np.inf
    out = aff.affmae_merge_fwd(up(feat).to(tdt), *args).float().cpu().numpy()
    has = (nbr[0, :n_keep] == hot).any(axis=1)
    assert has.any() and not has.all()
    assert np.all(out[0, has] == np.inf)
    assert np.array_equal(out[0, ~has], clean[0, ~has])


@pytest.mark.parametrize("N", [3000, 16000, 20001])
@pytest.mark.parametrize("same", [1, 2, 255, 256, 257, 600])
@pytest.mark.parametrize("distinct", [True, False])
def test_select_when_few_keys_share_the_leading_bits(N, same, distinct):
    """`same` scores in one run of 1024 neighbouring fp32 values (all different, or seven values repeated), the others
    spread widely, and the cut before, at the first of, inside, at the last of and after the run."""
    print(f"case select N={N} same={same} distinct={distinct}", flush=True)
    rng = np.random.default_rng(N + same)
    offs = rng.permutation(1024)[:same] if distinct else rng.integers(0, 7, size=same)
    run = (np.float32(1.0).view(np.int32) + offs.astype(np.int32)).view(np.float32)
    high = rng.uniform(3.0, 9.0, size=(N - same) // 3).astype(np.float32)
    low = -np.exp(rng.uniform(-20, 20, size=N - same - high.size)).astype(np.float32)
    score = rng.permutation(np.concatenate([run, high, low]))[None]
    for n_keep in sorted({high.size, high.size + 1, high.size + (same + 1) // 2, high.size + same, high.size + same + 1}):
        idx, _ = aff.affmae_merge_select(torch.from_numpy(score).cuda(), n_keep)
        assert np.array_equal(idx.cpu().numpy(), oracle.merge_select(score, n_keep)), n_keep


@pytest.mark.parametrize("dtype,B,N,C,K,n_keep,few", [
    ("bf16", 1, 1500, 64, 48, 1100, 3),    # nearly all pairs name three tokens: lists that do not fit a workgroup's LDS
    ("f32", 2, 700, 16, 32, 500, 1),       # ... one token, and the second image's lists behind the first's
    ("bf16", 1, 40, 8, 24, 40, 0),         # fewer tokens than parts of an image
    ("bf16", 1, 64, 40, 5, 64, 0),         # as many; 5 pieces in 8 lanes
    ("f32", 1, 65, 4, 16, 30, 0),          # one more: parts of two tokens, the last half full
    ("bf16", 2, 4161, 64, 64, 4161, 0),    # 64 pairs a token: the fewest tokens a workgroup takes, a wave for each
    ("f32", 1, 1025, 96, 3, 1000, 0),      # 24 pieces: two trips of 16 lanes
    ("bf16", 300, 70, 16, 9, 20, 0),       # many small images
])
def test_merge_sums_per_token(dtype, B, N, C, K, n_keep, few):
    """dfeat, dscore and dp for neighbour tables of any kind (tokens named by nobody, by few, by all anchors)."""
    print(f"case merge sums {dtype} B={B} N={N} C={C} K={K} n_keep={n_keep} few={few}", flush=True)
    rng = np.random.default_rng(N + C + K)
    coords = rng.uniform(0, 30, size=(B, N, 2)).astype(np.float32)
    nbr = np.stack([[rng.permutation(N)[:K] for _ in range(N)] for _ in range(B)]).astype(np.int32)
    if few:
        nbr[:, :, : K - 2] = rng.integers(N - few, N, size=(B, N, K - 2))
    feat, dout = (rng.normal(size=(B, n, C)).astype(np.float32) for n in (N, n_keep))
    score = rng.normal(size=(B, N)).astype(np.float32)
    tdt = torch.float32
    if dtype == "bf16":
        feat, dout, tdt = bf16_round(feat), bf16_round(dout), torch.bfloat16
    anchors = oracle.merge_select(score, n_keep)
    up = lambda x: torch.from_numpy(x).cuda()
    g = aff.affmae_merge_bwd(up(feat).to(tdt), up(coords), up(score), up(nbr), up(anchors), up(dout).to(tdt), 0.3)
    torch.cuda.synchronize()
    rg = oracle.merge_bwd(coords, feat, score, nbr, anchors, dout, 0.3)
    for name in ("dfeat", "dscore"):
        got = g[name].float().cpu().numpy().astype(np.float64)
        # fp32 sums of up to n_keep K terms (here at most 5e4, of both signs): 1e-5 of the largest holds as elsewhere
        assert np.abs(got - rg[name]).max() <= TOL[dtype] * np.abs(rg[name]).max(), name
    assert abs(float(g["dp"].cpu()) - rg["dp"]) <= TOL[dtype] * rg["dp_abs"]


def _check_merge_bwd(dtype, coords, feat, dout, score, nbr, n_keep, p=0.3):
    """Backward on the GPU against the oracle; the sums of a token have up to 5e4 terms of both signs, whose fp32 roundings stay below
    1e-5 of the largest value as elsewhere."""
    tdt = torch.float32
    if dtype == "bf16":
        feat, dout, tdt = bf16_round(feat), bf16_round(dout), torch.bfloat16
    anchors = oracle.merge_select(score, n_keep)
    up = lambda x: torch.from_numpy(x).cuda()
    g = aff.affmae_merge_bwd(up(feat).to(tdt), up(coords), up(score), up(nbr), up(anchors), up(dout).to(tdt), p)
    torch.cuda.synchronize()
    rg = oracle.merge_bwd(coords, feat, score, nbr, anchors, dout, p)
    for name in ("dfeat", "dscore"):
        got = g[name].float().cpu().numpy().astype(np.float64)
        assert np.abs(got - rg[name]).max() <= TOL[dtype] * np.abs(rg[name]).max(), name
    assert abs(float(g["dp"].cpu()) - rg["dp"]) <= TOL[dtype] * rg["dp_abs"]


def _two_places(B, N, K, rng):
    """Neighbour tables as along a curve: half of a token's neighbours around itself, half around some other place of the image."""
    own = np.arange(N)[None, :, None] + rng.permuted(np.tile(np.arange(K), (B, N, 1)), axis=2)[..., : K - K // 2] - K // 2
    other = rng.integers(0, N, size=(B, N, 1)) + rng.permuted(np.tile(np.arange(K), (B, N, 1)), axis=2)[..., : K // 2]
    return (np.concatenate([own, other], axis=2) % N).astype(np.int32)


@pytest.mark.parametrize("B,N,K,n_keep", [
    (1, 4096, 12, 1024),    # 64 ranges of tokens, the most whose cells have a bit each
    (1, 4160, 12, 1024),    # 65: rows and columns of cells
    (2, 9001, 16, 3000),
    (1, 40001, 8, 9000),    # more than 1024 ranges' worth of cells: as many as there can be, the last short
    (5, 700, 16, 200),      # a dozen ranges an image
])
def test_merge_finds_the_anchors_of_a_range(B, N, K, n_keep):
    print(f"case merge cells B={B} N={N} K={K} n_keep={n_keep}", flush=True)
    rng = np.random.default_rng(N + K)
    coords = rng.uniform(0, 30, size=(B, N, 2)).astype(np.float32)
    feat, dout = (rng.normal(size=(B, n, 8)).astype(np.float32) for n in (N, n_keep))
    _check_merge_bwd("f32", coords, feat, dout, rng.normal(size=(B, N)).astype(np.float32), _two_places(B, N, K, rng), n_keep)


@pytest.mark.parametrize("dtype,B,N,C,K,n_keep,popular", [
    ("bf16", 64, 1024, 64, 48, 256, None),    # ranges of 128 tokens, 6144 pairs where all are kept: two parts each
    ("f32", 64, 1024, 16, 64, 300, None),     # three parts of 43 tokens: fewer than lanes
    ("bf16", 64, 1000, 128, 64, 250, None),   # a last range that is short
    ("f32", 16, 8192, 8, 16, 5000, 300),      # a token that all anchors name, between others: more pairs than places by itself
    ("bf16", 16, 8192, 264, 9, 4500, 0),      # ... the first of its range, in rows of three pieces a lane
    ("bf16", 16, 8192, 8, 9, 4500, 255),      # ... the last
    ("bf16", 8, 16384, 64, 48, 4096, None),   # four parts a range, in workgroups of their own
    ("f32", 1, 140000, 4, 64, 52000, None),   # more ranges than are looked at for crowds
])
def test_merge_of_crowded_anchors(dtype, B, N, C, K, n_keep, popular):
    """Anchors that lie side by side, as where an importance score picks out a structure: several times as many pairs per token
    as on average."""
    print(f"case merge crowd {dtype} B={B} N={N} C={C} K={K} n_keep={n_keep} popular={popular}", flush=True)
    rng = np.random.default_rng(N + C + K)
    coords = rng.uniform(0, 30, size=(B, N, 2)).astype(np.float32)
    nbr = ((np.arange(N)[None, :, None] + rng.permuted(np.tile(np.arange(K), (B, N, 1)), axis=2) - K // 2) % N).astype(np.int32)
    if popular is not None:
        nbr[:, :, K // 2] = popular  # (a row may then hold it twice: it counts twice)
    score = (np.where(np.arange(N) < n_keep, 10.0, 0.0)[None] + rng.normal(size=(B, N))).astype(np.float32)
    feat, dout = (rng.normal(size=(B, n, C)).astype(np.float32) for n in (N, n_keep))
    _check_merge_bwd(dtype, coords, feat, dout, score, nbr, n_keep)
