"""GPU parity: affmae_knn against the CPU oracle, bit-exact on every index."""
import numpy as np
import pytest
import torch

import oracle
import paper_2602_16249_amd as aff
from workloads import CONFIGS, make_workload

pytestmark = pytest.mark.gpu


def _gpu_knn(coords, cluster_id, S, M, K):
    c = torch.from_numpy(coords).cuda()
    cid = torch.from_numpy(cluster_id).cuda() if cluster_id is not None else None
    nbr, near = aff.affmae_knn(c, cid, S, M, K)
    torch.cuda.synchronize()
    return nbr.cpu().numpy(), near.cpu().numpy()


SMALL = [
    # name, B, N, S, M, K
    ("tiny_f32", 1, 256, 256, 1, 16),          # the exact-kNN configuration as specified
    ("tiny_f32", 2, 256, 32, 8, 16),           # M == G: exact through the clustered path
    ("mae_pt_s1_1024", 3, 1024, 64, 8, 48),    # on-grid, ties everywhere
    ("mae_pt_s1_1024", 2, 960, 48, 5, 33),     # ragged sizes: S, M*S, K not multiples of 64
    ("ft_s1_1024", 1, 16384, 64, 8, 48),       # one full 1024px image
    ("merged_stage", 4, 1024, 32, 8, 48),
    ("knn_scale", 2, 2048, 64, 8, 48),
    ("knn_scale", 2, 2048, 64, 8, 64),         # K at the limit
    ("knn_scale", 2, 512, 8, 3, 1),            # K = 1: every token is its own nearest
    ("knn_scale", 1, 640, 10, 64, 64),         # M at the limit, odd S
    ("knn_scale", 1, 4096, 64, 64, 64),        # the most candidates the library takes (4096)
    ("tiny_f32", 2, 1024, 128, 8, 48),         # 1024 candidates: the most that registers hold
]


@pytest.mark.parametrize("name,B,N,S,M,K", SMALL)
def test_knn_matches_oracle(name, B, N, S, M, K):
    cfg = CONFIGS[name].scaled(B=B, N=N, S=S, M=M, K=K)
    if cfg.coords == "jitter_grid" and N != 16384:
        cfg = cfg.scaled(frame=8.0 * int(round(N ** 0.5)))
    print(f"case {name} B={B} N={N} S={S} M={M} K={K}", flush=True)
    w = make_workload(cfg, features=False)
    nbr, near = _gpu_knn(w["coords"], None, S, M, K)
    rnbr, rnear = oracle.knn(w["coords"], None, S, M, K)
    assert np.array_equal(near, rnear)
    assert np.array_equal(nbr, rnbr)


def test_knn_with_scattered_cluster_ids():
    rng = np.random.default_rng(5)
    B, N, S, M, K = 2, 768, 24, 6, 40
    coords = rng.uniform(0, 300, size=(B, N, 2)).astype(np.float32)
    cid = np.stack([rng.permutation(np.repeat(np.arange(N // S), S)) for _ in range(B)]).astype(np.int32)
    nbr, near = _gpu_knn(coords, cid, S, M, K)
    rnbr, rnear = oracle.knn(coords, cid, S, M, K)
    assert np.array_equal(near, rnear)
    assert np.array_equal(nbr, rnbr)


def test_knn_coincident_points_and_integer_grid():
    """All distances tie in groups: order is decided by the index alone."""
    rng = np.random.default_rng(6)
    B, N, S, M, K = 1, 512, 32, 16, 48
    coords = rng.integers(0, 5, size=(B, N, 2)).astype(np.float32)
    nbr, near = _gpu_knn(coords, None, S, M, K)
    rnbr, rnear = oracle.knn(coords, None, S, M, K)
    assert np.array_equal(near, rnear)
    assert np.array_equal(nbr, rnbr)


@pytest.mark.parametrize("S,M,K", [(64, 8, 48), (64, 8, 64), (16, 4, 1), (128, 8, 48)])
def test_knn_all_points_identical(S, M, K):
    """Every distance is 0: no distance threshold separates K candidates, the index decides everything."""
    B, N = 2, 1024
    coords = np.full((B, N, 2), 3.25, dtype=np.float32)
    nbr, near = _gpu_knn(coords, None, S, M, K)
    rnbr, rnear = oracle.knn(coords, None, S, M, K)
    assert np.array_equal(near, rnear)
    assert np.array_equal(nbr, rnbr)


@pytest.mark.parametrize("name", ["mae_pt_s1_1024", "ft_s1_1024", "merged_stage", "knn_scale"])
def test_knn_full_size_configs(name):
    """The benchmark's configurations at full size, every index compared."""
    cfg = CONFIGS[name]
    print(f"case {name} full size", flush=True)
    w = make_workload(cfg, features=False)
    nbr, near = _gpu_knn(w["coords"], w["cluster_id"], cfg.S, cfg.M, cfg.K)
    rnbr, rnear = oracle.knn(w["coords"], w["cluster_id"], cfg.S, cfg.M, cfg.K)
    assert np.array_equal(near, rnear)
    assert np.array_equal(nbr, rnbr)
    # the table produced without an explicit assignment (tokens are in cluster order) is the same
    nbr2, near2 = _gpu_knn(w["coords"], None, cfg.S, cfg.M, cfg.K)
    assert np.array_equal(nbr2, rnbr) and np.array_equal(near2, rnear)


RAGGED = [
    # name, B, N, S, M, K: the last cluster holds N - (G - 1) S tokens
    ("mae_pt_s1_1024", 2, 4000, 64, 8, 48),    # 62 clusters of 64 and one of 32
    ("knn_scale", 2, 481, 32, 3, 20),          # a last cluster of one token
    ("knn_scale", 3, 33, 32, 2, 1),            # two clusters, the second a single token
    ("merged_stage", 2, 1001, 32, 8, 48),      # N odd: nothing is a whole tile
    ("tiny_f32", 2, 1000, 128, 8, 48),         # 1024 candidate places, 104 tokens in the last cluster
    ("knn_scale", 1, 100, 64, 2, 100),         # M == G: exact search over 100 tokens, K = all of them... capped below
]


@pytest.mark.parametrize("name,B,N,S,M,K", RAGGED)
def test_knn_short_last_cluster(name, B, N, S, M, K):
    K = min(K, 64)
    cfg = CONFIGS[name].scaled(B=B, N=N, S=S, M=M, K=K)
    print(f"case ragged {name} B={B} N={N} S={S} M={M} K={K}", flush=True)
    w = make_workload(cfg, features=False)
    nbr, near = _gpu_knn(w["coords"], None, S, M, K)
    rnbr, rnear = oracle.knn(w["coords"], None, S, M, K)
    assert near.shape == rnear.shape == (B, -(-N // S), M)
    assert np.array_equal(near, rnear)
    assert np.array_equal(nbr, rnbr)
    # the same clusters given as an explicit (scattered) assignment
    rng = np.random.default_rng(N)
    perm = np.stack([rng.permutation(N) for _ in range(B)])
    coords = np.ascontiguousarray(np.take_along_axis(w["coords"], perm[..., None], axis=1))
    cid = (perm // S).astype(np.int32)
    nbr_s, near_s = _gpu_knn(coords, cid, S, M, K)
    rnbr_s, rnear_s = oracle.knn(coords, cid, S, M, K)
    assert np.array_equal(near_s, rnear_s)
    assert np.array_equal(nbr_s, rnbr_s)


@pytest.mark.parametrize("explicit", [False, True])
@pytest.mark.parametrize("S,M,K", [(20, 3, 40), (40, 4, 33), (40, 9, 48), (64, 8, 48), (64, 11, 48), (64, 16, 64),
                                   (100, 11, 17), (128, 12, 64), (100, 11, 48), (100, 11, 49), (256, 5, 64), (32, 40, 63)])
def test_knn_rows_and_ties(S, M, K, explicit):
    """Every row class of the search (candidates in 1, 2, .. 16 rows of registers, or streamed) on points of which a
    third coincide in a few places (up to 90 at one distance, more than a threshold can separate), a third sits on a
    coarse grid (ties everywhere) and a third is free; then the same points shrunk until squared distances are
    subnormal.  Contiguous clusters and the same clusters as an explicit, scattered assignment."""
    rng = np.random.default_rng(S * M + K)
    B, N = 2, 1500
    pts = rng.uniform(0, 200, size=(B, N, 2))
    pts[:, 0::3] = rng.uniform(0, 200, size=(B, 6, 2))[:, rng.integers(0, 6, size=(N + 2) // 3)]
    pts[:, 1::3] = np.round(pts[:, 1::3] / 8) * 8
    order = np.lexsort((pts[0, :, 1] // 40, pts[0, :, 0] // 40))
    for shrink in (1.0, 1e-22):
        coords = np.ascontiguousarray((pts[:, order] * shrink).astype(np.float32))
        cid = None
        if explicit:
            perm = np.stack([rng.permutation(N) for _ in range(B)])
            coords = np.ascontiguousarray(np.take_along_axis(coords, perm[..., None], axis=1))
            cid = np.ascontiguousarray((perm // S).astype(np.int32))
        nbr, near = _gpu_knn(coords, cid, S, M, K)
        rnbr, rnear = oracle.knn(coords, cid, S, M, K)
        assert np.array_equal(near, rnear)
        assert np.array_equal(nbr, rnbr)


def _reference_knn_by_bits(coords, S, M, K):
    """Near clusters and neighbours of contiguous clusters by (bits of the fp32 squared distance, index): NaN distances
    come after every other, as the library orders them (the C oracle compares values, which NaN has no order in)."""
    B, N, _ = coords.shape
    G = -(-N // S)

    def keys(q, x, idx):
        with np.errstate(invalid="ignore", over="ignore"):
            d = x - q
            d2 = d[:, 0] * d[:, 0] + d[:, 1] * d[:, 1]  # fp32, one operation at a time
        bits = np.where(np.isnan(d2), np.uint32(0x7fc00000), d2.view(np.uint32)).astype(np.uint64)
        return (bits << np.uint64(32)) | idx.astype(np.uint64)

    nbr = np.empty((B, N, K), dtype=np.int32)
    near = np.empty((B, G, M), dtype=np.int32)
    for b in range(B):
        with np.errstate(invalid="ignore"):
            cen = np.stack([np.cumsum(coords[b, c * S:(c + 1) * S].astype(np.float64), axis=0)[-1] /
                            len(coords[b, c * S:(c + 1) * S]) for c in range(G)]).astype(np.float32)
        for c in range(G):
            near[b, c] = np.argsort(keys(cen[c], cen, np.arange(G)))[:M]
            cand = np.concatenate([np.arange(e * S, min((e + 1) * S, N)) for e in near[b, c]])
            for i in range(c * S, min((c + 1) * S, N)):
                nbr[b, i] = cand[np.argsort(keys(coords[b, i], coords[b, cand], cand))[:K]]
    return nbr, near


@pytest.mark.parametrize("bad", [np.nan, np.inf, 1e30])
@pytest.mark.parametrize("N,S,M,K", [(320, 32, 4, 24), (500, 32, 6, 64), (300, 64, 5, 40), (1100, 50, 22, 33)])
def test_knn_without_enough_distances(N, S, M, K, bad):
    """Tokens whose coordinates are NaN, infinite or too large to square: a few scattered ones, a whole cluster, and so
    many that a token has fewer than K distances left.  Every index is a candidate's, ordered by the distance's bits."""
    print(f"case bad={bad} N={N} S={S} M={M} K={K}", flush=True)
    rng = np.random.default_rng(N + K)
    coords = rng.uniform(0, 100, size=(4, N, 2)).astype(np.float32)
    coords[0, rng.permutation(N)[:5], 0] = bad
    coords[1, S:2 * S, 1] = bad
    coords[2, rng.permutation(N)[:N - 7], 0] = bad
    coords[3, :, :] = bad
    nbr, near = _gpu_knn(coords, None, S, M, K)
    rnbr, rnear = _reference_knn_by_bits(coords, S, M, K)
    assert np.array_equal(near, rnear)
    assert np.array_equal(nbr, rnbr)
    # the same clusters as an explicit assignment
    cid = np.broadcast_to((np.arange(N) // S).astype(np.int32), (4, N)).copy()
    nbr_e, near_e = _gpu_knn(coords, cid, S, M, K)
    assert np.array_equal(near_e, rnear)
    assert np.array_equal(nbr_e, rnbr)


@pytest.mark.parametrize("explicit", [False, True])
@pytest.mark.parametrize("G,S,M,K", [(64, 8, 64, 40), (65, 8, 7, 33), (128, 8, 60, 48), (129, 8, 64, 64), (192, 8, 5, 17),
                                     (193, 8, 63, 20), (255, 8, 64, 48), (256, 16, 3, 40), (257, 16, 64, 64), (257, 8, 2, 9),
                                     (1023, 8, 64, 48), (1025, 16, 9, 48)])
def test_knn_cluster_counts(G, S, M, K, explicit):
    """Near clusters found by the search kernel (up to 256 clusters per image: one to four rows of 64 centroids, the last
    one full or not) and by the kernel of their own beyond, with many equal centroid distances: the first image's points
    sit on a lattice, eight per place, the second's are free.  The last cluster is short."""
    print(f"case G={G} S={S} M={M} K={K} explicit={explicit}", flush=True)
    rng = np.random.default_rng(G + M)
    N = G * S - S // 2
    coords = rng.uniform(0, 60, size=(2, N, 2)).astype(np.float32)
    place = np.arange(N) // 8
    coords[0] = np.stack([place % 9, place // 9 % 7], axis=-1)
    coords[1] = coords[1][np.lexsort((coords[1, :, 1] // 8, coords[1, :, 0] // 8))]
    cid = None
    if explicit:
        perm = np.stack([rng.permutation(N) for _ in range(2)])
        coords = np.ascontiguousarray(np.take_along_axis(coords, perm[..., None], axis=1))
        cid = np.ascontiguousarray((perm // S).astype(np.int32))
    nbr, near = _gpu_knn(coords, cid, S, M, K)
    rnbr, rnear = oracle.knn(coords, cid, S, M, K)
    assert np.array_equal(near, rnear)
    assert np.array_equal(nbr, rnbr)
