"""GPU parity: affmae_cluster against the CPU oracle, bit-exact on every index."""
import numpy as np
import pytest
import torch

import oracle
import paper_2602_16249_amd as aff
from workloads import CONFIGS, make_workload

pytestmark = pytest.mark.gpu


def _gpu_cluster(coords, S, frame):
    order, cid = aff.affmae_cluster(torch.from_numpy(coords).cuda(), S, frame)
    torch.cuda.synchronize()
    return order.cpu().numpy(), cid.cpu().numpy()


CASES = [
    # B, N, S, frame, recipe
    (1, 1, 1, (0.0, 0.0, 1.0, 1.0), "uniform"),          # a single token
    (2, 2, 2, (0.0, 0.0, 8.0, 8.0), "uniform"),
    (3, 100, 7, (0.0, 0.0, 64.0, 64.0), "uniform"),      # padded to 128, ragged last cluster
    (2, 4096, 64, (0.0, 0.0, 1024.0, 1024.0), "uniform"),
    (2, 8192, 64, (0.0, 0.0, 1024.0, 1024.0), "normal"),   # four whole chunks; points outside the frame clamp
    (2, 8193, 64, (-3.5, 7.25, 900.0, 333.0), "normal"),   # a fifth chunk of one token and pads
    (1, 40000, 48, (0.0, 0.0, 512.0, 512.0), "uniform"),   # merged by the network, padded to 65536: several global steps
    (2, 5000, 16, (0.0, 0.0, 16.0, 16.0), "lattice"),      # integer lattice: many equal keys, index decides
]


@pytest.mark.parametrize("B,N,S,frame,recipe", CASES)
def test_cluster_matches_oracle(B, N, S, frame, recipe):
    print(f"case B={B} N={N} S={S} frame={frame} {recipe}", flush=True)
    rng = np.random.default_rng(100 + N)
    x0, y0, w, h = frame
    if recipe == "uniform":
        coords = np.stack([rng.uniform(x0, x0 + w, size=(B, N)), rng.uniform(y0, y0 + h, size=(B, N))], axis=-1)
    elif recipe == "normal":
        coords = np.stack([rng.normal(x0 + w / 2, w, size=(B, N)), rng.normal(y0 + h / 2, h, size=(B, N))], axis=-1)
    else:
        coords = rng.integers(0, 16, size=(B, N, 2)).astype(np.float64)
    coords = coords.astype(np.float32)
    order, cid = _gpu_cluster(coords, S, frame)
    rorder, rcid = oracle.cluster(coords, S, frame)
    assert np.array_equal(order, rorder)
    assert np.array_equal(cid, rcid)


def test_cluster_all_points_identical():
    coords = np.full((2, 3000, 2), 5.5, dtype=np.float32)
    order, cid = _gpu_cluster(coords, 64, (0.0, 0.0, 10.0, 10.0))
    assert np.array_equal(order, np.tile(np.arange(3000, dtype=np.int32), (2, 1)))
    assert np.array_equal(cid[0], np.arange(3000) // 64)


@pytest.mark.parametrize("name", ["mae_pt_s1_1024", "ft_s1_1024", "merged_stage", "knn_scale"])
def test_cluster_full_size_configs(name):
    """The benchmark's configurations at full size.  Their tokens come from the generator already in curve
    order, so the clustering must return the identity; a shuffled copy must come back to the same order."""
    cfg = CONFIGS[name]
    print(f"case {name} full size", flush=True)
    w = make_workload(cfg, features=False)
    frame = (0.0, 0.0, float(cfg.frame), float(cfg.frame))
    order, cid = _gpu_cluster(w["coords"], cfg.S, frame)
    rorder, rcid = oracle.cluster(w["coords"], cfg.S, frame)
    assert np.array_equal(order, rorder) and np.array_equal(cid, rcid)
    ident = np.tile(np.arange(cfg.N, dtype=np.int32), (cfg.B, 1))
    assert np.array_equal(order, ident)
    assert np.array_equal(cid, w["cluster_id"])
    rng = np.random.default_rng(9)
    perm = np.stack([rng.permutation(cfg.N) for _ in range(cfg.B)])
    shuffled = np.take_along_axis(w["coords"], perm[..., None], axis=1)
    order2, _ = _gpu_cluster(shuffled, cfg.S, frame)
    rorder2, _ = oracle.cluster(shuffled, cfg.S, frame)
    assert np.array_equal(order2, rorder2)
    # gathering the shuffled tokens by the returned order restores the curve order (equal keys keep
    # their shuffled index order, so compare coordinates of distinct-key neighbours through the oracle only)
    back = np.take_along_axis(shuffled, order2[..., None].astype(np.int64), axis=1)
    o3, _ = oracle.cluster(back, cfg.S, frame)
    assert np.array_equal(o3, ident)


@pytest.mark.parametrize("N", [63, 64, 65, 255, 256, 257, 512, 513, 1024, 1025, 2047, 2048, 2049, 4096, 4097, 32768, 32769])
def test_cluster_sizes_at_the_edges(N):
    """One workgroup's words per thread (1 or 2) and runs (1, 2 or 4), one chunk or several, the most chunks that are ranked
    (16) and the first size that the network merges: points on a lattice, so that the index decides among many equal keys."""
    rng = np.random.default_rng(N)
    coords = rng.integers(0, 40, size=(2, N, 2)).astype(np.float32)
    coords[1] *= 0.37
    order, cid = _gpu_cluster(coords, 48, (0.0, 0.0, 40.0, 40.0))
    rorder, rcid = oracle.cluster(coords, 48, (0.0, 0.0, 40.0, 40.0))
    assert np.array_equal(order, rorder)
    assert np.array_equal(cid, rcid)


@pytest.mark.parametrize("B,N", [(511, 2049), (512, 2049), (512, 4096), (64, 32768), (32, 33000)])
def test_cluster_many_chunks(B, N):
    """Chunks of large images sorted in registers or, from 1024 of them on, through LDS: ranked, and merged by the network."""
    rng = np.random.default_rng(B + N)
    coords = rng.integers(0, 300, size=(B, N, 2)).astype(np.float32)
    order, cid = _gpu_cluster(coords, 64, (0.0, 0.0, 300.0, 300.0))
    rorder, rcid = oracle.cluster(coords, 64, (0.0, 0.0, 300.0, 300.0))
    assert np.array_equal(order, rorder)
    assert np.array_equal(cid, rcid)


@pytest.mark.parametrize("B,N", [(64, 4096), (65, 4096), (85, 2049), (103, 2050), (38, 4100), (39, 4100), (12, 16384), (13, 16384)])
def test_cluster_chunk_sizes(B, N):
    """The largest batches whose images are sorted in chunks of 512 and of 1024 words, and the next: a lattice, so that words of
    different chunks share keys, with a part of the points beyond the frame's far corner, where the largest key is."""
    print(f"case chunk sizes B={B} N={N}", flush=True)
    rng = np.random.default_rng(B + N)
    coords = rng.integers(0, 50, size=(B, N, 2)).astype(np.float32)
    coords[:, ::7] += 100.0
    order, cid = _gpu_cluster(coords, 64, (0.0, 0.0, 50.0, 50.0))
    rorder, rcid = oracle.cluster(coords, 64, (0.0, 0.0, 50.0, 50.0))
    assert np.array_equal(order, rorder)
    assert np.array_equal(cid, rcid)


def test_cluster_many_small_images():
    """2^24 images of two tokens: the batch is cut, as a launch cannot have 256 threads for each image of such a batch."""
    B = 1 << 24
    x = torch.rand(B, device="cuda")
    coords = torch.stack([torch.stack([x, x], -1), torch.stack([1 - x, 1 - x], -1)], dim=1).contiguous()
    order, cid = aff.affmae_cluster(coords, 1, (0.0, 0.0, 1.0, 1.0))
    q = (coords[..., 0].double() * 65536).floor().clamp(0, 65535)  # both axes alike: the curve follows it
    first = (q[:, 1] < q[:, 0]).int()
    assert torch.equal(order, torch.stack([first, 1 - first], dim=1))
    assert torch.equal(cid, torch.stack([first, 1 - first], dim=1))  # (its own inverse)
