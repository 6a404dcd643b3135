"""GPU parity: affmae_pla_fwd / affmae_pla_bwd against the CPU oracle.

Tolerance (per tensor, forward and every gradient): max|gpu - ref| / max|ref|
<= 1e-5 for fp32 storage and <= 2e-2 for bf16 storage; the oracle runs in
double precision on the same stored (already rounded) inputs."""
import numpy as np
import pytest
import torch

import oracle
import paper_2602_16249_amd as aff
from helpers import LSE_TOL, TOL, check_attention, kernels_of, rel_err, run_gpu_attention, run_oracle_attention, to_dev
from workloads import CONFIGS, make_features, make_workload, random_neighbours

pytestmark = pytest.mark.gpu


def test_tiny_fp32_config():
    """B=1, N=256, C=64, 2 heads, K=16 exact neighbours, fp32."""
    cfg = CONFIGS["tiny_f32"]
    w = make_workload(cfg)
    nbr = oracle.knn_bruteforce(w["coords"], cfg.K)
    errs = check_attention(w, nbr, "f32", 1.0 / np.sqrt(cfg.d))
    print(errs)


GATHER_CASES = [
    # dtype, B, N, H, d, K, blank, distinct
    ("f32", 2, 200, 2, 32, 16, False, True),
    ("f32", 1, 130, 3, 16, 7, True, False),    # repeats, odd sizes, blank token
    ("f32", 1, 96, 1, 64, 64, True, True),     # K at the limit
    ("f32", 2, 64, 4, 32, 1, False, True),     # K = 1: out = v[nbr]
    ("bf16", 2, 200, 2, 32, 48, False, True),
    ("bf16", 1, 130, 8, 32, 48, True, False),
    ("bf16", 1, 77, 2, 64, 33, True, True),
    ("bf16", 1, 300, 4, 16, 5, False, False),
    ("bf16", 2, 150, 2, 16, 64, True, False),  # two pieces per row, both trips full; tokens that nobody lists
    ("f32", 1, 90, 2, 16, 64, False, True),
    ("bf16", 1, 70, 1, 64, 64, False, True),
]


@pytest.mark.parametrize("dtype,B,N,H,d,K,blank,distinct", GATHER_CASES)
def test_arbitrary_neighbour_tables(dtype, B, N, H, d, K, blank, distinct):
    """No cluster promise: any indices, repeats allowed (gather kernels)."""
    print(f"case {dtype} B={B} N={N} H={H} d={d} K={K} blank={blank} distinct={distinct}", flush=True)
    rng = np.random.default_rng(100 + N + K)
    w = make_features(B, N, H, d, K, dtype, rng, blank=blank)
    nbr = random_neighbours(B, N, K, rng, distinct=distinct)
    check_attention(w, nbr, dtype, 1.0 / np.sqrt(d), blank=blank)


def test_no_bias_argument():
    rng = np.random.default_rng(3)
    w = make_features(1, 128, 2, 32, 12, "bf16", rng)
    w["bias"] = None
    nbr = random_neighbours(1, 128, 12, rng)
    check_attention(w, nbr, "bf16", 0.2)


CLUSTER_CASES = [
    # name, B, N, C, H, K, S, M, blank
    ("mae_pt_s1_1024", 2, 1024, 64, 2, 48, 64, 8, False),
    ("mae_pt_s1_1024", 1, 1024, 64, 2, 48, 64, 8, True),
    ("merged_stage", 3, 512, 256, 8, 48, 32, 8, False),
    ("knn_scale", 2, 1024, 128, 4, 48, 64, 8, False),
    ("knn_scale", 1, 960, 96, 3, 20, 48, 5, True),     # ragged: S=48, M=5, H=3
    ("merged_stage", 2, 512, 64, 2, 64, 16, 32, False),  # 32 candidate tiles per strip: two passes of the bias tile
    ("tiny_f32", 1, 256, 64, 2, 16, 256, 1, False),    # one cluster per image (exact kNN), bf16 storage here
    ("merged_stage", 2, 224, 96, 3, 8, 32, 3, True),   # K = 8: one 16-byte chunk of slots per query
    ("merged_stage", 2, 64, 64, 2, 1, 16, 2, False),   # K = 1: every token attends to itself only
    ("mae_pt_s1_1024", 2, 1000, 64, 2, 48, 64, 8, True),   # N % 16 = 8: short last strip and token tile, blank sums
    ("merged_stage", 3, 250, 256, 8, 16, 32, 4, False),    # N % 16 = 10, eight heads (four head groups per tile)
    ("knn_scale", 1, 33, 64, 2, 12, 16, 2, True),          # three strips, the last of one query
    ("merged_stage", 2, 250, 96, 3, 7, 32, 4, True),       # short last strip with single-entry items and one head per sweep
]


@pytest.mark.parametrize("name,B,N,C,H,K,S,M,blank", CLUSTER_CASES)
@pytest.mark.parametrize("promise", ["none", "promise", "plan"])
def test_clustered_tables(name, B, N, C, H, K, S, M, blank, promise):
    """kNN tables of small clustered token sets: without the cluster promise
    (gather kernels), with it (near_clusters; tiled kernels, plan rebuilt inside
    the call) and with a plan built once by affmae_pla_plan."""
    print(f"case {name} B={B} N={N} C={C} H={H} K={K} S={S} M={M} blank={blank} promise={promise}", flush=True)
    cfg = CONFIGS[name].scaled(B=B, N=N, C=C, H=H, K=K, S=S, M=M, dtype="bf16")
    w = make_workload(cfg, blank=blank)
    nbr, near = oracle.knn(w["coords"], None, S, M, K)
    check_attention(w, nbr, cfg.dtype, 1.0 / np.sqrt(cfg.d), near=near if promise != "none" else None, S=S, M=M,
                    blank=blank, use_plan=promise == "plan")


@pytest.mark.parametrize("scale", [1.5, 4.0])
@pytest.mark.parametrize("blank", [False, True])
def test_wide_range_of_scores(scale, blank):
    """Logits with a standard deviation of 8 to 20: the running maximum of the streaming softmax rises many
    times along the tiles and most probabilities underflow next to the largest ones."""
    print(f"case wide scores scale={scale} blank={blank}", flush=True)
    cfg = CONFIGS["mae_pt_s1_1024"].scaled(B=2, N=1024, dtype="bf16")
    w = make_workload(cfg, blank=blank)
    nbr, near = oracle.knn(w["coords"], None, cfg.S, cfg.M, cfg.K)
    check_attention(w, nbr, cfg.dtype, scale, near=near, S=cfg.S, M=cfg.M, blank=blank, use_plan=True)


@pytest.mark.parametrize("name", ["mae_pt_s1_1024", "ft_s1_1024", "merged_stage", "knn_scale"])
def test_full_size_configs(name):
    """The benchmark's configurations at full size in the launch configuration
    the benchmark times (cluster promise given), every element compared."""
    cfg = CONFIGS[name]
    print(f"case {name} full size", flush=True)
    w = make_workload(cfg)
    nbr, near = oracle.knn(w["coords"], None, cfg.S, cfg.M, cfg.K)
    errs = check_attention(w, nbr, cfg.dtype, 1.0 / np.sqrt(cfg.d), near=near, S=cfg.S, M=cfg.M, use_plan=True)
    print(errs)


def test_full_image_with_blank_tokens():
    """Two full 1024px images with blank tokens: the blank column in the tiled forward and backward, and
    the sums for dk_blank / dv_blank over 2048 strips."""
    cfg = CONFIGS["ft_s1_1024"].scaled(B=2)
    print("case ft_s1_1024 B=2 blank", flush=True)
    w = make_workload(cfg, blank=True)
    nbr, near = oracle.knn(w["coords"], None, cfg.S, cfg.M, cfg.K)
    errs = check_attention(w, nbr, cfg.dtype, 1.0 / np.sqrt(cfg.d), near=near, S=cfg.S, M=cfg.M, blank=True,
                           use_plan=True)
    print(errs)


@pytest.mark.parametrize("seed", range(16))
def test_random_shapes_through_the_tiled_kernels(seed):
    """Seeded random N (mostly not a multiple of 16 or of S), S, M, K, H, batch and blank tokens: neighbour table by
    the oracle's clustered search, tiled kernels with the plan rebuilt inside the call and with a plan built once."""
    rng = np.random.default_rng(9000 + seed)
    while True:
        S = int(rng.choice([16, 32, 48, 64]))
        N = int(rng.integers(1, 70 if seed % 4 == 0 else 1500))
        G = (N + S - 1) // S
        M = int(rng.integers(1, min(G, 8) + 1))
        kmax = min(64, (M - 1) * S + N - (G - 1) * S)
        if M * S <= 1024 and kmax >= 1:
            break
    K, H, B = int(rng.integers(1, kmax + 1)), int(rng.choice([1, 2, 3, 4, 8])), int(rng.integers(1, 4))
    blank = bool(rng.integers(0, 2))
    name = ["mae_pt_s1_1024", "merged_stage", "knn_scale"][int(rng.integers(0, 3))]
    print(f"case {name} B={B} N={N} S={S} M={M} K={K} H={H} blank={blank}", flush=True)
    cfg = CONFIGS[name].scaled(B=B, N=N, C=32 * H, H=H, K=K, S=S, M=M, dtype="bf16")
    w = make_workload(cfg, blank=blank)
    nbr, near = oracle.knn(w["coords"], None, S, M, K)
    for use_plan in (False, True):
        check_attention(w, nbr, "bf16", 1.0 / np.sqrt(32), near=near, S=S, M=M, blank=blank, use_plan=use_plan)


def test_instrumented_library_gives_the_same_bits():
    """The bench takes its per-kernel times in the instrumented twin library (the same sources with events around
    every launch): its tiled forward and backward results are bit-equal to the product library's."""
    from helpers import run_gpu_attention
    cfg = CONFIGS["ft_s1_1024"].scaled(B=1)
    print("case ft_s1_1024 B=1 product against instrumented library", flush=True)
    w = make_workload(cfg)
    nbr, near = oracle.knn(w["coords"], None, cfg.S, cfg.M, cfg.K)
    scale = 1.0 / np.sqrt(cfg.d)
    out, lse, g = run_gpu_attention(w, nbr, cfg.dtype, scale, near, cfg.S, cfg.M, use_plan=True)
    aff.use_timed_library(True)
    try:
        tout, tlse, tg = run_gpu_attention(w, nbr, cfg.dtype, scale, near, cfg.S, cfg.M, use_plan=True)
    finally:
        aff.use_timed_library(False)
    assert torch_equal(out, tout) and torch_equal(lse, tlse)
    for name in g:
        assert torch_equal(g[name], tg[name]), name


def torch_equal(a, b):
    import torch
    return a is None and b is None or torch.equal(a, b)


def test_gather_kernels_on_full_images():
    """Two full 1024px images without the cluster promise: the gather kernels at the benchmark's shape (16384
    queries per image: the list builder of the backward takes them in two sweeps), every element compared; the
    same with a table whose neighbours are drawn from the whole image (no locality: every token range of the list
    builder has to walk every query)."""
    cfg = CONFIGS["ft_s1_1024"].scaled(B=2)
    print("case ft_s1_1024 B=2 gather kernels", flush=True)
    w = make_workload(cfg, blank=True)
    nbr, _ = oracle.knn(w["coords"], None, cfg.S, cfg.M, cfg.K)
    print(check_attention(w, nbr, cfg.dtype, 1.0 / np.sqrt(cfg.d), blank=True))
    print("case ft_s1_1024 B=2 gather kernels, neighbours without locality", flush=True)
    rng = np.random.default_rng(77)
    nbr = random_neighbours(cfg.B, cfg.N, cfg.K, rng, distinct=False)
    print(check_attention(w, nbr, cfg.dtype, 1.0 / np.sqrt(cfg.d), blank=True))


@pytest.mark.parametrize("use_plan", [False, True])
@pytest.mark.parametrize("bias", [True, False])
def test_promise_with_permuted_neighbour_lists(use_plan, bias):
    """The cluster promise asks for distinct neighbours inside the near clusters, not for distance order: every
    token's list is shuffled (the oracle's results are invariant to that order up to the slot each bias value
    belongs to, and it gets the same shuffled table).  Also the tiled kernels without a bias tensor."""
    print(f"case permuted lists plan={use_plan} bias={bias}", flush=True)
    cfg = CONFIGS["knn_scale"].scaled(B=2, N=1024, C=64, H=2, dtype="bf16")
    w = make_workload(cfg, blank=True)
    nbr, near = oracle.knn(w["coords"], None, cfg.S, cfg.M, cfg.K)
    rng = np.random.default_rng(17)
    nbr = np.ascontiguousarray(rng.permuted(nbr, axis=2))
    if not bias:
        w["bias"] = None
    check_attention(w, nbr, cfg.dtype, 1.0 / np.sqrt(cfg.d), near=near, S=cfg.S, M=cfg.M, blank=True, use_plan=use_plan)


@pytest.mark.parametrize("N,tiled", [(4000, True), (4001, True), (3983, True)])
def test_short_last_cluster_end_to_end(N, tiled):
    """coords -> affmae_cluster -> affmae_knn -> affmae_pla_fwd / affmae_pla_bwd with N not a multiple of the
    cluster size (a masked batch keeps whatever number of tokens the mask leaves): curve order, neighbour table
    and near clusters bit-equal to the oracle, attention within the bf16 bound, in the tiled kernels: N = 4000
    (whole 16-token tiles, short last cluster), N = 4001 (a last strip and token tile of one token, which is also
    the whole last cluster), N = 3983 (fifteen tokens in the last tile)."""
    import torch
    print(f"case end to end N={N}", flush=True)
    S, M, K, H, d = 64, 8, 48, 2, 32
    cfg = CONFIGS["mae_pt_s1_1024"].scaled(B=2, N=N, C=H * d, H=H, K=K, S=S, M=M, dtype="bf16")
    w = make_workload(cfg)
    rng = np.random.default_rng(N)
    perm = np.stack([rng.permutation(N) for _ in range(cfg.B)])
    shuffled = np.ascontiguousarray(np.take_along_axis(w["coords"], perm[..., None], axis=1))
    frame = (0.0, 0.0, float(cfg.frame), float(cfg.frame))
    order, cid = aff.affmae_cluster(torch.from_numpy(shuffled).cuda(), S, frame)
    rorder, rcid = oracle.cluster(shuffled, S, frame)
    assert np.array_equal(order.cpu().numpy(), rorder) and np.array_equal(cid.cpu().numpy(), rcid)
    coords = np.ascontiguousarray(np.take_along_axis(shuffled, rorder[..., None].astype(np.int64), axis=1))
    nbr_d, near_d = aff.affmae_knn(torch.from_numpy(coords).cuda(), None, S, M, K)
    nbr, near = oracle.knn(coords, None, S, M, K)
    assert np.array_equal(nbr_d.cpu().numpy(), nbr) and np.array_equal(near_d.cpu().numpy(), near)
    assert (aff.load_library().affmae_pla_plan_bytes(cfg.B, N, K, S, M) > 0) == tiled
    check_attention(w, nbr, "bf16", 1.0 / np.sqrt(d), near=near, S=S, M=M, use_plan=tiled)


@pytest.mark.parametrize("N,S,M,K,same,B", [
    (2048, 16, 32, 40, True, 1),     # every strip touches the same three token tiles
    (700, 32, 16, 24, True, 1),      # the same with a short last strip
    (32768, 64, 8, 16, False, 1),    # large images: counted, scanned, filled and sorted in launches of their own
    (32785, 64, 8, 16, False, 1),
    (16384, 64, 8, 16, False, 1),    # the most token tiles of the one-launch reverse tables, and one more
    (16385, 64, 8, 16, False, 1),
    (8192, 64, 8, 16, False, 1),     # half of that
    (8200, 64, 8, 16, False, 1),
    (16384, 64, 8, 8, False, 8),     # more groups than workgroups: eight a workgroup, or seven and a last one with fewer
    (16384, 64, 8, 8, False, 7),
    (16304, 64, 8, 8, False, 7),
    (32768, 64, 8, 4, False, 16),    # large batches of large images, whole tiles and not
    (32769, 64, 8, 4, False, 16),
    (48, 16, 2, 8, False, 768),      # the most images of a few tiles in one launch
    (64, 16, 2, 8, False, 600),      # more images than workgroups wanted: one for each
    (48, 16, 2, 8, False, 769),      # more images of a few tiles than one launch serves well
])
def test_reverse_tables_of_the_plan(N, S, M, K, same, B):
    """dk and dv walk the plan's reverse tables: lists of more than 64 strips (all points coincide, so that the index
    decides and all queries share their neighbours) and both ways of building the tables."""
    print(f"case reverse tables B={B} N={N} S={S} M={M} K={K}", flush=True)
    cfg = CONFIGS["knn_scale"].scaled(B=B, N=N, C=32, H=1, K=K, S=S, M=M, dtype="bf16")
    w = make_workload(cfg)
    if same:
        w["coords"] = np.full_like(w["coords"], 2.5)
    nbr, near = oracle.knn(w["coords"], None, S, M, K)
    check_attention(w, nbr, cfg.dtype, 1.0 / np.sqrt(32), near=near, S=S, M=M, use_plan=True)


@pytest.mark.parametrize("N,B,strips", [
    (4096, 1, 60), (4096, 1, 100),     # one group that 65 or more strips touch beside the usual lists
    (16384, 1, 1000),                  # more entries than a workgroup of the one launch has room for at a time: in two steps
    (16384, 8, 1000), (8192, 3, 500),  # the same with several groups a workgroup
    (16400, 1, 60), (16400, 2, 300), (20480, 1, 1270),  # large images: lists of a group sorted by one wave each
])
def test_popular_groups_of_tiles(N, B, strips):
    """`strips` strips in a row have, beside their own surroundings, neighbours in the first cluster: lists of the reverse tables
    on both sides of 64 and of 1024 entries."""
    print(f"case popular groups B={B} N={N} strips={strips}", flush=True)
    S, M, K = 64, 5, 8
    rng = np.random.default_rng(strips)
    G = -(-N // S)
    near = np.stack([np.arange(M) + min(max(c - 1, 0), G - M) for c in range(G)]).astype(np.int32)
    first = (G - strips * 16 // S) // 2 + 3 if strips < G * S // 16 - 40 else 4
    far = (np.arange(G) >= max(first, M)) & (np.arange(G) < first + -(-strips * 16 // S))
    near[far, M - 1] = 0
    cand = (near[:, :, None] * S + np.arange(S)).reshape(G, M * S)
    nbr = np.empty((N, K), np.int32)
    for i in range(N):
        c = cand[i // S]
        nbr[i] = rng.choice(c[c < N], K, replace=False)
    w = make_features(B, N, 1, 32, K, "bf16", rng)
    many = lambda t: np.repeat(t[None], B, axis=0)
    check_attention(w, many(nbr), "bf16", 0.2, near=many(near), S=S, M=M, use_plan=True)


@pytest.mark.parametrize("N", [16, 512, 528, 4080, 4112, 8192 + 16])
def test_blank_sums_over_strips(N):
    """dk_blank / dv_blank add one part per strip, 32 x 8 strips per trip: 1, 32, 33, 255, 257 and 513 strips."""
    print(f"case blank sums N={N}", flush=True)
    cfg = CONFIGS["knn_scale"].scaled(B=1, N=N, C=32, H=1, K=8, S=16, M=min(4, N // 16), dtype="bf16")
    w = make_workload(cfg, blank=True)
    nbr, near = oracle.knn(w["coords"], None, cfg.S, cfg.M, cfg.K)
    check_attention(w, nbr, cfg.dtype, 1.0 / np.sqrt(32), near=near, S=cfg.S, M=cfg.M, blank=True, use_plan=True)


@pytest.mark.parametrize("dtype,d", [("f32", 16), ("f32", 32), ("f32", 64), ("bf16", 16), ("bf16", 32), ("bf16", 64)])
@pytest.mark.parametrize("K", ["1", "trip", "trip+1", "trips", "trips+1", "last-1", "64"])
def test_gather_trips(dtype, d, K):
    """Neighbour counts at the edges of one trip (64 * 16 bytes of rows) and of two, lists of more than 64 pairs under one
    token, and, in the longest case, more tokens than the grid with blank gradients covers in one go."""
    trip = 64 // (d * (4 if dtype == "f32" else 2) // 16)
    K = {"1": 1, "trip": trip, "trip+1": trip + 1, "trips": 2 * trip, "trips+1": min(2 * trip + 1, 64),
         "last-1": 65 - trip, "64": 64}[K]
    N = 4500 if K == 1 else 150
    print(f"case trips {dtype} d={d} K={K}", flush=True)
    rng = np.random.default_rng(K + d)
    w = make_features(1, N, 2, d, K, dtype, rng, blank=True)
    nbr = rng.integers(0, N, size=(1, N, K)).astype(np.int32)
    nbr[:, :, 0] = np.where(rng.uniform(size=(1, N)) < 0.6, 3, nbr[:, :, 0])
    check_attention(w, nbr, dtype, 1.0 / np.sqrt(d), blank=True)


def test_plan_of_many_small_images():
    """2^22 images of one token each: the one-launch reverse tables would need more threads than a launch can have.  The
    images repeat 1024 different ones, whose gradients a plan of 1024 images gives too."""
    B, few = 1 << 22, 1024
    print(f"case plan B={B} N=1", flush=True)
    g = torch.Generator(device="cuda").manual_seed(22)
    q, k, v, dout = (torch.randn(few, 1, 1, 32, device="cuda", generator=g).bfloat16() for _ in range(4))
    bias = torch.randn(few, 1, 1, 1, device="cuda", generator=g).bfloat16()
    kb, vb = (torch.randn(1, 32, device="cuda", generator=g).bfloat16() for _ in range(2))

    def run(n):
        rep = lambda t: t.repeat(n // few, 1, 1, 1)
        nbr = torch.zeros(n, 1, 1, dtype=torch.int32, device="cuda")
        plan = aff.affmae_pla_plan(nbr, nbr, 16, 1)
        a = (rep(q), rep(k), rep(v), rep(bias), nbr)
        out, lse = aff.affmae_pla_fwd(*a, 0.2, nbr, 16, 1, kb, vb, plan=plan)
        gr = aff.affmae_pla_bwd(*a, out, lse, rep(dout), 0.2, nbr, 16, 1, kb, vb, plan=plan)
        return [out, lse] + [gr[name] for name in ("dq", "dk", "dv", "dbias")]

    for big, small in zip(run(B), run(few)):
        assert small.float().abs().max() > 0
        assert torch.equal(big.view(B // few, *small.shape), small[None].expand(B // few, *small.shape))


def _near_table(B, N, S, M, K, spread, rng):
    """A table that keeps the cluster promise without coming from a search: cluster c is near to the M clusters around it
    (spread False) or to M clusters drawn from the whole image, and a token's K distinct neighbours are drawn from them."""
    G = N // S
    near = np.empty((B, G, M), np.int32)
    nbr = np.empty((B, N, K), np.int32)
    for b in range(B):
        for c in range(G):
            near[b, c] = rng.choice(G, M, replace=False) if spread else (np.arange(M) + min(max(c - M // 2, 0), G - M))
            cand = (near[b, c][:, None] * S + np.arange(S)).reshape(-1)
            for i in range(c * S, (c + 1) * S):
                nbr[b, i] = rng.choice(cand, K, replace=False)
    return nbr, near


@pytest.mark.parametrize("N,S,M,K,H,spread", [
    (512, 64, 4, 16, 2, False),    # 16 tiles: as many as the forward kernel holds
    (512, 32, 8, 48, 1, False),    # 16 .. 22 tiles: two stages
    (1024, 64, 5, 48, 2, False),   # 20 tiles: as many as the narrow kernels hold and keep in registers, less 4
    (1024, 64, 6, 56, 2, False),   # 24 tiles and rows of more than 48 values: three stages of the backward kernel
    (1024, 64, 8, 48, 1, False),   # 32 tiles, strips of 32 slots: more pairs than are held in registers
    (512, 16, 25, 33, 1, True),    # 32 tiles at most, an odd number of neighbours
    (2048, 16, 64, 64, 1, True),   # unions of the whole image (128 tiles), strips of 64 slots, every list of 128 strips
    (2096, 16, 40, 40, 2, True),   # the same with a last group of three strips
])
def test_unions_of_many_tiles(N, S, M, K, H, spread):
    """Groups of strips that touch from 16 to 131 token tiles together, at the sizes where the tiled kernels change the way
    they hold them: all in LDS, a second stage from registers, further stages from memory."""
    print(f"case unions N={N} S={S} M={M} K={K} H={H}", flush=True)
    rng = np.random.default_rng(N + M + K)
    nbr, near = _near_table(1, N, S, M, K, spread, rng)
    w = make_features(1, N, H, 32, K, "bf16", rng, blank=True)
    check_attention(w, nbr, "bf16", 1.0 / np.sqrt(32), near=near, S=S, M=M, blank=True, use_plan=True)


@pytest.mark.parametrize("K", [16, 15, 62])
@pytest.mark.parametrize("few", [1, 2, 3, 5, 8])
def test_strips_of_few_tiles_in_large_unions(few, K):
    """One strip of every group has neighbours in the image's first tiles only, the other three all over it: the first stage of
    the walk, which frees places for tiles still to come, is all that there is for the one."""
    print(f"case few tiles {few} K={K}", flush=True)
    N, S, H = 400, 16, 2
    few = max(few, -(-K // 16))
    G = N // S
    rng = np.random.default_rng(10 * K + few)
    near = np.broadcast_to(np.arange(G, dtype=np.int32), (1, G, G)).copy()
    nbr = np.stack([rng.choice(16 * few if i // 16 % 4 == 1 else N, K, replace=False) for i in range(N)]).astype(np.int32)[None]
    w = make_features(1, N, H, 32, K, "bf16", rng, blank=True)
    check_attention(w, nbr, "bf16", 0.2, near=near, S=S, M=G, blank=True, use_plan=True)


# (no blank column where it would leave the neighbours probabilities below fp32's range: the gradients would be compared with
# values that are not representable)
@pytest.mark.parametrize("low,high,blank", [(-3.0e4, -3.0e4, False), (-500.0, -500.0, False), (3.0e4, 3.0e4, False), (3.0e4, 3.0e4, True),
                                            (-60.0, 90.0, False), (-60.0, 90.0, True), (-200.0, 3.0, False)])
@pytest.mark.parametrize("N,S,M,K", [(256, 32, 4, 20), (1024, 64, 6, 48), (1001, 32, 4, 24)])
def test_scores_far_from_the_reference(N, S, M, K, low, high, blank):
    """The forward kernel takes its exponentials relative to the first pair of tiles and sums again, from memory, where that
    does not hold: all scores far below or above 0, and scores that rise by 150 to 200 with the neighbour's token number
    (bias rounded to bf16 beforehand; what is left of a large bias is exact in the oracle as well)."""
    print(f"case far scores N={N} low={low} high={high} blank={blank}", flush=True)
    cfg = CONFIGS["mae_pt_s1_1024"].scaled(B=1, N=N, C=64, H=2, K=K, S=S, M=M, dtype="bf16")
    w = make_workload(cfg, blank=blank)
    nbr, near = oracle.knn(w["coords"], None, S, M, K)
    ramp = low + (high - low) * nbr[:, :, None, :] / (N - 1.0)
    w["bias"] = torch.from_numpy((w["bias"] + ramp).astype(np.float32)).bfloat16().float().numpy()
    check_attention(w, nbr, "bf16", 1.0 / np.sqrt(32), near=near, S=S, M=M, blank=blank, use_plan=True)


@pytest.mark.parametrize("K", [15, 16, 17, 32, 46, 47, 48, 50, 56, 59, 60, 61, 62, 63, 64])
@pytest.mark.parametrize("N", [512, 493])
def test_rows_of_every_length(N, K):
    """Row lengths round the edges of the tiled kernels' classes (48, 60 and 64 values; 8, 2 or 1 of them moved at a time),
    and a bias that starts 2, 4 or 8 bytes off: the way its values reach LDS differs, the results may not in any bit."""
    print(f"case rows N={N} K={K}", flush=True)
    S, M = 32, 5
    w = make_workload(CONFIGS["knn_scale"].scaled(B=1, N=N, C=64, H=2, K=K, S=S, M=M, dtype="bf16"), blank=True)
    nbr, near = oracle.knn(w["coords"], None, S, M, K)
    scale = 1.0 / np.sqrt(32)
    check_attention(w, nbr, "bf16", scale, near=near, S=S, M=M, blank=True, use_plan=True)
    q, k, v, dout, bias = (to_dev(w[n], "bf16") for n in ("q", "k", "v", "dout", "bias"))
    nbr, near = (torch.from_numpy(np.ascontiguousarray(x, dtype=np.int32)).cuda() for x in (nbr, near))
    results = []
    for off in (0, 1, 2, 4):
        moved = torch.empty(bias.numel() + 8, dtype=bias.dtype, device="cuda")[off:off + bias.numel()].view(bias.shape)
        moved.copy_(bias)
        out, lse = aff.affmae_pla_fwd(q, k, v, moved, nbr, scale, near, S, M)
        g = aff.affmae_pla_bwd(q, k, v, moved, nbr, out, lse, dout, scale, near, S, M)
        results.append([out, lse] + [g[n] for n in sorted(g) if g[n] is not None])
    for other in results[1:]:
        assert all(torch_equal(a, b) for a, b in zip(results[0], other))


@pytest.mark.parametrize("short", [1, 5, 15])
@pytest.mark.parametrize("K,blank", [(24, False), (37, True), (48, True)])
def test_short_strip_as_a_full_one(short, K, blank):
    """The rows of an image's short last strip have the bits that they have in a full strip: the rows past its end, which have
    no neighbours, do not send it down another path (the second sum, for scores far from 0, rounds differently).  The full
    image's further queries repeat the neighbours of the last real one, so both calls touch the same token tiles."""
    print(f"case short strip by {short} K={K} blank={blank}", flush=True)
    N, S, M, H = 512, 32, 4, 3
    G, Nr = N // S, N - short
    rng = np.random.default_rng(100 * K + short)
    near = np.stack([np.arange(M) + min(max(c - 1, 0), G - M) for c in range(G)]).astype(np.int32)[None]
    nbr = np.empty((1, N, K), np.int32)
    for i in range(N):
        cand = (near[0, i // S][:, None] * S + np.arange(S)).reshape(-1)
        nbr[0, i] = rng.choice(cand[cand < Nr], K, replace=False) if i < Nr else nbr[0, Nr - 1]
    w = make_features(1, N, H, 32, K, "bf16", rng, blank=blank)
    q, k, v, bias = (to_dev(w[n], "bf16") for n in ("q", "k", "v", "bias"))
    kb, vb = (to_dev(w[n], "bf16") if blank else None for n in ("k_blank", "v_blank"))
    nbr, near = (torch.from_numpy(x).cuda() for x in (nbr, near))
    full = aff.affmae_pla_fwd(q, k, v, bias, nbr, 0.2, near, S, M, kb, vb)
    cut = aff.affmae_pla_fwd(*(x[:, :Nr].contiguous() for x in (q, k, v, bias, nbr)), 0.2, near, S, M, kb, vb)
    for a, b in zip(full, cut):
        assert torch.equal(a[:, :Nr], b)


@pytest.mark.parametrize("around", [96.0, -96.0, 3.0])
@pytest.mark.parametrize("N,K", [(512, 48), (505, 37)])
def test_lse_to_half_a_unit(N, K, around):
    """With q = 0 the scores are the bias and exact, so all that lse = log sum exp(bias) can be off by is its own rounding (half
    a unit in the last place) and the errors of the exponentials and of the logarithm: each term 2^-22 relative at most, the
    logarithm one unit of a value below 8 (times ln 2)."""
    print(f"case lse N={N} K={K} around {around}", flush=True)
    S, M = 32, 4
    rng = np.random.default_rng(K)
    nbr, near = oracle.knn(rng.uniform(0, 100, size=(1, N, 2)).astype(np.float32), None, S, M, K)
    w = make_features(1, N, 2, 32, K, "bf16", rng)
    w["q"] = np.zeros_like(w["q"])
    w["bias"] = (around + 0.5 * rng.integers(-4, 5, size=w["bias"].shape)).astype(np.float32)  # (exact in bf16)
    args = [to_dev(w[n], "bf16") for n in ("q", "k", "v", "bias")]
    nbr, near = (torch.from_numpy(np.ascontiguousarray(x, dtype=np.int32)).cuda() for x in (nbr, near))
    _, lse = aff.affmae_pla_fwd(*args, nbr, 0.2, near, S, M)
    b = w["bias"].astype(np.float64)
    exact = b.max(-1) + np.log(np.exp(b - b.max(-1, keepdims=True)).sum(-1))
    err = np.abs(lse.cpu().numpy().astype(np.float64) - exact)
    assert (err <= 0.5 * np.spacing(np.abs(exact).astype(np.float32)) + 2.0 ** -22 + 2.0 ** -21 * np.log(2.0)).all()


def test_largest_probability_is_exact():
    """Two neighbours of values 1 and -1 and exact scores: out = w1 - w2, and an error d of one of the two probabilities changes
    it by 2 w1 w2 d.  Relative to the larger score one of them is 1, and only the other is rounded to bf16 (by 2^-8 at most).
    Half of a strip's queries have no neighbour in its first pair of tiles."""
    print("case largest probability", flush=True)
    N, H, rng = 64, 16, np.random.default_rng(9)
    nbr = np.empty((1, N, 2), np.int32)
    for i in range(N):
        tile = 2 * (i % 16 // 8) + i % 2  # queries 8..15 of a strip: tiles 2 and 3
        nbr[0, i] = 16 * tile + 2 * rng.integers(0, 8) + np.arange(2)
    w = make_features(1, N, H, 32, 2, "bf16", rng)
    q, k = (to_dev(w[n], "bf16") for n in ("q", "k"))
    v = torch.ones_like(q)
    v[:, 1::2] = -1
    bias = torch.from_numpy(rng.uniform(0.25, 1.0, size=(1, N, H, 2)).astype(np.float32)).bfloat16().cuda()
    near = torch.zeros(1, 1, 1, dtype=torch.int32, device="cuda")
    out, _ = aff.affmae_pla_fwd(torch.zeros_like(q), k, v, bias, torch.from_numpy(nbr).cuda(), 0.2, near, N, 1)
    p = bias.double().softmax(-1)
    exact = (p[..., 0] - p[..., 1])[..., None]
    bound = 2.0 ** -8 * (2 * p.prod(-1)[..., None] + exact.abs()) * (1 + 2.0 ** -7) + 2.0 ** -21  # rounding of p, of out; fp32
    assert ((out.double() - exact).abs() <= bound).all()


@pytest.mark.parametrize("N,K", [(512, 48), (505, 21)])
def test_masked_neighbours_and_a_low_blank_score(N, K):
    """A bias of the storage type's lowest value on all neighbours of some queries and on half of those of others, beside a blank
    column of score -200: it takes the whole weight of the former, and none of the latter's."""
    print(f"case masked neighbours N={N} K={K}", flush=True)
    S, M = 32, 4
    rng = np.random.default_rng(N)
    nbr, near = oracle.knn(rng.uniform(0, 100, size=(1, N, 2)).astype(np.float32), None, S, M, K)
    w = make_features(1, N, 2, 32, K, "bf16", rng, blank=True)
    w["q"][..., 0] = 4.0
    w["k_blank"][:] = 0.0
    w["k_blank"][:, 0] = -50.0
    w["k"][..., 0] = 0.0
    lowest = float(torch.finfo(torch.bfloat16).min)
    w["bias"][:, ::3] = lowest
    w["bias"][:, 1::3, :, ::2] = lowest
    out, lse, g = run_gpu_attention(w, nbr, "bf16", 1.0, near, S, M, True, True)
    rout, rlse, rg = run_oracle_attention(w, nbr, 1.0, True)
    assert rel_err(lse, rlse) <= LSE_TOL
    for name, got, ref in [("out", out, rout)] + [(n, g[n], rg[n]) for n in rg if n != "dk_blank"]:
        assert rel_err(got, ref) <= TOL["bf16"], name
    # dk_blank is 0 but for roundings: dS = <dout, v_blank> - <dout, out> with out = v_blank, two fp32 sums of 32 products
    terms = np.abs(w["dout"] * w["v_blank"]).sum(-1) * np.abs(w["q"]).max(-1)
    assert np.abs(g["dk_blank"].cpu().numpy()).max() <= 64 * 2.0 ** -24 * terms.sum(1).max()


@pytest.mark.parametrize("N,K", [(1024, 48), (1001, 24), (1024, 62), (1024, 37)])
def test_slots_that_the_plan_does_not_hold(N, K):
    """Neighbours outside the near clusters break the promise; the tiled kernels leave them out, and their slots of dbias are 0
    (and add nothing to a relative-position table), not what LDS held from the launch before."""
    print(f"case foreign neighbours N={N} K={K}", flush=True)
    S, M, H = 64, 3, 2
    G = -(-N // S)
    rng = np.random.default_rng(K)
    near = np.stack([np.arange(M) + min(max(c - 1, 0), G - M) for c in range(G)]).astype(np.int32)[None]
    nbr = np.empty((1, N, K), np.int32)
    for i in range(N):
        cand = (near[0, i // S][:, None] * S + np.arange(S)).reshape(-1)
        nbr[0, i] = rng.choice(cand[cand < N], K, replace=False)
    foreign = np.zeros((1, N, K), bool)
    foreign[0, ::2, 1::5] = True
    far = np.where(np.arange(N) < N // 2, N - 1 - rng.integers(0, S, size=N) % 32, rng.integers(0, S, size=N))
    broken = np.where(foreign, far[None, :, None], nbr).astype(np.int32)
    w = make_features(1, N, H, 32, K, "bf16", rng)
    q, k, v, dout = (to_dev(w[n], "bf16") for n in ("q", "k", "v", "dout"))
    R, rate = 2, 0.1
    coords = torch.from_numpy(rng.uniform(0, 100, size=(1, N, 2)).astype(np.float32)).cuda()
    table = torch.from_numpy(rng.normal(size=(H, 5, 5)).astype(np.float32)).bfloat16().cuda()
    nbr, broken, near = (torch.from_numpy(x).cuda() for x in (nbr, broken, near))
    diff = coords[0][broken[0].long()] - coords[0][:, None]
    cell = ((diff * rate).round().clamp(-R, R).long() + R)
    cell = cell[..., 1] * 5 + cell[..., 0]
    bias = table.reshape(H, 25)[:, cell].permute(1, 0, 2)[None].contiguous()
    foreign = torch.from_numpy(foreign).cuda()[:, :, None].expand(1, N, H, K)

    def run(n):
        out, lse = aff.affmae_pla_fwd(q, k, v, bias, n, 0.2, near, S, M)
        return aff.affmae_pla_bwd(q, k, v, bias, n, out, lse, dout, 0.2, near, S, M)["dbias"]

    run(nbr)
    dbias = run(broken)
    assert (dbias[foreign] == 0).all() and (dbias[~foreign] != 0).float().mean() > 0.9
    if K % 8 == 0:
        out, lse = aff.affmae_pla_fwd_relpos(q, k, v, coords, table, broken, 0.2, rate, near, S, M)
        got = aff.affmae_pla_bwd_relpos(q, k, v, coords, table, broken, out, lse, dout, 0.2, rate, near, S, M)["drel_table"]
        sums = torch.zeros(H, 25, dtype=torch.float64, device="cuda")
        for h in range(H):
            sums[h].index_add_(0, cell.reshape(-1), dbias[0, :, h].double().reshape(-1))
        # the same bf16 values of dS, added up in fp64 and rounded to fp32 per workgroup
        assert (got.double().view(H, 25) - sums).abs().max() <= 2.0 ** -20 * dbias.double().abs().sum()


@pytest.mark.parametrize("B,N,K,S,M", [(2, 1000, 1, 64, 16), (2, 1000, 3, 64, 16), (3, 70, 24, 64, 2), (5, 10, 8, 64, 1),
                                       (2, 130, 33, 48, 3)])
def test_plans_with_room_for_less_than_the_near_clusters(B, N, K, S, M):
    """A plan has room for as many token tiles a strip as it has neighbours, or as the image has, where its near clusters hold
    more: neighbours drawn from all of them, so that the room is used up."""
    print(f"case plan room B={B} N={N} K={K} S={S} M={M}", flush=True)
    rng = np.random.default_rng(N + K)
    G = -(-N // S)
    near = np.stack([np.stack([rng.choice(G, M, replace=False) for _ in range(G)]) for _ in range(B)]).astype(np.int32)
    nbr = np.empty((B, N, K), np.int32)
    for b in range(B):
        for i in range(N):
            cand = (near[b, i // S][:, None] * S + np.arange(S)).reshape(-1)
            nbr[b, i] = rng.choice(cand[cand < N], K, replace=False)
    w = make_features(B, N, 2, 32, K, "bf16", rng, blank=True)
    check_attention(w, nbr, "bf16", 0.2, near=near, S=S, M=M, blank=True, use_plan=True)


@pytest.mark.parametrize("N", [57344, 57349, 57327])
@pytest.mark.parametrize("K,S,M", [(13, 64, 16), (3, 16, 1)])
def test_plans_on_both_sides_of_the_tile_table(N, K, S, M):
    """Images of 3584 token tiles, the most whose tiles the plan kernel looks up in LDS, of one more, and with a short last tile:
    as many candidate tiles as there may be, in distant clusters, and one; lists that are no multiple of a query's four lanes."""
    print(f"case tile table N={N} K={K} S={S} M={M}", flush=True)
    rng = np.random.default_rng(N + K)
    G = -(-N // S)
    own = np.arange(G)
    near = np.stack([own] + [(own + 1 + i * (G // M)) % G for i in range(M - 1)], axis=1).astype(np.int32)
    near = rng.permuted(near, axis=1)
    cand = (near[:, :, None] * S + np.arange(S)).reshape(G, M * S)
    pick = np.argsort(rng.random((N, M * S), dtype=np.float32) + 2.0 * (cand[np.arange(N) // S] >= N), axis=1)[:, :K]
    nbr = np.take_along_axis(cand[np.arange(N) // S], pick, axis=1).astype(np.int32)[None]
    w = make_features(1, N, 1, 32, K, "bf16", rng)
    check_attention(w, nbr, "bf16", 0.2, near=near[None], S=S, M=M, use_plan=True)


@pytest.mark.parametrize("dtype,d", [("f32", 16), ("f32", 32), ("f32", 64), ("bf16", 16), ("bf16", 64)])
@pytest.mark.parametrize("B,N,H,K,S,M,blank", [  # (448 to 512 workgroups: all but the smallest K by the kernels in question)
    (16, 1024, 2, 48, 64, 8, False),
    (10, 1000, 3, 37, 64, 8, True),   # a short last strip and token tile, odd K and H
    (64, 512, 1, 64, 16, 32, True),   # the longest rows; unions of many stages
    (120, 90, 2, 17, 48, 2, False),   # a group of two strips, the last one short; the fewest neighbours that fp32 d = 32 takes
    (7, 4099, 1, 24, 32, 6, True),
    (3, 2064, 5, 33, 64, 5, False),   # the last group of one strip
    (7, 2051, 2, 3, 64, 2, True),     # the shortest rows (d = 16)
    (7, 2051, 2, 9, 64, 2, True),     # ... (bf16 d = 64)
    (7, 2051, 2, 16, 64, 3, True),    # ... (fp32 d = 64)
    # and where some of the types are served by the gather kernels
    (8, 1024, 2, 48, 64, 8, False),
    (6, 1000, 3, 37, 64, 8, True),    # a short last strip and token tile, odd K and H
    (32, 512, 1, 64, 16, 32, True),   # the longest rows; unions of many stages
    (64, 90, 2, 16, 48, 2, False),    # a group of two strips, the last one short
    (4, 4099, 1, 24, 32, 6, True),
    (2, 2064, 5, 33, 64, 5, False),   # the last group of one strip
    (2, 2051, 4, 1, 64, 2, True),     # K = 1 (the gather kernels)
    (2, 2051, 4, 16, 64, 3, True),
])
def test_plans_for_other_types_and_heads(dtype, d, B, N, H, K, S, M, blank):
    """fp32 storage, and bf16 with head sizes other than 32, on a plan: products on fp32 operands.  The bar of the gather
    kernels (1e-5 and 2e-2 of the largest value), and scores spread so widely that the reference has to move."""
    print(f"case wide {dtype} d={d} B={B} N={N} H={H} K={K} S={S} M={M} blank={blank}", flush=True)
    cfg = CONFIGS["knn_scale" if N % 16 else "mae_pt_s1_1024"].scaled(B=B, N=N, C=H * d, H=H, K=K, S=S, M=M, dtype=dtype)
    w = make_workload(cfg, blank=blank)
    nbr, near = oracle.knn(w["coords"], None, S, M, K)
    run = lambda: check_attention(w, nbr, dtype, 1.0 / np.sqrt(d), near=near, S=S, M=M, blank=blank, use_plan=True)
    kernels = kernels_of(run)[1]
    if 448 <= B * -(-N // 64) * H <= 512:
        wide = K >= {("f32", 16): 3, ("f32", 32): 17, ("f32", 64): 16, ("bf16", 16): 3, ("bf16", 64): 9}[dtype, d]
        assert ("pla_fwd_wide_kernel" in kernels, "pla_bwd_wide_key_kernel" in kernels) == (wide, wide), kernels
    # logits with a standard deviation of 8: scores below 64, whose products and sum round to 2^-19 a few times over, as does lse, so
    # that p = exp(s - lse) is off by up to 1e-5; p (dP - D) and its sums over terms of both signs by a few times that
    check_attention(w, nbr, dtype, 8.0 / np.sqrt(d), near=near, S=S, M=M, blank=blank, use_plan=True, tol=4e-5 if dtype == "f32" else None)


@pytest.mark.parametrize("dtype,d,B,N,H,K,blank,wide", [
    ("bf16", 16, 16, 1024, 4, 2, False, False),   # rows of p would not fit the workspace of the gather kernels
    ("bf16", 16, 16, 1024, 4, 3, False, True),
    ("bf16", 64, 16, 1024, 4, 9, False, True),
    ("bf16", 64, 64, 17, 8, 9, False, False),     # ... nor here, where the strips are half empty
    ("f32", 16, 16, 1024, 8, 3, True, False),     # ... nor beside the parts of the blank gradients
    ("f32", 16, 16, 1024, 8, 5, True, True),
    ("f32", 64, 16, 1024, 4, 24, True, True),
    ("f32", 32, 1, 1024, 4, 24, False, False),    # too few workgroups
    ("f32", 32, 16, 1024, 2, 17, False, True),    # 512 workgroups: a full round
    ("f32", 32, 16, 1024, 2, 16, False, False),
    ("f32", 32, 9, 1024, 4, 64, False, False),    # 576: little of a second one
    ("f32", 32, 12, 1024, 4, 48, False, True),    # 768: half of it
    ("f32", 32, 12, 1024, 4, 47, False, False),
    ("f32", 16, 9, 1024, 4, 24, False, False),
    ("f32", 16, 9, 1024, 4, 15, False, True),
    ("f32", 64, 9, 1024, 4, 48, False, True),
    ("f32", 64, 9, 1024, 4, 47, False, False),
    ("bf16", 64, 12, 1024, 4, 16, False, False),
    ("bf16", 64, 12, 1024, 4, 17, False, True),
    ("bf16", 64, 16, 1024, 4, 8, False, False),
    ("bf16", 16, 4, 1024, 4, 3, False, True),     # 256
])
def test_forward_and_backward_take_the_same_way(dtype, d, B, N, H, K, blank, wide):
    """fp32 storage and head sizes other than 32 on a plan: the kernels with products on fp32 operands serve both directions or none."""
    print(f"case ways {dtype} d={d} B={B} N={N} H={H} K={K} blank={blank}", flush=True)
    S, rng = 16 if N < 64 else 64, np.random.default_rng(K)
    M = min(-(-N // S), 4)
    w = make_features(B, N, H, d, K, dtype, rng, blank=blank)
    nbr, near = oracle.knn(rng.uniform(0, 100, size=(B, N, 2)).astype(np.float32), None, S, M, K)
    run = lambda: check_attention(w, nbr, dtype, 1.0 / np.sqrt(d), near=near, S=S, M=M, blank=blank, use_plan=True)
    _, kernels = kernels_of(run)
    assert ("pla_fwd_wide_kernel" in kernels, "pla_bwd_wide_key_kernel" in kernels) == (wide, wide), kernels


@pytest.mark.parametrize("dtype,d,K", [("bf16", 16, 24), ("bf16", 64, 37), ("f32", 16, 37), ("f32", 64, 48)])
def test_slots_that_the_plan_does_not_hold_in_fp32_products(dtype, d, K):
    """As test_slots_that_the_plan_does_not_hold, for the kernels with products on fp32 operands: dbias of such a slot is 0
    whatever the bias there is."""
    print(f"case foreign neighbours {dtype} d={d} K={K}", flush=True)
    B, N, H, S, M = 16, 1024, 4, 64, 3
    G = N // S
    rng = np.random.default_rng(K + d)
    near = np.stack([np.arange(M) + min(max(c - 1, 0), G - M) for c in range(G)]).astype(np.int32)
    cand = (near[:, :, None] * S + np.arange(S)).reshape(G, M * S)[np.arange(N) // S]
    nbr = np.take_along_axis(cand, np.argsort(rng.random((N, M * S)), axis=1)[:, :K], axis=1)
    foreign = np.zeros((N, K), bool)
    foreign[::2, 1::5] = True
    nbr = np.where(foreign, np.where(np.arange(N) < N // 2, N - 1, 0)[:, None], nbr).astype(np.int32)
    w = make_features(B, N, H, d, K, dtype, rng)
    q, k, v, dout, bias = (to_dev(w[n], dtype) for n in ("q", "k", "v", "dout", "bias"))
    nbr_d, near_d = (torch.from_numpy(np.broadcast_to(x, (B, *x.shape)).copy()).cuda() for x in (nbr, near))
    plan = aff.affmae_pla_plan(nbr_d, near_d, S, M)
    scale = 1.0 / np.sqrt(d)

    def run():
        out, lse = aff.affmae_pla_fwd(q, k, v, bias, nbr_d, scale, near_d, S, M, plan=plan)
        return aff.affmae_pla_bwd(q, k, v, bias, nbr_d, out, lse, dout, scale, near_d, S, M, plan=plan)["dbias"]

    dbias, kernels = kernels_of(run)
    assert "pla_bwd_wide_query_kernel" in kernels
    f = torch.from_numpy(foreign).cuda()[None, :, None].expand(B, N, H, K)
    assert (bias[f] != 0).float().mean() > 0.9
    assert (dbias[f] == 0).all() and (dbias[~f] != 0).float().mean() > 0.9


WIDE_TYPES = [("f32", 16), ("f32", 32), ("f32", 64), ("bf16", 16), ("bf16", 64)]


@pytest.mark.parametrize("dtype,d", WIDE_TYPES)
@pytest.mark.parametrize("strips", [64, 65, 128, 129])
def test_popular_groups_of_tiles_in_fp32_products(dtype, d, strips):
    """As test_popular_groups_of_tiles: the key side walks a group's list in parts of 64 strips, two buffers in turn."""
    print(f"case popular groups {dtype} d={d} strips={strips}", flush=True)
    B, N, H, K, S, M = 7, 4096, 1, 20, 64, 5
    G = N // S
    rng = np.random.default_rng(strips + d)
    near = np.stack([np.arange(M) + min(max(c - 1, 0), G - M) for c in range(G)]).astype(np.int32)
    own = int((near == 0).any(axis=1).sum()) * S // 16  # strips around the first cluster
    far = strips - own
    first = 8
    near[first : first + -(-far * 16 // S), M - 1] = 0
    cand = (near[:, :, None] * S + np.arange(S)).reshape(G, M * S)
    score = rng.random((N, M * S))
    named = np.zeros(N, bool)
    named[first * S : first * S + far * 16] = True
    score[~named & (np.arange(N) >= first * S), (M - 1) * S :] += 2.0  # (the rest of the last cluster: no neighbour there)
    nbr = np.take_along_axis(cand[np.arange(N) // S], np.argsort(score, axis=1)[:, :K], axis=1).astype(np.int32)
    assert (nbr.reshape(N // 16, -1) < S).any(axis=1).sum() == strips
    w = make_features(B, N, H, d, K, dtype, rng)
    many = lambda t: np.repeat(t[None], B, axis=0)
    run = lambda: check_attention(w, many(nbr), dtype, 1.0 / np.sqrt(d), near=many(near), S=S, M=M, use_plan=True)
    assert "pla_bwd_wide_key_kernel" in kernels_of(run)[1]


@pytest.mark.parametrize("dtype,d", WIDE_TYPES)
@pytest.mark.parametrize("M", [15, 16, 17, 20])
def test_unions_of_many_tiles_in_fp32_products(dtype, d, M):
    """Strips of a group with no tile in common: unions of 60, 64, 68 and 80 tiles, whose numbers are fetched 64 at a time."""
    print(f"case unions {dtype} d={d} M={M}", flush=True)
    B, N, H, K, S = 4, 4096, 2, 48, 16
    G = N // S
    rng = np.random.default_rng(M + d)
    c = np.arange(G)[:, None]
    near = ((c % 4) * (G // 4) + (c // 4 + np.arange(M)) % (G // 4)).astype(np.int32)
    cand = (near[:, :, None] * S + np.arange(S)).reshape(G, M * S)
    nbr = np.take_along_axis(cand[np.arange(N) // S], np.argsort(rng.random((N, M * S)), axis=1)[:, :K], axis=1).astype(np.int32)
    assert len(np.unique(nbr[:64] // 16)) == 4 * M
    w = make_features(B, N, H, d, K, dtype, rng, blank=True)
    many = lambda t: np.repeat(t[None], B, axis=0)
    run = lambda: check_attention(w, many(nbr), dtype, 1.0 / np.sqrt(d), near=many(near), S=S, M=M, blank=True, use_plan=True)
    assert "pla_bwd_wide_query_kernel" in kernels_of(run)[1]


def test_exponential_of_the_fp32_products():
    """The exponential over its range: without queries the scores are the bias, and with unit vectors as values the outputs are exp(bias)
    over their sum.  The exponential rounds its argument's fraction once (half a unit at 1/2: 2^-26 ln 2 of the result), 2^fraction to one unit
    (2^-23 at most), the sum and the quotient to half of one each: below 3 2^-23 altogether, and exactly 0 from -104 on."""
    B, N, H, d, K, S, M = 7, 4096, 1, 32, 32, 64, 1
    rng = np.random.default_rng(5)
    x = np.where(rng.random((B, N, H, K)) < 0.05, rng.uniform(-400, -104, size=(B, N, H, K)), -(rng.random((B, N, H, K)) ** 3) * 80.0)
    x = x.astype(np.float32)
    x[..., 0] = 0.0
    nbr = (np.arange(N)[:, None] // S * S + np.arange(K)).astype(np.int32)
    near = (np.arange(N // S)[:, None]).astype(np.int32)
    v = np.zeros((B, N, H, d), np.float32)
    v[:, np.arange(N), 0, np.arange(N) % d] = 1.0
    up = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    q, k, v, bias = up(np.zeros((B, N, H, d), np.float32)), up(rng.normal(size=(B, N, H, d)).astype(np.float32)), up(v), up(x)
    nbr_d, near_d = (up(np.repeat(t[None], B, axis=0)) for t in (nbr, near))
    plan = aff.affmae_pla_plan(nbr_d, near_d, S, M)
    (out, _), kernels = kernels_of(lambda: aff.affmae_pla_fwd(q, k, v, bias, nbr_d, 0.25, near_d, S, M, plan=plan))
    assert "pla_fwd_wide_kernel" in kernels
    e = np.exp(x.astype(np.float64))
    ref = e / e.sum(axis=-1, keepdims=True)
    got = out.cpu().numpy().astype(np.float64)
    assert np.all(got[x < -104.0] == 0.0) and (x < -104.0).sum() > 10000
    some = x > -87.0 + np.log(32.0)  # (normal results)
    assert np.abs(got[some] / ref[some] - 1.0).max() <= 3 * 2.0 ** -23
