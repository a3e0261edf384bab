"""GPU parity of gl_knn_graph and gl_pool_keys against the CPU oracle."""
import zlib

import numpy as np
import pytest
import torch

import oracle as O
from gpu_helpers import check_close, check_idx, from_dev, require_gpu, to_dev
from paper_2604_21290_amd import inputs as I

pytestmark = pytest.mark.gpu


def _say(*a):
    print("[gpu-test]", *a, flush=True)


def _knn_case(x: I.Stored, k, d, keys: I.Stored | None = None, rows=None, label=""):
    from paper_2604_21290_amd import api
    xd = to_dev(x)
    kd = to_dev(keys) if keys is not None else None
    _say("knn", label, tuple(x.shape), "M", None if keys is None else keys.shape[1], "k", k, "d", d)
    idx = api.knn_graph(xd, k, d, keys=kd)
    torch.cuda.synchronize()
    D = O.knn_distances(x.value, None if keys is None else keys.value, rows=rows)
    return check_idx(idx.cpu().numpy(), D, k, d, rows=rows, label=label)


# -- the workloads at full size (sampled rows where N = 3136) -----------------
@pytest.mark.parametrize("name", ["single", "vig_ti", "vig_b", "hires", "vig_ti_448", "vig_s",
                                  "pyr_s3", "pyr_s4"])
def test_knn_workload_full(name):
    require_gpu()
    from paper_2604_21290_amd import api
    w = I.WORKLOADS[name]
    x = I.make_features(w)
    rows = None
    if w.N > 500:
        rows = np.sort(np.random.default_rng(99).choice(w.N, 384, replace=False))
    xd = to_dev(x)
    D = O.knn_distances(x.value, rows=rows)
    for d in sorted(set(w.dilations)):
        _say("knn", name, "d", d)
        idx = api.knn_graph(xd, w.k, d)
        torch.cuda.synchronize()
        st = check_idx(idx.cpu().numpy(), D, w.k, d, rows=rows, label=f"{name} d={d}")
        _say(name, "d", d, st)


@pytest.mark.parametrize("name", ["pyr_s1", "pyr_s2"])
def test_knn_pooled_workload_full(name):
    """Pooled keys: the pool is checked against the oracle pool, and the graph
    against the oracle evaluated on the GPU's stored keys (teacher forcing)."""
    require_gpu()
    from paper_2604_21290_amd import api
    w = I.WORKLOADS[name]
    x = I.make_features(w)
    xd = to_dev(x)
    _say("pool", name)
    keys = api.pool_keys(xd, w.H, w.W, w.pool_r)
    torch.cuda.synchronize()
    ks = from_dev(keys)
    check_close(ks.value, O.pool_keys_ref(x.value, w.H, w.W, w.pool_r), w.dtype, f"pool {name}")
    rows = np.sort(np.random.default_rng(98).choice(w.N, min(w.N, 512), replace=False))
    idx = api.knn_graph(xd, w.k, w.dilations[0], keys=keys)
    torch.cuda.synchronize()
    D = O.knn_distances(x.value, ks.value, rows=rows)
    _say(name, check_idx(idx.cpu().numpy(), D, w.k, w.dilations[0], rows=rows, label=name))


# -- edge cases -------------------------------------------------------------------
EDGE = [
    # label, B, N, M (None = keys are x), C, k, d, dtype, features
    ("ragged_rows_k1", 2, 37, None, 8, 1, 1, I.BF16, "unit"),
    ("k_equals_M_fp32", 1, 5, None, 4, 5, 1, I.F32, "unit"),
    ("k_equals_M_bf16", 1, 16, None, 16, 16, 1, I.BF16, "unit"),
    ("pooled_like_small_M", 2, 50, 13, 16, 4, 3, I.BF16, "unit"),
    ("chunk_boundary_257_maxKK", 1, 70, 257, 32, 16, 4, I.BF16, "unit"),
    ("three_chunks", 2, 100, 600, 24, 9, 2, I.BF16, "normal"),
    ("max_M_4096", 1, 48, 4096, 16, 16, 4, I.BF16, "unit"),
    ("max_M_fp32", 1, 33, 4096, 8, 8, 8, I.F32, "unit"),
    ("C_tail_bf16", 2, 60, None, 40, 9, 1, I.BF16, "unit"),
    ("C_tail_fp32", 2, 60, None, 12, 9, 3, I.F32, "unit"),
    ("wide_C_bf16", 1, 40, None, 1024, 9, 4, I.BF16, "unit"),
    ("unnormalised_fp32", 3, 196, None, 192, 9, 2, I.F32, "normal"),
    ("KK_33_R4", 1, 196, None, 64, 11, 3, I.BF16, "normal"),
    # more than 256 keys on small grids (up to 512 tiles of 16 rows in any width): the
    # in-register kernel in chunks of 256 keys, the last one ragged; the widest
    # rows that larger grids stream; fp32
    ("small_grid_M333", 2, 90, 333, 96, 16, 2, I.BF16, "normal"),
    ("small_grid_C768_bf16", 1, 70, 300, 768, 9, 1, I.BF16, "unit"),
    ("small_grid_C384_fp32", 1, 70, 300, 384, 9, 2, I.F32, "normal"),
    ("small_grid_C160_R4", 2, 64, 784, 160, 16, 4, I.BF16, "unit"),
    ("small_grid_fp32_C96", 1, 130, 3136, 96, 16, 2, I.F32, "normal"),
    # streamed, more than 256 workgroups of 128 rows: the four-wave form of the
    # narrow rows
    ("stream_four_waves_B33", 33, 1000, 400, 64, 9, 2, I.BF16, "normal"),
    # LDS-staged wide kernel (bf16, C >= 256, M <= 256): key-row buckets 64 / 128 /
    # 224 / 256, a partial last stage (C = 520), K' = 64, one query row
    ("wide_M64_bucket", 2, 50, 64, 512, 9, 2, I.BF16, "unit"),
    ("wide_M65_C520_KK64", 1, 33, 65, 520, 16, 4, I.BF16, "normal"),
    ("wide_M200_ragged", 3, 97, 200, 512, 9, 3, I.BF16, "unit"),
    ("wide_M256_max", 1, 70, 256, 640, 16, 2, I.BF16, "unit"),
    ("wide_self_unnormalised", 2, 196, None, 640, 9, 1, I.BF16, "normal"),
    ("wide_N1", 2, 1, 30, 512, 3, 1, I.BF16, "unit"),
    ("wide_C264_partial", 2, 45, 100, 264, 9, 2, I.BF16, "normal"),
]


@pytest.mark.parametrize("case", EDGE, ids=[c[0] for c in EDGE])
def test_knn_edges(case):
    require_gpu()
    label, B, N, M, C, k, d, dt, feat = case
    seed = zlib.crc32(label.encode()) % 10000
    x = I.random_features(seed, B, N, C, dt, unit=(feat == "unit"))
    keys = None if M is None else I.random_features(seed + 1, B, M, C, dt, unit=(feat == "unit"))
    _say(label, _knn_case(x, k, d, keys, label=label))


# Keys resident in LDS, 64 query rows per workgroup (bf16, M <= 256, 32 < C <=
# 160, at least 384 workgroups): every key-tile bucket (4 / 8 / 13 / 16 tiles),
# two to five contraction steps' worth of channels with partial last steps,
# both norm orders (below and from C = 128), K' up to 64, ragged last row
# tiles.  Sampled rows keep the oracle fast.
RESIDENT = [
    # label, B, N, M, C, k, d
    ("res_pyr_like_ragged", 16, 2049, 196, 80, 9, 1),
    ("res_C40_M100_KK18", 32, 1000, 100, 40, 9, 2),
    ("res_C128_M256_KK64", 8, 4100, 256, 128, 16, 4),
    ("res_C72_M64", 16, 2048, 64, 72, 9, 3),
    ("res_C56_M209", 16, 2048, 209, 56, 9, 1),
    ("res_C96_M17_k1", 16, 2047, 17, 96, 1, 1),
    ("res_C128_wide_order", 16, 1600, 196, 128, 9, 1),
    ("res_C136_M150_KK18", 32, 800, 150, 136, 9, 2),
    ("res_C160_M256_KK64", 8, 3100, 256, 160, 16, 4),
    # 8-wave workgroups of 128 rows (at most 256 of them), a 12-row last tile
    ("res_8_waves_tail12", 2, 12300, 200, 64, 9, 2),
]


@pytest.mark.parametrize("case", RESIDENT, ids=[c[0] for c in RESIDENT])
def test_knn_resident(case):
    require_gpu()
    label, B, N, M, C, k, d = case
    seed = zlib.crc32(label.encode()) % 10000
    x = I.random_features(seed, B, N, C, I.BF16, unit=False)
    keys = I.random_features(seed + 1, B, M, C, I.BF16, unit=False)
    rows = np.sort(np.random.default_rng(seed).choice(N, 256, replace=False))
    _say(label, _knn_case(x, k, d, keys, rows=rows, label=label))


def test_knn_resident_duplicates_and_zero_rows():
    """Zero query rows, zero key rows and duplicated key rows on the
    resident-key kernel: ties resolve to the lower key index."""
    require_gpu()
    g = np.random.default_rng(11)
    B, N, M, C = 8, 4096, 150, 64
    a = g.standard_normal((B, N, C))
    kv = g.standard_normal((B, M, C))
    a[:, ::7] = 0.0
    kv[:, 10] = 0.0
    kv[:, 20:40] = kv[:, 0:20]
    x = I.store(a, I.BF16)
    keys = I.store(kv, I.BF16)
    rows = np.sort(np.concatenate([np.arange(0, 70, 7), g.choice(N, 246, replace=False)]))
    rows = np.unique(rows)
    for d in (1, 3):
        _say("resident dup/zero", _knn_case(x, 9, d, keys, rows=rows, label=f"res dup d={d}"))


@pytest.mark.parametrize("C", [32, 512])
def test_knn_duplicates_and_zero_rows(C):
    require_gpu()
    g = np.random.default_rng(5)
    a = g.standard_normal((2, 64, C))
    a[:, 40] = a[:, 3]          # exact duplicate: row 40's nearest must be 3
    a[:, 50] = a[:, 3]
    a[:, 10] = 0.0              # zero rows
    a[:, 20] = 0.0
    for dt in (I.BF16, I.F32):
        x = I.store(a, dt)
        st = _knn_case(x, 6, 1, label=f"dups {dt}")
        from paper_2604_21290_amd import api
        idx = api.knn_graph(to_dev(x), 6, 1).cpu().numpy()
        assert (idx[:, 40, :3] == [3, 40, 50]).all() and (idx[:, 3, :3] == [3, 40, 50]).all()
        assert set(idx[0, 10, :2]) == {10, 20}
        _say("dups", dt, st)


def test_knn_clustered_mixture_small():
    require_gpu()
    w = I.Workload("mix", 2, 20, 20, 32, 16, (2,), I.BF16, seed=77, features="mixture")
    x = I.make_features(w)
    _say(_knn_case(x, 16, 2, label="mixture 20x20"))


def test_knn_deterministic():
    require_gpu()
    from paper_2604_21290_amd import api
    x = to_dev(I.make_features(I.with_batch(I.WORKLOADS["hires"], 2)))
    a = api.knn_graph(x, 16, 2)
    b = api.knn_graph(x, 16, 2)
    torch.cuda.synchronize()
    assert torch.equal(a, b)


def test_pool_edges():
    require_gpu()
    from paper_2604_21290_amd import api
    # windows of r = 2 and 4 take the kernels that issue the whole window at
    # once (both storage types); r = 1 and 3 take the loop
    for (B, H, W, C, r, dt) in [(2, 8, 12, 16, 4, I.BF16), (1, 6, 6, 8, 3, I.F32),
                                (3, 10, 10, 24, 1, I.BF16), (1, 28, 28, 160, 2, I.F32),
                                (2, 8, 16, 12, 4, I.F32), (3, 6, 10, 40, 2, I.BF16)]:
        x = I.random_features(H * W + C, B, H * W, C, dt, unit=False)
        _say("pool", B, H, W, C, r, dt)
        k = api.pool_keys(to_dev(x), H, W, r)
        torch.cuda.synchronize()
        got = from_dev(k).value
        check_close(got, O.pool_keys_ref(x.value, H, W, r), dt, "pool edge")
        if r == 1:
            assert np.array_equal(got, x.value)


# -- the streamed kernel --------------------------------------------------------------
def _streams(B, N):
    """Whether builds against more than 256 keys are streamed on this grid: past
    1024 tiles of 16 rows all are, up to 512 none (up to 256 streamed workgroups)."""
    tiles = B * ((N + 15) // 16)
    assert tiles > 1024 or tiles <= 512
    return tiles > 1024


STREAM = [
    # label, B, N, M, C, k, d, dtype: key counts one past and far from a chunk's
    # edge and the most of them, every number of contraction steps of either type
    # (C padded up to 2, 3, 4, 6, 8, 12, 16, 20 or 24), each list length
    ("M257_KK64", 17, 970, 257, 32, 16, 4, I.BF16),
    ("ragged_M333", 12, 1390, 333, 96, 16, 2, I.BF16),
    ("max_M_KK64", 11, 1500, 4096, 16, 16, 4, I.BF16),
    ("max_M_fp32", 11, 1500, 4096, 8, 8, 8, I.F32),
    ("C160_KK64", 33, 510, 784, 160, 16, 4, I.BF16),
    ("fp32_C96_M3136", 17, 970, 3136, 96, 16, 2, I.F32),
    ("C104", 33, 500, 300, 104, 9, 1, I.BF16),
    ("C256", 33, 500, 300, 256, 9, 2, I.BF16),
    ("C384", 33, 500, 300, 384, 9, 4, I.BF16),
    ("C488", 33, 500, 280, 488, 9, 1, I.BF16),
    ("C640", 33, 500, 260, 640, 16, 2, I.BF16),
    ("C768", 33, 500, 300, 768, 9, 1, I.BF16),
    ("fp32_C36", 33, 500, 300, 36, 9, 1, I.F32),
    ("fp32_C64", 33, 500, 300, 64, 9, 4, I.F32),
    ("fp32_C128", 33, 500, 300, 128, 9, 1, I.F32),
    ("fp32_C192", 33, 500, 300, 192, 9, 2, I.F32),
    ("fp32_C252", 33, 500, 300, 252, 9, 1, I.F32),
    ("fp32_C320", 33, 500, 300, 320, 9, 4, I.F32),
    ("fp32_C384", 33, 500, 300, 384, 9, 2, I.F32),
]


@pytest.mark.parametrize("case", STREAM, ids=[c[0] for c in STREAM])
def test_knn_streamed(case):
    """Other keys than queries, on grids past 1024 tiles of 16 rows."""
    require_gpu()
    from paper_2604_21290_amd import api
    label, B, N, M, C, k, d, dt = case
    assert _streams(B, N) and M > 256, label
    seed = zlib.crc32(label.encode()) % 10000
    x = I.random_features(seed, B, N, C, dt, unit=False)
    keys = I.random_features(seed + 1, B, M, C, dt, unit=False)
    _say("streamed", label)
    idx = api.knn_graph(to_dev(x), k, d, keys=to_dev(keys)).cpu().numpy()
    rows = np.unique(np.linspace(0, N - 1, 48).astype(int))
    for b in (0, B // 2, B - 1):
        D = O.knn_distances(x.value[b:b + 1], keys.value[b:b + 1], rows=rows)
        check_idx(idx[b:b + 1], D, k, d, rows=rows, label=f"{label} image {b}")


@pytest.mark.parametrize("B,N,C,dt", [(17, 970, 64, I.BF16), (17, 970, 200, I.F32), (1, 970, 64, I.BF16)])
def test_knn_many_keys_duplicates_and_zero_rows(B, N, C, dt):
    """Zero query and key rows and duplicated keys among more than 256, streamed
    and in-register: ties go to the lower index."""
    require_gpu()
    g = np.random.default_rng(17)
    a = g.standard_normal((B, N, C))
    kv = g.standard_normal((B, 333, C))
    a[:, ::7] = 0.0
    kv[:, 10] = 0.0
    kv[:, 300:320] = kv[:, 0:20]
    rows = np.unique(np.concatenate([np.arange(0, 70, 7), g.choice(N, 60, replace=False)]))
    for d in (1, 3):
        _say("many keys dup/zero", B, N, C, dt, d,
             _knn_case(I.store(a, dt), 9, d, I.store(kv, dt), rows=rows, label=f"dup d={d}"))


# -- one lane's keys nearest ---------------------------------------------------------
ONE_LANE = [
    # label, B, N, M, C, k, d, dtype: the kernel that builds the graph
    ("tile_r1_fp32", 1, 40, 196, 36, 9, 1, I.F32),
    ("tile_r2", 1, 40, 256, 80, 9, 2, I.BF16),
    ("tile_r4_fp32", 2, 17, 196, 64, 12, 3, I.F32),
    ("wide_r1", 2, 50, 196, 192, 9, 1, I.BF16),
    ("wide_r1_k16", 1, 33, 250, 136, 16, 1, I.BF16),
    ("wide_r2", 2, 50, 196, 192, 9, 3, I.BF16),
    ("wide_r4", 1, 50, 224, 320, 16, 4, I.BF16),
    ("wide_few_keys", 2, 50, 49, 192, 9, 1, I.BF16),
    ("resident_r1", 8, 3136, 196, 80, 9, 1, I.BF16),
    ("resident_r2", 8, 3136, 208, 64, 9, 2, I.BF16),
    ("resident_r4_16_tiles", 8, 3136, 256, 40, 16, 4, I.BF16),
    ("tile_r1_three_chunks", 1, 130, 700, 96, 9, 1, I.BF16),
    ("tile_r4_fp32_three_chunks", 1, 65, 520, 52, 12, 4, I.F32),
    ("stream_r1", 17, 970, 700, 96, 9, 1, I.BF16),
    ("stream_r2", 17, 970, 600, 200, 9, 3, I.BF16),
    ("stream_r4_fp32", 17, 970, 520, 52, 12, 4, I.F32),
]


@pytest.mark.parametrize("case", ONE_LANE, ids=[c[0] for c in ONE_LANE])
def test_nearest_keys_in_one_lane(case):
    """The selection keeps a lane's few smallest candidates in order and looks at
    its others only when those may not do.  Here the nearest keys of every row
    are those of one lane (indices 5, 21, 37, ...), at angles far enough apart
    to rank the same in any precision."""
    require_gpu()
    from paper_2604_21290_amd import api
    label, B, N, M, C, k, d, dt = case
    if M > 256:
        assert _streams(B, N) == label.startswith("stream"), label
    g = np.random.default_rng(M + C)
    u = g.standard_normal(C)
    u /= np.linalg.norm(u)
    keys = g.standard_normal((M, C))
    keys -= (keys @ u)[:, None] * u          # everything else at right angles to u
    keys /= np.linalg.norm(keys, axis=1, keepdims=True)
    lane = np.arange(5, M, 16)
    ang = g.permutation(0.1 + 1.2 * np.arange(len(lane)) / len(lane))
    keys[lane] = np.cos(ang)[:, None] * u + np.sin(ang)[:, None] * keys[lane]
    x = u + 0.02 * g.standard_normal((B, N, C)) / np.sqrt(C)
    xs, ks = I.store(x, dt), I.store(np.broadcast_to(keys, (B, M, C)).copy(), dt)
    print("[gpu-test] one lane", label, flush=True)
    idx = api.knn_graph(to_dev(xs), k, d, keys=to_dev(ks))
    torch.cuda.synchronize()
    rows = np.unique(np.linspace(0, N - 1, 40).astype(int))
    got = idx.cpu().numpy()
    check_idx(got, O.knn_distances(xs.value, ks.value, rows=rows), k, d, rows=rows, label=label)
    near = min(len(lane), k * d)
    assert (got[:, :, :(near + d - 1) // d] % 16 == 5).all(), label


# -- large key sets: the streamed kernel and, on small grids, the in-register one ------
TWO_KERNELS = [
    # label, B, N, C, k, d, dtype; B images are streamed, one is not
    ("two_steps", 26, 641, 40, 9, 2, I.BF16),
    ("three_steps_k16", 12, 1400, 96, 16, 2, I.BF16),
    ("four_steps_k64", 20, 830, 120, 16, 4, I.BF16),
    ("six_steps", 33, 513, 192, 9, 3, I.BF16),
    ("eight_steps", 40, 450, 248, 9, 1, I.BF16),
    ("twelve_steps", 61, 269, 384, 9, 2, I.BF16),
    ("twenty_steps", 30, 560, 640, 9, 1, I.BF16),
    ("fp32_ragged", 33, 513, 36, 12, 3, I.F32),
    ("fp32_wide", 65, 257, 204, 9, 1, I.F32),
]


@pytest.mark.parametrize("case", TWO_KERNELS, ids=[c[0] for c in TWO_KERNELS])
def test_stream_and_tile_agree(case):
    """The two kernels rank the same packed keys: a batch past 1024 tiles of 16
    rows (streamed) and its first and last image alone (in-register) give the
    same graph, which is the oracle's."""
    require_gpu()
    from paper_2604_21290_amd import api
    label, B, N, C, k, d, dt = case
    assert _streams(B, N) and not _streams(1, N)
    x = I.random_features(N + C, B, N, C, dt, unit=False)
    xd = to_dev(x)
    _say("stream and tile", label)
    all_ = api.knn_graph(xd, k, d)
    for b in (0, B - 1):
        one = api.knn_graph(xd[b:b + 1].contiguous(), k, d)
        torch.cuda.synchronize()
        assert torch.equal(one[0], all_[b]), (label, b)
    rows = np.unique(np.linspace(0, N - 1, 24).astype(int))
    check_idx(all_[:1].cpu().numpy(), O.knn_distances(x.value[:1], rows=rows), k, d, rows=rows,
              label=label)


# -- ... and the widths whose limit lies below 1024 tiles ------------------------------
GRID_RULE = [
    # B images of N nodes, 513..1024 tiles of 16 rows: rows of whole 128-byte lines
    # past 512 or 768 tiles and one image less, other widths, two rounds of streamed
    # workgroups
    (9, 1000, 128, I.BF16), (8, 1024, 128, I.BF16), (13, 1000, 64, I.BF16), (12, 1024, 64, I.BF16),
    (16, 1024, 72, I.BF16), (9, 1024, 320, I.BF16), (13, 1024, 304, I.BF16), (13, 1024, 600, I.BF16),
    (20, 784, 384, I.BF16), (13, 1024, 160, I.F32), (12, 1024, 160, I.F32), (16, 1024, 128, I.F32),
]


@pytest.mark.parametrize("B,N,C,dt", GRID_RULE)
def test_grid_rule_edges(B, N, C, dt):
    """A batch on either side of its width's limit and its first and last image
    alone give the same graph, which is the oracle's."""
    require_gpu()
    from paper_2604_21290_amd import api
    x = I.random_features(N + C, B, N, C, dt, unit=False)
    xd = to_dev(x)
    _say("grid rule", B, N, C, dt)
    all_ = api.knn_graph(xd, 9, 2)
    for b in (0, B - 1):
        one = api.knn_graph(xd[b:b + 1].contiguous(), 9, 2)
        torch.cuda.synchronize()
        assert torch.equal(one[0], all_[b]), b
    rows = np.unique(np.linspace(0, N - 1, 24).astype(int))
    check_idx(all_[:1].cpu().numpy(), O.knn_distances(x.value[:1], rows=rows), 9, 2, rows=rows)


# -- rows that are not finite, against more than 256 keys -----------------------------
NON_FINITE = [
    # label, B, N, C, k, d, dtype
    ("k18", 26, 641, 40, 9, 2, I.BF16),
    ("k9_eight_steps", 40, 450, 248, 9, 1, I.BF16),
    ("k64_fp32", 33, 513, 36, 16, 4, I.F32),
]


@pytest.mark.parametrize("case", NON_FINITE, ids=[c[0] for c in NON_FINITE])
def test_non_finite_rows_by_grid(case):
    """A row with a NaN or an infinity has no distance to any other.  Against more
    than 256 keys such keys are in no list, on a large grid (streamed) and on a
    small one (in-register): a row's graph does not hang on its batch."""
    require_gpu()
    from paper_2604_21290_amd import api
    label, B, N, C, k, d, dt = case
    assert _streams(B, N) and not _streams(1, N) and N > 256
    g = np.random.default_rng(N)
    x = to_dev(I.random_features(N + C, B, N, C, dt, unit=False))
    bad = torch.from_numpy(g.random((B, N)) < 0.1).cuda()
    # the last image: too few finite rows to fill a list
    bad[-1] = torch.arange(N, device="cuda") % 150 != 0
    bad[-1, 1] = False
    col = torch.from_numpy(g.integers(0, C, (B, N))).cuda()
    val = torch.tensor([float("nan"), float("inf"), -float("inf")], device="cuda")
    val = val[torch.from_numpy(g.integers(0, 3, (B, N))).cuda()].to(x.dtype)
    at = torch.nonzero(bad, as_tuple=True)
    x[at[0], at[1], col[at]] = val[at]
    _say("non-finite", label)
    all_ = api.knn_graph(x, k, d)
    torch.cuda.synchronize()
    good = ~bad[:-1]
    for b in (0, B - 2):
        idx = all_[b][good[b]].long()
        assert int(idx.max()) < N and not bool(bad[b][idx].any()), (label, b)
    for b in (0, B - 2, B - 1):
        one = api.knn_graph(x[b:b + 1].contiguous(), k, d)
        torch.cuda.synchronize()
        assert torch.equal(one[0], all_[b]), (label, b)
