"""GPU parity: sdllm_block_attention against the fp64 oracle (paper Eq. 8 and the paragraph after
it).  Bar: max-abs error <= 1e-5 for fp32 and <= 2e-2 for bf16."""
import numpy as np
import pytest
import torch

import workloads as wl
from oracle import block_attention as oracle_attention
from gpu_util import attn_to_dev, attn_to_f64, to_f64_host, attention_error_ratio

pytestmark = pytest.mark.gpu

TOL = {"fp32": 1e-5, "bf16": 2e-2}


def run_gpu(sd, t, P, scale=0.0, kv_splits=0):
    d = attn_to_dev(t)
    n_keep = d["keep_idx"].shape[0]
    out = sd.block_attention(d["q_block"], d["q_suffix"] if n_keep else None,
                             d["k_cache"] if P else None, d["v_cache"] if P else None,
                             d["k_block"], d["v_block"],
                             d["k_suffix"] if n_keep else None, d["v_suffix"] if n_keep else None,
                             d["keep_idx"] if n_keep else None, P, scale=scale, kv_splits=kv_splits)
    torch.cuda.synchronize()
    return to_f64_host(out)


def oracle(t, P, scale=None):
    f = attn_to_f64(t)
    return oracle_attention(f["q_block"], f["q_suffix"], f["k_cache"], f["v_cache"], f["k_block"], f["v_block"],
                            f["k_suffix"], f["v_suffix"], f["keep_idx"], P, scale)


def oracle_abs_v(t, P, scale=None):
    """The oracle on |V|: the per-element scale of the bf16 error bound (gpu_util.attention_error_ratio)."""
    f = attn_to_f64(t)
    return oracle_attention(f["q_block"], f["q_suffix"], f["k_cache"], np.abs(f["v_cache"]), f["k_block"],
                            np.abs(f["v_block"]), f["k_suffix"], np.abs(f["v_suffix"]), f["keep_idx"], P, scale)


def assert_bf16_close(got, t, P, scale=None, what=""):
    want = oracle(t, P, scale)
    err = float(np.abs(got - want).max())
    ratio = attention_error_ratio(got, want, oracle_abs_v(t, P, scale))
    print(f"{what} max-abs err {err:.3e} (bar 2e-2), err / element-wise bf16 bound {ratio:.3f} (bar 1)")
    assert err <= TOL["bf16"]
    assert ratio <= 1.0


def test_attention_cfg1_fp32(gpu_lib):
    w = wl.WORKLOADS["cfg1"]
    t = wl.make_attention_inputs(w, seed=0)
    got = run_gpu(gpu_lib, t, w.P)
    want = oracle(t, w.P)
    err = np.abs(got - want).max()
    print(f"cfg1 fp32 max-abs err {err:.3e}")
    assert got.shape == (1, 4, 48, 64)
    assert err <= TOL["fp32"]


@pytest.mark.parametrize("B,Hq,Hkv,D,P,cap,K,S,keep", [
    (1, 1, 1, 4, 0, 0, 1, 0, ()),                 # single key, no cache, no suffix
    (2, 4, 2, 64, 37, 40, 32, 50, (0, 3, 4, 49)), # GQA, ragged key count
    (1, 2, 2, 128, 130, 200, 7, 9, tuple(range(9))),
    (1, 3, 1, 256, 5, 5, 3, 2, (1,)),
])
def test_attention_fp32_shapes(gpu_lib, B, Hq, Hkv, D, P, cap, K, S, keep):
    t = wl.make_custom_attention_inputs("fp32", B, Hq, Hkv, D, P, max(cap, 1), K, max(S, 1), keep, seed=D + P)
    got = run_gpu(gpu_lib, t, P)
    want = oracle(t, P)
    assert np.abs(got - want).max() <= TOL["fp32"]


@pytest.mark.parametrize("B,Hq,Hkv,D,P,K,S,keep,nr", [
    # one 16-row block per workgroup, the keys shared by up to eight waves: more waves than key blocks, a last block of
    # one key, a full one, head widths off the 16- and 64-element grid
    (1, 4, 4, 20, 14, 3, 0, (), 1),
    (2, 4, 2, 80, 31, 17, 40, (0, 1, 5, 39), 1),
    (1, 2, 1, 128, 112, 16, 64, tuple(range(16, 48)), 1),         # suffix blocks on consecutive rows
    (1, 2, 1, 132, 50, 15, 33, tuple(range(0, 33, 2)), 1),        # ... on scattered rows; D > 128: four waves
    (9, 1, 1, 64, 33, 5, 0, (), 1),                               # group count that does not fit the 8 chip parts
    # enough groups for the chip: the keys in one, two and four shares of at least four blocks, or one of fewer
    (64, 32, 32, 16, 64, 1, 0, (), 1),
    (32, 32, 32, 8, 90, 1, 7, (2, 6), 1),
    (32, 16, 16, 64, 235, 3, 0, (), 1),
    (32, 64, 32, 132, 20, 2, 0, (), 1),
    # two, four and eight row blocks per workgroup (from 512 row blocks on), one workgroup per group
    (16, 16, 16, 32, 10, 30, 0, (), 2),
    (16, 64, 16, 64, 20, 16, 0, (), 4),
    (16, 64, 16, 16, 7, 31, 1, (0,), 8),
    (16, 64, 16, 144, 9, 16, 0, (), 4),
])
def test_attention_fp32_workgroup_shapes(gpu_lib, B, Hq, Hkv, D, P, K, S, keep, nr):
    p = gpu_lib.attn_params(gpu_lib.FP32, B, Hq, Hkv, D, P, P + 3, K, S, len(keep))
    assert gpu_lib.plan_attention(p).rows_per_workgroup == 16 * nr
    t = wl.make_custom_attention_inputs("fp32", B, Hq, Hkv, D, P, P + 3, K, max(S, 1), keep, seed=D + P)
    got = run_gpu(gpu_lib, t, P)
    assert np.abs(got - oracle(t, P)).max() <= TOL["fp32"]


@pytest.mark.parametrize("D", [68, 80, 100, 128])
@pytest.mark.parametrize("P,K,S,keep", [
    (700, 32, 0, ()),                                             # several blocks per wave, all in the cache
    (403, 33, 300, tuple(range(0, 300, 3))),                      # blocks over a seam, kept rows scattered, a partial last block
    (0, 5, 200, tuple(range(7, 180)) + (199,)),                   # no cache; runs of kept rows that start at any row
    (11, 1, 0, ()),                                               # one partial block, one wave with work
])
def test_attention_fp32_k_through_lds(gpu_lib, D, P, K, S, keep):
    """Head widths whose K goes through LDS: every route a block's rows can take, and padded head widths."""
    t = wl.make_custom_attention_inputs("fp32", 2, 6, 2, D, P, P + 3, K, max(S, 1), keep, seed=D + P)
    got = run_gpu(gpu_lib, t, P)
    assert np.abs(got - oracle(t, P)).max() <= TOL["fp32"]


@pytest.mark.parametrize("B,Hq,Hkv,D,P,K,S,keep,nr,workgroups", [
    # several workgroups per group and a last one whose waves do not all have rows: 15 row blocks as 8 x 2, 4 x 4, 2 x 8
    (8, 20, 5, 16, 20, 57, 9, (0, 8), 2, 320),
    (16, 20, 5, 16, 20, 57, 9, (0, 8), 4, 320),
    (28, 20, 5, 16, 20, 57, 9, (0, 8), 8, 288),                   # 140 groups: padded to 144 for the 8 chip parts
    (8, 20, 5, 132, 20, 57, 9, (0, 8), 2, 320),
    # 25 groups, which do not fit the 8 chip parts: 21 row blocks as 11 x 2, 43 as 11 x 4, 83 as 11 x 8
    (25, 8, 1, 16, 20, 40, 9, (3, 4), 2, 275),
    (25, 17, 1, 16, 9, 40, 0, (), 4, 275),
    (25, 33, 1, 16, 9, 40, 0, (), 8, 275),
])
def test_attention_fp32_several_row_tiles(gpu_lib, B, Hq, Hkv, D, P, K, S, keep, nr, workgroups):
    p = gpu_lib.attn_params(gpu_lib.FP32, B, Hq, Hkv, D, P, P, K, S, len(keep))
    plan = gpu_lib.plan_attention(p)
    assert (plan.rows_per_workgroup, plan.workgroups) == (16 * nr, workgroups)
    rows = Hq // Hkv * (K + len(keep))
    assert -(-rows // 16) % nr != 0                               # row blocks of a group that fill no whole workgroup
    t = wl.make_custom_attention_inputs("fp32", B, Hq, Hkv, D, P, P, K, max(S, 1), keep, seed=B + D)
    got = run_gpu(gpu_lib, t, P)
    assert np.abs(got - oracle(t, P)).max() <= TOL["fp32"]


@pytest.mark.parametrize("D", [80, 128])
@pytest.mark.parametrize("B,Hq,Hkv,P,K,S,keep,nr,workgroups", [
    (8, 20, 5, 20, 57, 9, (0, 8), 2, 320),                        # two, four, eight row blocks per workgroup, the last workgroup
    (16, 20, 5, 20, 57, 9, (0, 8), 4, 320),                       # of a group not full; five key blocks, the last partial; with
    (28, 20, 5, 20, 57, 9, (0, 8), 8, 288),                       # eight row blocks a wave has all of the keys and nothing merges
    (12, 32, 32, 48, 16, 0, (), 1, 384),                          # most workgroups, fewest keys for K through LDS
    (12, 32, 32, 47, 16, 0, (), 1, 384),                          # one key fewer, or more workgroups: K in registers
    (13, 32, 32, 48, 16, 0, (), 1, 416),
])
def test_attention_fp32_k_through_lds_row_tiles(gpu_lib, D, B, Hq, Hkv, P, K, S, keep, nr, workgroups):
    p = gpu_lib.attn_params(gpu_lib.FP32, B, Hq, Hkv, D, P, P, K, S, len(keep))
    plan = gpu_lib.plan_attention(p)
    assert (plan.rows_per_workgroup, plan.workgroups) == (16 * nr, workgroups)
    t = wl.make_custom_attention_inputs("fp32", B, Hq, Hkv, D, P, P, K, max(S, 1), keep, seed=B + D + P)
    got = run_gpu(gpu_lib, t, P)
    assert np.abs(got - oracle(t, P)).max() <= TOL["fp32"]


@pytest.mark.parametrize("D,P,K,first,nkeys", [
    (64, 300, 20, 0, 16),           # the first key block: every score of one wave's first block is -inf
    (64, 300, 20, 80, 16),          # ... of another wave
    (128, 300, 20, 0, 128),         # ... of all eight waves
    (256, 100, 5, 48, 16),          # four waves
    (64, 16, 9, 0, 16),             # two key blocks
])
def test_attention_fp32_scores_that_overflow(gpu_lib, D, P, K, first, nkeys):
    """Finite inputs whose scores lie below the fp32 range for some keys: those keys have weight zero, the others
    share the row."""
    t = wl.make_custom_attention_inputs("fp32", 1, 2, 1, D, P, P, K, 1, (), seed=D + first)
    for name in ("q_block", "k_cache", "k_block"):
        t[name][..., 0] = 0.0
    t["q_block"][..., 0] = 1e20
    t["k_cache"][:, :, first:first + nkeys, 0] = -1e20
    got = run_gpu(gpu_lib, t, P)
    assert np.abs(got - oracle(t, P)).max() <= TOL["fp32"]


@pytest.mark.parametrize("D", [4, 20, 52, 80, 124, 132, 252])
def test_attention_fp32_infinite_last_element_of_k(gpu_lib, D):
    """A key whose last element makes its scores -inf has weight zero, also where the head does not fill the 16-element
    slices of the kernel."""
    t = wl.make_custom_attention_inputs("fp32", 1, 2, 1, D, 37, 40, 5, 9, (2, 3, 8), seed=D)
    for name in ("q_block", "q_suffix"):
        t[name][..., D - 1] = np.abs(t[name][..., D - 1]) + 0.1
    t["k_cache"][:, :, 3, D - 1] = -np.inf
    t["k_block"][:, :, 4, D - 1] = -np.inf
    t["k_suffix"][:, :, 8, D - 1] = -np.inf
    got = run_gpu(gpu_lib, t, 37)
    assert np.abs(got - oracle(t, 37)).max() <= TOL["fp32"]


@pytest.mark.parametrize("D,P,K", [(64, 37, 4), (80, 11, 4), (128, 300, 5), (256, 61, 2), (4, 0, 1)])
def test_attention_fp32_infinite_last_row_of_v(gpu_lib, D, P, K):
    """The last key's V row is infinite in one column and the number of keys is no multiple of the key block: that
    column of the output is infinite, the others are what they are without it."""
    assert (P + K) % 16 != 0
    t = wl.make_custom_attention_inputs("fp32", 1, 2, 1, D, P, max(P, 1), K, 1, (), seed=D)
    t["v_block"][:, :, K - 1, 1] = np.inf
    got, want = run_gpu(gpu_lib, t, P), oracle(t, P)
    assert np.isposinf(want[..., 1]).all() and np.isposinf(got[..., 1]).all()
    keep = np.arange(D) != 1
    assert np.abs(got[..., keep] - want[..., keep]).max() <= TOL["fp32"]


def test_attention_fp32_more_groups_than_one_grid_row(gpu_lib):
    """1025 x 65535 heads of one query and one key, whose output is the key's V row: 2^32 work-items and more."""
    B, H, D = 1025, 65535, 4
    q, k = (torch.ones((B, H, 1, D), device="cuda") for _ in range(2))
    v = torch.randn((B, H, 1, D), device="cuda")
    assert gpu_lib.plan_attention(gpu_lib.attn_params(gpu_lib.FP32, B, H, H, D, 0, 0, 1, 0, 0)).workgroups * 64 >= 1 << 32
    out = gpu_lib.block_attention(q, None, None, None, k, v, None, None, None, 0)
    assert torch.equal(out, v)


@pytest.mark.parametrize("kv_splits", [0, 1, 2, 3])
def test_attention_small_bf16(gpu_lib, kv_splits):
    w = wl.WORKLOADS["small_bf16"]             # GQA 4/2, P=107, K=32, s=33: ragged key and query tiles
    t = wl.make_attention_inputs(w, seed=0)
    got = run_gpu(gpu_lib, t, w.P, kv_splits=kv_splits)
    assert_bf16_close(got, t, w.P, what=f"small_bf16 splits={kv_splits}")


@pytest.mark.parametrize("B,Hq,Hkv,D,P,cap,K,S,keep,splits", [
    (1, 1, 1, 128, 0, 0, 1, 0, (), 0),                          # one query, one key
    (1, 2, 2, 128, 0, 0, 32, 0, (), 0),                         # no cache, no suffix
    (2, 2, 1, 64, 64, 64, 32, 40, (0, 1, 2, 39), 0),            # D = 64, GQA
    (1, 8, 2, 128, 100, 128, 32, 64, tuple(range(0, 64, 2)), 2),# g = 4: 256 virtual rows, two query tiles
    (1, 7, 1, 128, 63, 64, 32, 10, (9,), 0),                    # g = 7, key count 96 = tile boundary + 32
    (3, 2, 2, 128, 257, 300, 64, 70, tuple(range(63)) + (69,), 4),
    (1, 1, 1, 64, 1000, 1000, 5, 3, (0, 2), 7),                 # few queries, many keys, odd split count
])
def test_attention_bf16_shapes(gpu_lib, B, Hq, Hkv, D, P, cap, K, S, keep, splits):
    t = wl.make_custom_attention_inputs("bf16", B, Hq, Hkv, D, P, max(cap, 1), K, max(S, 1), keep, seed=P + K)
    got = run_gpu(gpu_lib, t, P, kv_splits=splits)
    assert_bf16_close(got, t, P, what="bf16 shape")


@pytest.mark.parametrize("B,Hq,Hkv,D,P,cap,K,S,keep,splits", [
    # a wave moves 16-row slabs of a key tile; a slab that lies in one tensor and (for the suffix) maps to
    # consecutive rows takes a scalar-base path, every other slab a per-row path: hit both and their borders
    (1, 2, 2, 128, 48, 64, 32, 100, tuple(range(5, 53)) + (99,), 0),      # window not starting at 0, then a jump
    (2, 2, 1, 128, 40, 40, 24, 90, tuple(range(0, 64)), 0),               # P, K off the slab grid: straddling slabs
    (1, 1, 1, 128, 64, 64, 32, 64, tuple(range(0, 8)) + tuple(range(9, 17)) + tuple(range(17, 49)), 0),  # one gap inside a slab
    (1, 2, 2, 64, 32, 48, 32, 300, tuple(range(100, 164)) + (299,), 2),   # D = 64, late window, split keys
    (1, 4, 1, 128, 0, 0, 48, 200, tuple(range(200)), 3),                  # no cache: block slabs, then a long run
    (1, 1, 1, 128, 16, 16, 16, 40, tuple(range(1, 40, 1)), 0),            # run ends 1 short of a slab
])
def test_attention_bf16_slab_paths(gpu_lib, B, Hq, Hkv, D, P, cap, K, S, keep, splits):
    t = wl.make_custom_attention_inputs("bf16", B, Hq, Hkv, D, P, max(cap, 1), K, max(S, 1), keep, seed=3 * P + K + S)
    got = run_gpu(gpu_lib, t, P, kv_splits=splits)
    assert_bf16_close(got, t, P, what="bf16 slab-path")


@pytest.mark.parametrize("shape,B,Hq,Hkv,D,P,cap,K,S,keep,splits", [
    # shape 1: two 4-wave groups on the same rows alternate key tiles and merge through LDS.  Odd and even tile
    # counts (the second group then has one tile less or as many), ragged last tile, tiles that straddle the cache /
    # block / suffix borders, gaps in keep_idx, D = 64, a forced split, two query tiles, 32-row waves
    (1, 1, 2, 2, 128, 300, 300, 32, 40, tuple(range(0, 30)) + (39,), 1),      # 363 keys: 6 tiles, the last ragged
    (1, 2, 2, 1, 128, 270, 280, 24, 50, tuple(range(3, 43)), 1),              # 334 keys: 6 tiles; nothing on the slab grid
    (1, 1, 3, 3, 128, 256, 256, 32, 64, tuple(range(0, 32)), 1),              # 320 keys: exactly 5 tiles (odd)
    (1, 1, 2, 2, 128, 200, 256, 32, 80, tuple(range(0, 80, 2)), 1),           # gathered suffix with gaps: per-row transfers
    (1, 2, 2, 2, 64, 500, 512, 32, 33, tuple(range(33)), 1),                  # D = 64, 565 keys: 9 tiles
    (1, 1, 2, 2, 128, 1000, 1024, 32, 64, tuple(range(0, 63)) + (63,), 2),    # two splits of 9 tiles, each shared by two groups
    (1, 1, 8, 2, 128, 400, 400, 16, 20, tuple(range(0, 16)), 1),              # GQA 4:1, 128 rows per K/V head: two query tiles
    (1, 1, 1, 1, 128, 4100, 4100, 64, 64, tuple(range(0, 63)) + (63,), 2),    # 128 rows on 4228 keys: 32-row waves, 67 tiles
    (1, 1, 1, 1, 128, 4100, 4100, 50, 64, tuple(range(0, 40)), 2),            # the same with 90 rows: ragged 32-row blocks
    # shape 2: two groups on different rows (256 per workgroup) share every key tile through a three-stage ring
    (2, 1, 4, 1, 128, 100, 128, 64, 70, tuple(range(0, 64)), 0),              # 512 rows = 2 full workgroups, 228 keys: 4 tiles
    (0, 1, 8, 2, 128, 37, 40, 32, 40, tuple(range(0, 33)), 0),                # 260 rows per head, 2 key tiles: the 4-wave workgroup
    (2, 1, 9, 1, 128, 70, 70, 32, 40, tuple(range(2, 28)), 0),                # 522 rows: 3 workgroups, the last with 10 rows
    (2, 2, 8, 1, 64, 130, 140, 32, 60, tuple(range(0, 60, 1))[:36], 0),       # D = 64, 544 rows, 198 keys
    (2, 1, 16, 2, 128, 5, 8, 32, 33, tuple(range(33)), 0),                    # 520 rows on 70 keys: 2 tiles, ring deeper than the stream
    (2, 1, 8, 1, 128, 0, 0, 64, 1, (0,), 3),                                  # 520 rows, no cache, forced splits of one tile
])
def test_attention_bf16_workgroup_shapes(gpu_lib, shape, B, Hq, Hkv, D, P, cap, K, S, keep, splits):
    """The 8-wave workgroup shapes at sizes the oracle checks element by element (every output element, the
    element-wise bf16 bound).  `shape` is the workgroup shape the plan must pick for the case (the split count is
    given where the automatic one would cut a small batch into splits too short to share)."""
    sd = gpu_lib
    t = wl.make_custom_attention_inputs("bf16", B, Hq, Hkv, D, P, max(cap, 1), K, max(S, 1), keep, seed=7 * P + K + len(keep))
    pl = sd.plan_attention(sd.attn_params(sd.BF16, B, Hq, Hkv, D, P, max(cap, 1), K, max(S, 1), len(keep), 0.0, splits))
    assert pl.workgroup_shape == shape, (pl.workgroup_shape, pl.kv_splits, pl.key_tiles_per_split)
    got = run_gpu(sd, t, P, kv_splits=splits)
    assert_bf16_close(got, t, P, what=f"workgroup shape {pl.workgroup_shape}, {pl.kv_splits} split(s), "
                                      f"{pl.key_tiles_per_split} tiles per split:")


@pytest.mark.parametrize("shape,rows,B,Hq,Hkv,D,P,K,S,keep", [
    (0, 64, 1, 8, 1, 128, 500, 64, 70, tuple(range(64))),                     # 1024 rows on 628 keys: 16 query tiles, splits
    (1, 64, 2, 8, 1, 64, 700, 40, 60, tuple(range(1, 52))),                   # D = 64, 728 rows, the last tile ragged, two groups alternate key tiles
    (0, 64, 1, 16, 1, 128, 900, 20, 33, tuple(range(0, 26, 2))),              # 528 rows: nine query tiles, five splits
    (1, 128, 3, 36, 4, 128, 3000, 32, 50, tuple(range(40))),                  # 648 rows: 128-row tiles, the last with 8 rows; 16 key tiles a split
    (0, 128, 6, 64, 16, 128, 500, 64, 96, tuple(range(96))),                  # 640 rows = 5 tiles of 128, more than one round
])
def test_attention_bf16_many_rows_few_groups(gpu_lib, shape, rows, B, Hq, Hkv, D, P, K, S, keep):
    """From 512 query rows per K/V head on, the smaller workgroups that the plan picks where few groups share the chip."""
    sd = gpu_lib
    t = wl.make_custom_attention_inputs("bf16", B, Hq, Hkv, D, P, P, K, S, keep, seed=7 * P + K + len(keep))
    pl = sd.plan_attention(sd.attn_params(sd.BF16, B, Hq, Hkv, D, P, P, K, S, len(keep), 0.0, 0))
    assert (pl.workgroup_shape, pl.rows_per_workgroup) == (shape, rows)
    got = run_gpu(sd, t, P)
    assert_bf16_close(got, t, P, what=f"{rows} rows, {pl.kv_splits} split(s), {pl.key_tiles_per_split} tiles per split:")


@pytest.mark.parametrize("spread,shift", [(1.0, 0.0), (0.1, 0.0), (2.0, 0.0), (1.0, 2.0), (1.0, 20.0)])
@pytest.mark.parametrize("B,Hq,Hkv,D,P,K,S,keep", [
    (1, 8, 1, 128, 500, 64, 70, tuple(range(64))),
    (2, 8, 1, 64, 700, 40, 60, tuple(range(1, 52))),
])
def test_attention_bf16_row_sum_of_64_row_workgroups(gpu_lib, B, Hq, Hkv, D, P, K, S, keep, spread, shift):
    """From 512 rows per K/V head the plan may take 64-row workgroups, whose softmax row sum adds probabilities rounded to bf16,
    or 256-row ones, which add fp32 probabilities: the output's error against 64 bits does not grow by that.  The two differ
    only in rounding, over B Hq (K + kept) D outputs: 1 % is ten times what their ratio exceeds 1 by at most."""
    sd = gpu_lib
    t = wl.make_custom_attention_inputs("bf16", B, Hq, Hkv, D, P, P, K, S, keep, seed=P + len(keep))
    for name in ("q_block", "q_suffix", "k_cache", "k_block", "k_suffix"):
        t[name] = wl.f32_to_bf16_bits(wl.bf16_bits_to_f32(t[name]) * np.float32(spread))
    for name in ("v_cache", "v_block", "v_suffix"):
        t[name] = wl.f32_to_bf16_bits(wl.bf16_bits_to_f32(t[name]) + np.float32(shift))
    pl = sd.plan_attention(sd.attn_params(sd.BF16, B, Hq, Hkv, D, P, P, K, S, len(keep), 0.0, 0))
    other = sd.plan_attention(sd.attn_params(sd.BF16, B, Hq, Hkv, D, P, P, K, S, len(keep), 0.0, pl.kv_splits))
    assert (pl.rows_per_workgroup, other.rows_per_workgroup, other.kv_splits) == (64, 256, pl.kv_splits)
    want = oracle(t, P)
    error = [float(np.sqrt(((run_gpu(sd, t, P, kv_splits=n) - want) ** 2).sum())) for n in (0, pl.kv_splits)]
    assert error[0] <= 1.01 * error[1], error


def _random_case(seed):
    """A seeded random problem: small enough for the oracle, wide enough to reach every workgroup shape, both head
    dims, GQA ratios up to 8, empty caches / suffixes, forced and automatic key splits."""
    g = np.random.Generator(np.random.Philox(key=1000 + seed))
    D = int(g.choice([64, 128]))
    Hkv = int(g.integers(1, 4))
    ratio = int(g.choice([1, 1, 2, 4, 7, 8]))
    B = int(g.integers(1, 4))
    K = int(g.choice([1, 7, 16, 32, 33, 64]))
    P = int(g.choice([0, 5, 63, 64, 130, 333, 700, 1500]))
    cap = P + int(g.integers(0, 40))
    S = int(g.choice([0, 1, 9, 40, 80]))
    n_keep = int(g.integers(0, S + 1))
    keep = tuple(sorted(g.choice(S, size=n_keep, replace=False).tolist())) if n_keep else ()
    splits = int(g.choice([0, 0, 1, 2, 3]))
    return B, ratio * Hkv, Hkv, D, P, cap, K, S, keep, splits


@pytest.mark.parametrize("seed", range(48))
def test_attention_bf16_random_shapes(gpu_lib, seed):
    """Seeded random shapes against the oracle, every output element, with the element-wise bf16 bound."""
    sd = gpu_lib
    B, Hq, Hkv, D, P, cap, K, S, keep, splits = _random_case(seed)
    t = wl.make_custom_attention_inputs("bf16", B, Hq, Hkv, D, P, max(cap, 1), K, max(S, 1), keep, seed=seed)
    pl = sd.plan_attention(sd.attn_params(sd.BF16, B, Hq, Hkv, D, P, max(cap, 1), K, max(S, 1), len(keep), 0.0, splits))
    got = run_gpu(sd, t, P, kv_splits=splits)
    assert_bf16_close(got, t, P, what=f"seed {seed}: B{B} H{Hq}/{Hkv} D{D} P{P} K{K} kept {len(keep)}/{S}, shape "
                                      f"{pl.workgroup_shape}, {pl.kv_splits} split(s) of {pl.key_tiles_per_split} tiles:")


@pytest.mark.parametrize("std,scale,splits", [(8.0, 1.0, 0), (8.0, 1.0, 3), (0.01, 0.0, 0), (30.0, 0.5, 1)])
def test_attention_bf16_extreme_score_ranges(gpu_lib, std, scale, splits):
    """Scores far outside the usual range: Q, K ~ N(0, std^2) with scale 1 puts |score| in the hundreds to tens of
    thousands (the softmax is all but one-hot and the running reference exponent jumps by hundreds between tiles),
    std 0.01 makes it all but uniform.  No overflow, no NaN, the oracle's result within the bf16 bound."""
    B, Hq, Hkv, D, P, K, S = 2, 4, 2, 128, 700, 32, 64
    keep = tuple(range(0, 64, 3))
    t = wl.make_custom_attention_inputs("bf16", B, Hq, Hkv, D, P, P, K, S, keep, seed=int(std * 100) + splits, std=std)
    # values stay N(0, 1): only the scores are extreme
    v = wl.make_custom_attention_inputs("bf16", B, Hq, Hkv, D, P, P, K, S, keep, seed=99, std=1.0)
    for name in ("v_cache", "v_block", "v_suffix"):
        t[name] = v[name]
    got = run_gpu(gpu_lib, t, P, scale=scale, kv_splits=splits)
    assert np.isfinite(got).all()
    assert_bf16_close(got, t, P, scale=(scale if scale > 0 else None), what=f"std {std} scale {scale} splits {splits}:")


def test_attention_bf16_keep_all_equals_full_context(gpu_lib):
    """Keeping every suffix row = dense attention over the concatenated sequence: feed the same rows
    through the cache operand instead and compare the two GPU results with each other and the oracle."""
    B, Hq, Hkv, D, P, K, S = 1, 2, 2, 128, 40, 32, 56
    t = wl.make_custom_attention_inputs("bf16", B, Hq, Hkv, D, P, P, K, S, tuple(range(S)), seed=9)
    got = run_gpu(gpu_lib, t, P)
    want = oracle(t, P)
    assert np.abs(got - want).max() <= TOL["bf16"]


def test_attention_bf16_scale_param_and_determinism(gpu_lib):
    w = wl.WORKLOADS["small_bf16"]
    t = wl.make_attention_inputs(w, seed=3)
    a = run_gpu(gpu_lib, t, w.P, scale=0.05, kv_splits=2)
    b = run_gpu(gpu_lib, t, w.P, scale=0.05, kv_splits=2)
    assert (a == b).all()                                   # fixed merge order: bit-identical reruns
    want = oracle(t, w.P, 0.05)
    assert np.abs(a - want).max() <= TOL["bf16"]


def test_attention_cfg2_full(gpu_lib):
    w = wl.WORKLOADS["cfg2"]
    t = wl.make_attention_inputs(w, seed=0)
    got = run_gpu(gpu_lib, t, w.P)
    want = oracle(t, w.P)
    err = np.abs(got - want).max()
    worst, ratio = _check_pairs(got, _host_slicer(t), _all_pairs(w), 1, t["keep_idx"], w.P)
    print(f"cfg2 max-abs err {err:.3e} (|out| max {np.abs(want).max():.3f}), err / element-wise bf16 bound {ratio:.3f}")
    assert err <= TOL["bf16"] and ratio <= 1.0
    # the same data with scale-free N(0,1)-like spread: multiply q by sqrt(128) via the scale parameter
    got2 = run_gpu(gpu_lib, t, w.P, scale=1.0)
    want2 = oracle(t, w.P, 1.0)
    assert np.abs(got2 - want2).max() <= TOL["bf16"]


def _pair_oracle(sub, keep, P, absolute_v=False):
    """Oracle for one (batch, head) pair given its eight operand slices (host float64)."""
    vs = [np.abs(sub[k]) if absolute_v else sub[k] for k in ("v_cache", "v_block", "v_suffix")]
    return oracle_attention(sub["q_block"], sub["q_suffix"], sub["k_cache"], vs[0], sub["k_block"], vs[1],
                            sub["k_suffix"], vs[2], keep, P)[0, 0]


def _check_pairs(got, slicer, pairs, g, keep, P):
    """Compares `got[b, hq]` with the oracle for every pair: the stated 2e-2 absolute bar and the element-wise
    bound of the bf16 arithmetic (gpu_util.attention_error_ratio).  Returns (worst abs error, worst ratio)."""
    worst, worst_ratio = 0.0, 0.0
    for (b, hq) in pairs:
        sub = slicer(b, hq, hq // g)
        want = _pair_oracle(sub, keep, P)
        want_abs = _pair_oracle(sub, keep, P, absolute_v=True)
        worst = max(worst, float(np.abs(got[b, hq] - want).max()))
        worst_ratio = max(worst_ratio, attention_error_ratio(got[b, hq], want, want_abs))
    return worst, worst_ratio


def _host_slicer(t):
    def f(b, hq, kv):
        return {k: wl.to_f64(v[b:b + 1, (hq if k.startswith("q_") else kv):(hq if k.startswith("q_") else kv) + 1])
                for k, v in t.items() if k != "keep_idx"}
    return f


def _all_pairs(w):
    return [(b, h) for b in range(w.B) for h in range(w.Hq)]


def _cfg3b_pairs(w):
    """>= 32 pairs of cfg3B that cover every (batch, KV head) residue modulo the 8 XCDs the launch maps work
    units to; each pair carries all 8 query tiles of its head."""
    g = np.random.Generator(np.random.Philox(key=33))
    pairs = set()
    units = [(b, h) for b in range(w.B) for h in range(w.Hq)]
    for r in range(8):                                       # unit id = b * Hkv + kvh (one split): 4 per residue
        cand = [u for u in units if (u[0] * w.Hkv + u[1] // (w.Hq // w.Hkv)) % 8 == r]
        for i in g.choice(len(cand), size=4, replace=False):
            pairs.add(cand[int(i)])
    pairs |= {(0, 0), (w.B - 1, w.Hq - 1)}
    return sorted(pairs)


@pytest.mark.parametrize("name", ["cfg3A", "cfg3B", "cfg4", "cfgBC"])
def test_attention_full_size(gpu_lib, name):
    """Full-size launch in the configuration the bench times.  cfg3A, cfg4, cfgBC: EVERY (batch, head) pair
    against the oracle; cfg3B (1 GFLOP of fp64 per pair): 34 pairs that hit every XCD residue of the work-unit
    map, all query tiles of each."""
    w = wl.WORKLOADS[name]
    t = wl.make_attention_inputs(w, seed=0)
    got = run_gpu(gpu_lib, t, w.P)
    assert np.isfinite(got).all()
    pairs = _cfg3b_pairs(w) if name == "cfg3B" else _all_pairs(w)
    worst, ratio = _check_pairs(got, _host_slicer(t), pairs, w.Hq // w.Hkv, t["keep_idx"], w.P)
    print(f"{name}: {len(pairs)} of {w.B * w.Hq} pairs, max-abs err {worst:.3e} (bar 2e-2), "
          f"worst err / element-wise bf16 bound {ratio:.3f} (bar 1)")
    assert worst <= TOL["bf16"]
    assert ratio <= 1.0


@pytest.mark.parametrize("name", ["cfg2", "cfg3A", "cfg3B", "cfg4", "cfg5", "cfgBC"])
def test_attention_full_size_every_key_counted_once(gpu_lib, name):
    """Full size, every output element of every (batch, head, row), bench launch configuration.  With all-zero
    queries every score is 0 and the softmax is uniform, so the output is the plain mean of the composed V rows
    (the scale -> 0 closed form that also pins the oracle).  V holds small integers everywhere -- also in cache
    rows beyond P and in suffix rows that are not kept -- so every partial sum is exact in fp32 and the kernel's
    result is the exact mean rounded twice: a key that is dropped, duplicated or taken from a wrong row (any
    group, any XCD slot, any split) moves the mean by ~1/Nkv, several times the 2^-8 relative bar."""
    sd = gpu_lib
    w = wl.WORKLOADS[name]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(97)
    dt = torch.bfloat16

    def ints(*shape):
        return torch.randint(-2, 3, shape, generator=gen, device="cuda").to(dt)

    B, Hq, Hkv, D, K, S, cap, P = w.B, w.Hq, w.Hkv, w.D, w.K, w.S, w.cap, w.P
    keep = torch.from_numpy(wl.make_keep_idx(w)).cuda()
    nk = int(keep.shape[0])
    qb = torch.zeros((B, Hq, K, D), dtype=dt, device="cuda")
    qs = torch.zeros((B, Hq, max(S, 1), D), dtype=dt, device="cuda")
    kc, kb, ks = ints(B, Hkv, cap, D), ints(B, Hkv, K, D), ints(B, Hkv, max(S, 1), D)   # keys: anything finite
    vc, vb, vs = ints(B, Hkv, cap, D), ints(B, Hkv, K, D), ints(B, Hkv, max(S, 1), D)
    out = sd.block_attention(qb, qs if nk else None, kc, vc, kb, vb, ks if nk else None, vs if nk else None,
                             keep if nk else None, P)
    torch.cuda.synchronize()
    # closed form on the host, from the composition rule of Eq. 8 (integer sums, exact)
    vsum = vc[:, :, :P].double().sum(2) + vb.double().sum(2)
    if nk:
        vsum = vsum + vs[:, :, keep.long()].double().sum(2)
    mean = (vsum / w.Nkv).cpu().numpy()                                   # [B, Hkv, D]
    got = out.double().cpu().numpy()                                      # [B, Hq, Nq, D]
    want = np.repeat(mean, Hq // Hkv, axis=1)[:, :, None, :]
    err = np.abs(got - want)
    bar = 2.0 ** -8 * np.abs(want) + 1e-12
    print(f"{name}: every-key-once check over {got.size} elements, worst err / bar {float((err / bar).max()):.3f}; "
          f"a dropped key of value 1 would be {1.0 / w.Nkv / (2.0 ** -8 * np.abs(want).mean()):.1f} x the mean bar")
    assert (err <= bar).all()


def test_attention_rejects_bad_arguments(gpu_lib):
    sd = gpu_lib
    w = wl.WORKLOADS["small_bf16"]
    d = attn_to_dev(wl.make_attention_inputs(w, seed=0))
    with pytest.raises(sd.SdllmError) as e:       # prefix_len beyond the cache capacity
        sd.block_attention(d["q_block"], d["q_suffix"], d["k_cache"], d["v_cache"], d["k_block"], d["v_block"],
                           d["k_suffix"], d["v_suffix"], d["keep_idx"], w.cap + 1)
    assert e.value.status == sd.ERR_INVALID_ARG
    with pytest.raises(sd.SdllmError) as e:       # workspace too small for a forced split
        sd.block_attention(d["q_block"], d["q_suffix"], d["k_cache"], d["v_cache"], d["k_block"], d["v_block"],
                           d["k_suffix"], d["v_suffix"], d["keep_idx"], w.P, kv_splits=2,
                           workspace=torch.zeros(64, dtype=torch.uint8, device="cuda"))
    assert e.value.status == sd.ERR_WORKSPACE


def test_workspace_reuse_with_garbage(gpu_lib):
    """A workspace needs no initialisation and carries nothing between calls: one buffer, filled with
    garbage, serves attention and unmask calls of different shapes one after the other."""
    from oracle import confidence_unmask as oracle_unmask
    sd = gpu_lib
    ws = torch.full((64 << 20,), 0xA5, dtype=torch.uint8, device="cuda")
    for rep, (name, splits) in enumerate([("small_bf16", 3), ("small_bf16", 2), ("cfg2", 0), ("small_bf16", 4)]):
        w = wl.WORKLOADS[name]
        t = wl.make_attention_inputs(w, seed=rep)
        d = attn_to_dev(t)
        out = sd.block_attention(d["q_block"], d["q_suffix"], d["k_cache"], d["v_cache"], d["k_block"], d["v_block"],
                                 d["k_suffix"], d["v_suffix"], d["keep_idx"], w.P, kv_splits=splits, workspace=ws)
        torch.cuda.synchronize()
        assert np.abs(to_f64_host(out) - oracle(t, w.P)).max() <= TOL["bf16"], (name, splits)
        u = wl.make_unmask_inputs(wl.WORKLOADS["small_bf16"], seed=rep)
        tk = torch.from_numpy(u["tokens"]).cuda()
        mk = torch.from_numpy(u["masked"]).cuda()
        lg = torch.from_numpy(u["logits"].view(np.int16)).view(torch.bfloat16).cuda()
        sd.confidence_unmask(lg, tk, mk, 0.9, 0.3, workspace=ws)
        torch.cuda.synchronize()
        ref = oracle_unmask(wl.to_f64(u["logits"]), u["tokens"], u["masked"], float(np.float32(0.9)), float(np.float32(0.3)))
        assert (tk.cpu().numpy() == ref["tokens"]).all() and (mk.cpu().numpy() == ref["masked"]).all()


def test_attention_cfg5_layer0_all_pairs_and_sampled_layers(gpu_lib):
    """Long-context stack shape (P = 5120, 64-row block, 64 kept of 960): inputs are drawn on the device
    (seed + layer), the oracle sees the same bits copied back.  Layer 0: every (batch, head) pair; a seeded sample
    of three pairs in each of six other layers, the last one included."""
    sd = gpu_lib
    w = wl.WORKLOADS["cfg5"]
    g = w.Hq // w.Hkv
    rng = np.random.Generator(np.random.Philox(key=55))
    plan = [(0, _all_pairs(w))]
    for layer in (5, 11, 13, 22, 27, 31):
        plan.append((layer, [(int(rng.integers(w.B)), int(rng.integers(w.Hq))) for _ in range(3)]))
    worst, ratio, n = 0.0, 0.0, 0
    for layer, pairs in plan:
        d = wl.make_attention_inputs_device(w, seed=0, layer=layer)
        out = sd.block_attention(d["q_block"], d["q_suffix"], d["k_cache"], d["v_cache"], d["k_block"], d["v_block"],
                                 d["k_suffix"], d["v_suffix"], d["keep_idx"], w.P)
        torch.cuda.synchronize()
        assert torch.isfinite(out.float()).all()
        keep = d["keep_idx"].cpu().numpy()
        got = out.double().cpu().numpy()

        def slicer(b, hq, kv, d=d):
            return {k: d[k][b:b + 1, (hq if k.startswith("q_") else kv):(hq if k.startswith("q_") else kv) + 1]
                    .double().cpu().numpy() for k in d if k != "keep_idx"}

        wl_, rl_ = _check_pairs(got, slicer, pairs, g, keep, w.P)
        worst, ratio, n = max(worst, wl_), max(ratio, rl_), n + len(pairs)
        del d, out
    print(f"cfg5: {n} pairs over {len(plan)} layers, max-abs err {worst:.3e} (bar 2e-2), "
          f"worst err / element-wise bf16 bound {ratio:.3f} (bar 1)")
    assert worst <= TOL["bf16"]
    assert ratio <= 1.0


def test_attention_cfg2_relative_error(gpu_lib):
    """cfg2 draws Q/K/V with std 1/sqrt(128), so outputs are ~0.01 and the absolute 2e-2 bar alone would
    be loose: also require 2e-2 relative to the largest output magnitude."""
    w = wl.WORKLOADS["cfg2"]
    t = wl.make_attention_inputs(w, seed=1)
    got = run_gpu(gpu_lib, t, w.P)
    want = oracle(t, w.P)
    assert np.abs(got - want).max() <= 2e-2 * np.abs(want).max()
