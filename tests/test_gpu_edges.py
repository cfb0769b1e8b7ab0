"""GPU parity at the sizes where a kernel's own partition of the work ends: remainders of its steps, the shortest and
the longest lists, tile shapes off the beaten track.  Against the oracle, with the tolerances of the parity tests."""
import numpy as np
import pytest

from paper_2407_08330_amd import inputs
from test_gpu_bwd import run_bwd_case
from test_gpu_cross import _compare_schedule, run_cross_case
from test_gpu_fwd import run_fwd_case
from gpu_common import compare_layout, say, to_dev_i32

pytestmark = pytest.mark.gpu


def _padded(docs, n):
    level = np.stack([np.concatenate([l, np.full(n - l.shape[0], -1, np.int32)]) for l, _ in docs])
    parent = np.stack([np.concatenate([p, np.full(n - p.shape[0], -1, np.int32)]) for _, p in docs])
    return level, parent


@pytest.mark.parametrize("tile,D,windowed", [((96, 96), 64, False), ((32, 32), 128, False), ((128, 128), 64, True),
                                             ((64, 96), 128, True)])
def test_fp32_rows_lists_and_tile_shapes(oracle, tile, D, windowed):
    # the fp32 kernels take a wave per row, four rows per workgroup, 256 key slots per round and 16 keys per step: an odd
    # number of rows, groups of 1, 15, 16, 17, 255-257 siblings, and one of 700 that needs several rounds
    docs = [inputs.document_from_sections([[1, 14, 15], [16, 17], [254, 255, 256]], 850),
            inputs.document_from_sections([[700, 3], [1]], 721)]
    level, parent = _padded(docs, 851)
    say(f"[fp32 edges] tile {tile} d={D} windowed={windowed}")
    run_fwd_case(oracle, level, parent, 3, D, "f32", 31, tile=tile, windowed=windowed)
    run_bwd_case(oracle, level, parent, 3, D, "f32", 32, tile=tile, windowed=windowed)
    run_bwd_case(oracle, level, parent, 1, D, "f32", 33, tile=tile, windowed=windowed, edges=6)


@pytest.mark.parametrize("tile,D", [((128, 64), 64), ((64, 32), 128)])
def test_cross_few_visible_positions_at_tile_edges(oracle, tile, D):
    # the dK/dV pass works on the visible positions by rank: their number at and around the edges of a wave's 32 rows and
    # of the row tiles, one sample with two, and an encoder length that no zero-writing workgroup divides
    n_enc = 1217
    counts = (2, 32, 33, 127, 128, 129, 304)
    level = np.full((len(counts), n_enc), 3, np.int32)
    rng = np.random.default_rng(5)
    for b, c in enumerate(counts):
        level[b, rng.choice(n_enc, c, replace=False)] = 1
    say(f"[cross edges] {counts} of {n_enc} positions visible, tile {tile} d={D}")
    run_cross_case(oracle, level, 100, 2, 2, D, "bf16", 41, tile=tile, poison_invisible=True)


@pytest.mark.parametrize("tile,heads", [((128, 64), 10), ((128, 64), 11), ((64, 32), 12), ((64, 32), 13)])
def test_cross_few_visible_positions_d128_in_large_grids(oracle, tile, heads):
    # three roles per tile are 49 workgroups per head (84 on 64-row tiles): fewer and more than the 512 (1024) that are on the
    # chip at the same time; on 64 x 32 tiles dK and dV take one role where there are more
    n_enc = 1217
    counts = (2, 32, 33, 127, 128, 129, 304)
    level = np.full((len(counts), n_enc), 3, np.int32)
    rng = np.random.default_rng(7)
    for b, c in enumerate(counts):
        level[b, rng.choice(n_enc, c, replace=False)] = 1
    say(f"[cross edges] d=128, {heads} heads, tile {tile}")
    run_cross_case(oracle, level, 100, 2, heads, 128, "bf16", 43, tile=tile, poison_invisible=True)


@pytest.mark.parametrize("n_dec,n_enc,heads", [(60, 700, 1), (60, 700, 9), (700, 60, 9), (129, 1500, 17), (1500, 129, 17), (65, 4100, 3)])
def test_cross_backward_tiles_of_both_sides_and_the_longer_sides_rest(oracle, n_dec, n_enc, heads):
    # the grid of the backward's roles has two parts, each cut into equal shares by itself: the tiles that the decoder's and
    # the encoder's rows both have, and the rest of the longer side (the last case: lists cut into pieces, more dQ tiles)
    level = np.full((2, n_enc), 3, np.int32)
    level[1, n_enc // 2:] = -1
    for tile in ((128, 64), (64, 32)):
        for D in (64, 128):
            say(f"[cross edges] {n_dec} x {n_enc} x {heads} heads, tile {tile} d={D}")
            run_cross_case(oracle, level, n_dec, 8, heads, D, "bf16", 44, tile=tile)


def test_cross_select_on_long_encoders(oracle):
    # more than 8 groups of 64 positions per wave of the selecting workgroup, a ragged last group
    import paper_2407_08330_amd as hdt
    level = np.random.default_rng(6).integers(-1, 4, size=(3, 20011)).astype(np.int32)
    lay = hdt.hdt_build_cross_layout(to_dev_i32(level), 70, 4, tile_m=128, tile_n=64)
    assert lay.info()["compact_rows"] > 0
    for b in range(level.shape[0]):
        f_ref, t_ref = oracle.cross_schedule(level[b], 70, 4, 128, 64)
        _compare_schedule(lay, f_ref, b, "forward")
        _compare_schedule(lay.transposed(), t_ref, b, "transposed")


@pytest.mark.parametrize("heads", [1, 8, 9, 257, 514])
def test_every_row_tile_is_worked_on_whatever_their_number(oracle, heads):
    # the grid is cut into 8 equal shares per round: numbers of row tiles (1 and 2 per head) below, at and above them
    docs = [inputs.document_from_sections([[20, 40]], 70)]
    level, parent = _padded(docs, 70)
    for tile in ((128, 64), (64, 32)):
        say(f"[grid edges] {heads} heads, tile {tile}")
        run_fwd_case(oracle, level, parent, heads, 64, "bf16", 51, tile=tile)
        run_bwd_case(oracle, level, parent, heads, 128 if heads < 10 else 64, "bf16", 52, tile=tile)


@pytest.mark.parametrize("n", [1024, 2049, 33791, 33792, 70001])
def test_index_vectors_and_parents_across_workgroup_shares(oracle, n):
    # a workgroup takes a share of 1024 positions (more from 64 shares on) and counts siblings in LDS for 33 * 1024
    # parents at a time: lengths at those edges, roots whose virtual parent falls into the next window, siblings scattered
    # over all shares
    import paper_2407_08330_amd as hdt
    rng = np.random.default_rng(n)
    doc = inputs.pseudo_section_document(rng, n)[:2]
    forest = (np.where(rng.random(n) < 0.01, 0, 1).astype(np.int32), np.full(n, -1, np.int32))
    roots = np.flatnonzero(forest[0] == 0)
    forest[1][forest[0] == 1] = rng.choice(roots, size=int((forest[0] == 1).sum())) if roots.size else -1
    forest[0][rng.random(n) < 0.01] = -1
    level, parent = np.stack([doc[0], forest[0]]), np.stack([doc[1], np.where(forest[0] >= 0, forest[1], -1)])
    dead = parent >= 0
    dead[dead] = np.concatenate([level[b][parent[b][parent[b] >= 0]] < 0 for b in range(2)])
    parent[dead] = -1   # parents that became pads
    say(f"[hpe edges] n={n}")
    got = hdt.hdt_index_vectors(to_dev_i32(level), to_dev_i32(parent), 3).cpu().numpy()
    levels = np.stack([doc[0], rng.integers(-1, 6, size=n).astype(np.int32), np.full(n, 5, np.int32)])
    levels[2, 0], levels[2, -1] = 4, 3   # every position looks back to the first one; the last finds nothing
    par = hdt.hdt_parents_from_levels(to_dev_i32(levels)).cpu().numpy()
    for b in range(2):
        np.testing.assert_array_equal(got[b], oracle.index_vectors(level[b], parent[b], 3), err_msg=f"sample {b}")
    for b in range(2):
        np.testing.assert_array_equal(par[b], oracle.parents_from_levels(levels[b]), err_msg=f"levels {b}")
    assert (par[2, 1:-1] == 0).all() and par[2, 0] == -1 and par[2, -1] == -1


def _shuffled(level, parent, rng):
    n = level.shape[0]
    perm = rng.permutation(n)
    lv, pr = np.empty(n, np.int32), np.empty(n, np.int32)
    lv[perm] = level
    pr[perm] = np.where(parent >= 0, perm[np.maximum(parent, 0)], -1)
    return lv, pr


@pytest.mark.parametrize("bm,bn,n_keys", [(128, 64, 2048), (128, 64, 2049), (64, 32, 1024), (64, 32, 1025), (96, 96, 2016), (96, 96, 2017)])
def test_key_lists_at_the_length_that_fits_lds(oracle, bm, bn, n_keys):
    # a root and its children: every row sees every key, and a workgroup's lists (two of them on 64-row tiles) hold
    # exactly as many keys as stay in LDS, or one more
    import paper_2407_08330_amd as hdt
    level = np.ones((2, n_keys), np.int32)
    level[:, 0] = 0
    parent = np.zeros((2, n_keys), np.int32)
    parent[:, 0] = -1
    level[1], parent[1] = _shuffled(level[1], parent[1], np.random.default_rng(n_keys))
    lay = hdt.hdt_build_layout(to_dev_i32(level), to_dev_i32(parent), tile_m=bm, tile_n=bn)
    compare_layout(oracle, lay, level, parent, bm, bn)


@pytest.mark.parametrize("bm,bn", [(128, 64), (64, 32)])
@pytest.mark.parametrize("n", [8191, 8192, 8193, 8257])
@pytest.mark.parametrize("edges", [7, 6, 1])
def test_key_lists_around_a_wave_batch_of_positions(oracle, bm, bn, n, edges):
    # up to 8 groups of 64 positions per wave stay in registers (8192 positions); one more group, a ragged one; document
    # order and shuffled positions; directed masks (the two bitmaps of a tile differ)
    import paper_2407_08330_amd as hdt
    rng = np.random.default_rng(n)
    doc = inputs.pseudo_section_document(rng, n)[:2]
    pair = [doc, _shuffled(*doc, rng)]
    level, parent = np.stack([d[0] for d in pair]), np.stack([d[1] for d in pair])
    lay = hdt.hdt_build_layout(to_dev_i32(level), to_dev_i32(parent), tile_m=bm, tile_n=bn, edges=edges)
    compare_layout(oracle, lay, level, parent, bm, bn, edges=edges)


def test_buffer_cache_makes_room_for_the_sizes_in_use(oracle):
    # more sizes than the cache of destroyed layouts' buffers holds (16 blocks); the size built from then on stays cached: its
    # builds neither take nor give back device memory
    import torch
    import paper_2407_08330_amd as hdt
    wl = inputs.make_workload(1)
    for n in range(1024, 1024 + 20 * 4096, 4096):
        level = np.full((1, n), 1, np.int32)
        level[0, 0], parent = 0, np.zeros((1, n), np.int32)
        parent[0, 0] = -1
        hdt.hdt_build_layout(to_dev_i32(level), to_dev_i32(parent), tile_m=32, tile_n=32).destroy()
    ids = to_dev_i32(wl.level), to_dev_i32(wl.parent)
    hdt.hdt_build_layout(*ids).destroy()
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    for _ in range(5):
        lay = hdt.hdt_build_layout(*ids)
        assert torch.cuda.mem_get_info()[0] == free
        lay.destroy()
        assert torch.cuda.mem_get_info()[0] == free
    lay = hdt.hdt_build_layout(*ids)
    compare_layout(oracle, lay, wl.level, wl.parent, 128, 64)
    hdt.hdt_release_cached_memory()


@pytest.mark.parametrize("tile,heads", [((128, 64), 42), ((128, 64), 43), ((64, 32), 42), ((64, 32), 43)])
def test_bwd_d128_around_the_size_where_its_roles_change(oracle, tile, heads):
    # three roles per tile while 2048 waves hold them (512 workgroups of four, 1024 of two): 4 row tiles of 128 (8 of 64)
    # per head, 42 heads are 504 (1008) workgroups, 43 are 516 (1032) and take two roles
    level, parent = _padded([inputs.document_from_sections([[60, 50, 33], [80, 70, 41, 44], [30, 20, 48]], 500)], 500)
    say(f"[bwd edges] d=128, {heads} heads, tile {tile}")
    run_bwd_case(oracle, level, parent, heads, 128, "bf16", 61, tile=tile)
    run_bwd_case(oracle, level, parent, heads, 128, "bf16", 62, tile=tile, edges=6)


def test_directed_masks_both_schedules_from_one_launch(oracle):
    # the two builds of a directed mask share a launch: a guess of the arrays' sizes that is too small (many keys per row
    # after a small document) is made good, a capacity that is too small and invalid ids are refused, waiting or deferred
    import paper_2407_08330_amd as hdt
    wl = inputs.make_workload(1)
    n = 4096
    level, parent = np.ones((1, n), np.int32), np.zeros((1, n), np.int32)
    level[0, 0], parent[0, 0] = 0, -1
    for deferred in (False, True):
        hdt.hdt_build_layout(to_dev_i32(wl.level), to_dev_i32(wl.parent)).destroy()
        lay = hdt.hdt_build_layout(to_dev_i32(level), to_dev_i32(parent), edges=6, deferred=deferred)
        assert lay.status() >= 0
        compare_layout(oracle, lay, level, parent, 128, 64, edges=6)
        compare_layout(oracle, lay.transposed(), level, parent, 128, 64, edges=3)
    for name, ids, kw in (("HDT_ERR_SHAPE", (level, parent), dict(capacity=100)),
                          ("HDT_ERR_HIERARCHY", (level, np.where(parent < 0, -1, n).astype(np.int32)), {})):
        with pytest.raises(hdt.HdtError) as e:
            hdt.hdt_build_layout(to_dev_i32(ids[0]), to_dev_i32(ids[1]), edges=6, **kw)
        assert e.value.name == name and "deferred" not in str(e.value)
        lay = hdt.hdt_build_layout(to_dev_i32(ids[0]), to_dev_i32(ids[1]), edges=6, deferred=True, **kw)
        with pytest.raises(hdt.HdtError) as e:
            lay.status()
        assert e.value.name == name


@pytest.mark.parametrize("bm,bn", [(128, 64), (64, 32)])
@pytest.mark.parametrize("n", [4095, 4096, 4097])
@pytest.mark.parametrize("edges", [7, 6])
def test_key_lists_around_the_length_where_workgroups_grow(oracle, bm, bn, n, edges):
    # 512 threads per workgroup up to 4096 positions (one batch of 8 groups per wave), 1024 beyond, one schedule and two
    import paper_2407_08330_amd as hdt
    rng = np.random.default_rng(n)
    tree = inputs.listops_like_tree(rng, n)
    pair = [tree, _shuffled(*inputs.pseudo_section_document(rng, n)[:2], rng)]
    level, parent = np.stack([d[0] for d in pair]), np.stack([d[1] for d in pair])
    lay = hdt.hdt_build_layout(to_dev_i32(level), to_dev_i32(parent), tile_m=bm, tile_n=bn, edges=edges)
    compare_layout(oracle, lay, level, parent, bm, bn, edges=edges)
    if edges == 6:
        compare_layout(oracle, lay.transposed(), level, parent, bm, bn, edges=3)
