"""GPU parity: hierarchical positional encoding (index vectors, sinusoidal table, fused add) against the
oracle.  Index vectors are integers: bit-exact.  Table: float32 values of a double evaluation, 1e-6.
Add: fp32 1e-5; bf16 x is rounded once after the add: half an ulp at |x + HPE| < 8 is 1.6e-2 -> 2e-2."""
import numpy as np
import pytest

from paper_2407_08330_amd import inputs
from gpu_common import from_dev, say, to_dev_bf16, to_dev_i32

pytestmark = pytest.mark.gpu


def _index_vectors(level, parent, L):
    import paper_2407_08330_amd as hdt
    return hdt.hdt_index_vectors(to_dev_i32(level), to_dev_i32(parent), L).cpu().numpy()


def _check_index_vectors(oracle, level, parent, L):
    got = _index_vectors(level, parent, L)
    for b in range(level.shape[0]):
        np.testing.assert_array_equal(got[b], oracle.index_vectors(level[b], parent[b], L), err_msg=f"sample {b}")
    return got


@pytest.mark.parametrize("config", [1, 2, 3])
def test_index_vectors_on_benchmark_documents(oracle, config):
    wl = inputs.make_workload(config, batch=2)
    say(f"[hpe] index vectors, config {config} documents")
    _check_index_vectors(oracle, wl.level, wl.parent, 3)


def test_index_vectors_deep_trees_ragged_and_shuffled(oracle):
    rng = np.random.default_rng(8)
    for n in (1, 63, 1025, 3000, 4097, 9001):
        lv, pr = inputs.listops_like_tree(rng, n, max_nodes=max(1, n - 3))
        say(f"[hpe] ListOps-shaped tree n={n} depth {lv.max()}")
        _check_index_vectors(oracle, lv[None], pr[None], 20)
        _check_index_vectors(oracle, lv[None], pr[None], 4)       # deeper levels are cut
    # a document whose positions are shuffled (siblings scattered over the chunks) + an all-pad sample
    wl = inputs.make_workload(3, batch=1)
    n = wl.n_pos
    perm = rng.permutation(n)
    level = np.empty(n, np.int32)
    parent = np.empty(n, np.int32)
    level[perm] = wl.level[0]
    parent[perm] = np.where(wl.parent[0] >= 0, perm[np.maximum(wl.parent[0], 0)], -1)
    say("[hpe] shuffled positions + all-pad sample")
    lv = np.stack([level, np.full(n, -1, np.int32)])
    pr = np.stack([parent, np.full(n, -1, np.int32)])
    got = _check_index_vectors(oracle, lv, pr, 3)
    assert (got[1] == 0).all()


def test_index_vectors_forest_with_pads_in_front(oracle):
    level = np.array([[-1, 1, -1, 1, 2, 1]], np.int32)
    parent = np.array([[-1, -1, -1, -1, 3, -1]], np.int32)
    got = _check_index_vectors(oracle, level, parent, 2)
    assert got[0].tolist() == [[0, 0], [1, 0], [0, 0], [2, 0], [2, 1], [3, 0]]


def _parents(level):
    import paper_2407_08330_amd as hdt
    return hdt.hdt_parents_from_levels(to_dev_i32(level)).cpu().numpy()


@pytest.mark.parametrize("config", [1, 3])
def test_parents_from_levels_on_benchmark_documents(oracle, config):
    wl = inputs.make_workload(config)
    say(f"[hpe] parents from levels, config {config}: B={wl.batch} N={wl.n_pos}")
    got = _parents(wl.level)
    for b in range(wl.batch):
        np.testing.assert_array_equal(got[b], oracle.parents_from_levels(wl.level[b]), err_msg=f"sample {b}")
    np.testing.assert_array_equal(got, wl.parent)   # and the generator's own parents


def test_parents_from_levels_trees_ragged_lengths_and_odd_levels(oracle):
    rng = np.random.default_rng(77)
    for n in (1, 63, 64, 65, 1023, 1025, 3000):
        lv, _ = inputs.listops_like_tree(np.random.default_rng(n), n)
        # a second sample: random levels (a forest in no particular order), pads sprinkled in, and levels the
        # library does not know (they get no parent and are nobody's parent)
        rnd = rng.integers(-1, 6, size=n).astype(np.int32)
        rnd[rng.random(n) < 0.02] = 40
        rnd[rng.random(n) < 0.02] = -7
        level = np.stack([lv, rnd])
        say(f"[hpe] parents from levels, n={n}")
        got = _parents(level)
        np.testing.assert_array_equal(got[0], oracle.parents_from_levels(level[0]))
        known = np.where((rnd >= 0) & (rnd < 32), rnd, -1).astype(np.int32)
        np.testing.assert_array_equal(got[1], oracle.parents_from_levels(known))
    hand = np.array([[-1, 3, 0, 1, 2, -1, 3, 3, 1, 0, 2, 1, 3]], np.int32)
    np.testing.assert_array_equal(_parents(hand)[0], [-1, -1, -1, 2, 3, -1, 4, 4, 2, -1, 8, 9, 10])


def test_hpe_table(oracle):
    import paper_2407_08330_amd as hdt
    for rows, d in ((700, 768), (33, 64)):
        t = hdt.hdt_hpe_table(rows, d).cpu().numpy()
        ref = oracle.hpe(np.arange(rows, dtype=np.int32)[:, None], d)
        err = np.abs(t - ref).max()
        say(f"[hpe] table {rows}x{d}: max error {err:.2e}")
        assert err <= 1e-6


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("table_rows", [0, 40, 1024])
def test_hpe_add(oracle, dtype, table_rows):
    import torch
    import paper_2407_08330_amd as hdt
    wl = inputs.make_workload(3, batch=2)      # sample 0 holds the 600-token sentence: indices up to 600
    B, N, d, L = 2, wl.n_pos, 768, 3
    p = hdt.hdt_index_vectors(to_dev_i32(wl.level), to_dev_i32(wl.parent), L)
    rng = np.random.default_rng(77)
    x = rng.standard_normal((B, N, d), dtype=np.float32)
    if dtype == "bf16":
        x = inputs.round_to_bf16(x)
        x_dev = to_dev_bf16(x)
    else:
        x_dev = torch.from_numpy(x).cuda()
    table = hdt.hdt_hpe_table(table_rows, d) if table_rows else None
    hdt.hdt_hpe_add(p, table, x_dev)
    torch.cuda.synchronize()
    got = from_dev(x_dev)
    p_host = p.cpu().numpy()
    assert p_host.max() >= 600
    worst = 0.0
    for b in range(B):
        ref = x[b].astype(np.float64) + oracle.hpe(p_host[b], d)
        worst = max(worst, np.abs(got[b] - ref).max())
    tol = 2e-2 if dtype == "bf16" else 1e-5
    say(f"[hpe] add {dtype}, table rows {table_rows}: max error {worst:.2e} (tol {tol})")
    assert worst <= tol


@pytest.mark.parametrize("levels", [1, 2, 3, 4, 5])
def test_index_vectors_of_few_levels(oracle, levels):
    """The first columns of the vectors of a deep forest, for every number of levels with a kernel of its own."""
    import paper_2407_08330_amd as hdt
    n = 517
    level, parent = map(np.stack, zip(*(inputs.listops_like_tree(np.random.default_rng(b), n) for b in range(3))))
    level[1, 400:], parent[1, 400:] = -1, -1
    parent[1][parent[1] >= 400] = -1
    got = hdt.hdt_index_vectors(to_dev_i32(level), to_dev_i32(parent), levels).cpu().numpy()
    for b in range(3):
        np.testing.assert_array_equal(got[b], oracle.index_vectors(level[b], parent[b], 25)[:, :levels])


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("levels", [1, 2, 3, 4, 5, 9])
@pytest.mark.parametrize("n,d", [(1, 8), (2, 24), (63, 520), (130, 64)])
def test_hpe_add_levels_and_edges(oracle, dtype, levels, n, d):
    """Odd numbers of positions, channels that end inside a wave, groups of levels.  Inside the table the result is one rounding
    of fp32 sums in the order of the levels, the same bits in torch; with indices beyond it, the definition: up to 9 table values
    of error 1e-6 and 10 additions below 16 (2^-21 each)."""
    import torch
    import paper_2407_08330_amd as hdt
    rng = np.random.default_rng([levels, n, d])
    rows = 40
    table = hdt.hdt_hpe_table(rows, d)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    for beyond in (False, True):
        p = rng.integers(0, rows, (3, n, levels))
        p[:, 1::2][rng.random(p[:, 1::2].shape) < 0.5] = 7
        p[:, ::3] = 7  # rows that repeat, and that do not
        if beyond:
            p[rng.random(p.shape) < 0.02] = 600
            p[0, -1, -1] = 55
        x = torch.from_numpy(rng.standard_normal((3, n, d), dtype=np.float32)).cuda().to(dt)
        p_dev, got = to_dev_i32(p), x.clone()
        hdt.hdt_hpe_add(p_dev, table, got)
        if beyond:
            ref = x.double().cpu().numpy() + np.stack([oracle.hpe(q, d) for q in p])
            err = np.abs(got.double().cpu().numpy() - ref) - (np.abs(ref) * 2.0 ** -8 if dtype == "bf16" else 0)
            assert err.max() <= 9e-6 + 10 * 2.0 ** -21
        else:
            acc = torch.zeros((3, n, d), device="cuda")
            for l in range(levels):
                acc += table[p_dev[:, :, l].long()]
            assert torch.equal(got, (x.float() + acc).to(dt))


def test_index_vectors_of_trees_against_documents():
    """Trees put hundreds of runs into a chunk of positions, and every run looks at those in front of it; documents have a dozen.
    130 samples of 8192 positions: 4.4 times as long (115 us to 26.1), 5.6 (150 to 26.8) where the look is a branch that falls
    badly; the bound lies between the two."""
    import torch
    import paper_2407_08330_amd as hdt
    n, batch = 8192, 130

    def us(make):
        level, parent = (to_dev_i32(np.stack([x[b % 4] for b in range(batch)])) for x in zip(*(make(np.random.default_rng(b)) for b in range(4))))
        out = torch.empty((batch, n, 3), dtype=torch.int32, device="cuda")
        ws = torch.empty(hdt.load_library().hdt_index_vectors_workspace_bytes(batch, n), dtype=torch.uint8, device="cuda")
        begin, end = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        times = []
        for _ in range(8):
            begin.record()
            for _ in range(10):
                hdt.hdt_index_vectors(level, parent, 3, out=out, workspace=ws)
            end.record()
            end.synchronize()
            times.append(begin.elapsed_time(end) * 100)
        return min(times)

    assert us(lambda rng: inputs.listops_like_tree(rng, n)) < 5 * us(lambda rng: inputs.pseudo_section_document(rng, n, (10, 80))[:2])


def add_us(p, table, x):
    import torch
    import paper_2407_08330_amd as hdt
    begin, end = (torch.cuda.Event(enable_timing=True) for _ in range(2))
    times = []
    for _ in range(8):
        begin.record()
        for _ in range(10):
            hdt.hdt_hpe_add(p, table, x)
        end.record()
        end.synchronize()
        times.append(begin.elapsed_time(end) * 100)
    return min(times)


@pytest.mark.parametrize("rows", [0, 40])
def test_hpe_add_evaluates_a_repeated_index_once(rows):
    """Beyond the table a position's values take longer than everything else of the add, and positions come in pairs: with the
    indices of the first of a pair also in the second there is half as much to evaluate (four fifths of the time allowed)."""
    import torch
    import paper_2407_08330_amd as hdt
    n, d = 4096, 512
    x = torch.zeros((1, n, d), device="cuda")
    table = hdt.hdt_hpe_table(rows, d) if rows else None
    i = torch.arange(n, device="cuda", dtype=torch.int32)

    def us(p):
        p = (p + 50).view(1, n, 1).expand(1, n, 3).contiguous()
        return add_us(p, table, x)

    assert us(i // 2) < 0.8 * us(i)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_hpe_add_of_a_fifth_level_costs_a_level(dtype):
    """Five levels go through a form of their own; 1.3 (bf16) and 1.1 times as long as four, 1.9 and 1.35 where a form takes eight
    rows and half of the waves for them."""
    import torch
    import paper_2407_08330_amd as hdt
    n, d = 8192, 768
    x = torch.zeros((4, n, d), device="cuda", dtype=torch.bfloat16 if dtype == "bf16" else torch.float32)
    table = hdt.hdt_hpe_table(64, d)
    i = torch.arange(n, device="cuda", dtype=torch.int32)

    def us(levels):
        runs = [max(1, 400 // 5 ** l) for l in range(levels - 1)] + [1]
        return add_us(torch.stack([(i // r) % 60 for r in runs], dim=1).expand(4, n, levels).contiguous(), table, x)

    assert us(5) < (1.6 if dtype == "bf16" else 1.22) * us(4)


def test_hpe_argument_errors():
    import torch
    import paper_2407_08330_amd as hdt
    lv = torch.zeros((1, 64), dtype=torch.int32, device="cuda")
    with pytest.raises(hdt.HdtError) as e:
        hdt.hdt_index_vectors(lv, lv.clone() - 1, 0)
    assert e.value.name == "HDT_ERR_INVALID_ARG"
    with pytest.raises(hdt.HdtError) as e:
        hdt.hdt_index_vectors(lv, lv.clone() - 1, 3, workspace=torch.empty(16, dtype=torch.uint8, device="cuda"))
    assert e.value.name == "HDT_ERR_INVALID_ARG"
    with pytest.raises(hdt.HdtError) as e:
        hdt.hdt_hpe_table(4, 12)       # d_model not a multiple of 8
    assert e.value.name == "HDT_ERR_INVALID_ARG"


@pytest.mark.parametrize("n", [1000, 8192, 70001])
def test_parents_written_over_their_levels(oracle, n):
    # the caller has no more use for the levels and gives the same array for the parents
    import paper_2407_08330_amd as hdt
    rng = np.random.default_rng(n)
    level = np.stack([inputs.pseudo_section_document(rng, n)[0], rng.integers(-1, 6, size=n).astype(np.int32)])
    want = np.stack([oracle.parents_from_levels(lv) for lv in level])
    for _ in range(3):
        both = to_dev_i32(level)
        assert hdt.hdt_parents_from_levels(both, out=both) is both
        np.testing.assert_array_equal(both.cpu().numpy(), want)


@pytest.mark.parametrize("batch,n", [(1, 65537), (2, 66000), (40, 8000), (64, 5000), (65, 3073), (85, 3584)])
def test_parents_where_the_last_workgroups_of_a_sample_have_no_positions(oracle, batch, n):
    # chunks that do not divide evenly: the shares behind the last chunk are empty
    rng = np.random.default_rng(n)
    kinds = [inputs.pseudo_section_document(rng, n)[0], rng.integers(-1, 6, size=n).astype(np.int32)]
    want = [oracle.parents_from_levels(lv) for lv in kinds]
    got = _parents(np.stack([kinds[b % 2] for b in range(batch)]))
    for k, w in enumerate(want[:batch]):
        assert (got[k::2] == w[None]).all()


def _ordinals_walked_up(level, parent, L):
    """Index vectors of one sample in whole-array steps, for lengths the oracle takes minutes for."""
    n = level.shape[0]
    group = np.where((parent >= 0) & (parent < n), parent, n)
    group[level < 0] = n + 1 + np.arange(int((level < 0).sum()))   # pads are nobody's siblings
    order = np.argsort(group, kind="stable")
    first = np.r_[True, group[order][1:] != group[order][:-1]]
    rank = np.arange(n) - np.maximum.accumulate(np.where(first, np.arange(n), 0))
    ordinal = np.empty(n, np.int32)
    ordinal[order] = rank + 1
    p, at = np.zeros((n, L), np.int32), np.where(level >= 0, np.arange(n), -1)
    while (at >= 0).any():
        i = np.flatnonzero(at >= 0)
        l = level[at[i]]
        here = (l >= 1) & (l <= L)
        p[i[here], l[here] - 1] = ordinal[at[i[here]]]
        at[i] = parent[at[i]]
    return p


@pytest.mark.parametrize("batch,n", [(1, 2048), (15, 33791), (16, 33792), (17, 33792), (1, 131072), (1, 131073), (129, 2049), (257, 1025)])
def test_index_vectors_around_the_lines_between_their_kernels(oracle, batch, n):
    # several windows of parents: shares up to 16 samples and 131072 positions, one chain per sample beyond; and batches
    # that leave two shares and one per sample.  Documents, and runs of siblings whose parents lie anywhere in front
    import paper_2407_08330_amd as hdt
    rng = np.random.default_rng(n + batch)
    level, parent = (np.array(x) for x in inputs.pseudo_section_document(rng, n)[:2])
    run = rng.integers(1, 90, size=n)
    anchors = np.sort(rng.choice(n, n // 50, replace=False))
    anchors[0] = 0
    far_level = np.full(n, 2, np.int32)
    far_level[anchors] = 1
    far_level[rng.random(n) < 0.01] = -1
    far_level[0] = 0
    real = np.flatnonzero(far_level == 1)
    far_parent = np.repeat(rng.choice(real, size=n), run)[:n].astype(np.int32)
    far_parent[far_level == 1] = np.where(rng.random(int((far_level == 1).sum())) < 0.5, 0, -1)
    far_parent[(far_level < 0) | (np.arange(n) == 0)] = -1
    ids = [(level, parent), (far_level, far_parent)]
    got = hdt.hdt_index_vectors(to_dev_i32(np.stack([ids[b % 2][0] for b in range(batch)])),
                                to_dev_i32(np.stack([ids[b % 2][1] for b in range(batch)])), 3).cpu().numpy()
    for k, (lv, pr) in enumerate(ids[:batch]):
        want = _ordinals_walked_up(lv, pr, 3)
        if n <= 2049:
            np.testing.assert_array_equal(want, oracle.index_vectors(lv, pr, 3))
        assert (got[k::2] == want[None]).all(), f"{('document', 'parents anywhere')[k]}"


def test_index_vectors_take_time_in_proportion():
    # four times the positions of one document, and sixteen times the samples: at most twice that, and at most half that (a
    # batch fills the chip), in time
    import torch
    import paper_2407_08330_amd as hdt

    def ms(batch, n):
        level, parent = inputs.pseudo_section_document(np.random.default_rng(1), n)[:2]
        lv, pr = (to_dev_i32(np.tile(x, (batch, 1))) for x in (level, parent))
        out = torch.empty((batch, n, 3), dtype=torch.int32, device="cuda")
        times = []
        for _ in range(6):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(5):
                hdt.hdt_index_vectors(lv, pr, 3, out=out)
            b.record()
            torch.cuda.synchronize()
            times.append(a.elapsed_time(b) / 5)
        return min(times)

    long = ms(1, 1 << 18), ms(1, 1 << 20)
    wide = ms(32, 8192), ms(512, 8192)
    say(f"[hpe] index vectors: 2^18, 2^20 positions {long[0]:.3f}, {long[1]:.3f} ms; 32, 512 samples {wide[0]:.4f}, {wide[1]:.4f} ms")
    assert long[1] <= 8 * long[0] and wide[1] <= 8 * wide[0]
