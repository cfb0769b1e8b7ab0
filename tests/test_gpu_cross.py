"""GPU parity: decoder cross-attention over a level subset of the encoder positions (paper Sec. 4.2) against
the oracle: the two schedules bit-exact, forward and backward element by element (tolerances as for
self-attention: bf16 2e-2 on O and 5e-2 relative on gradients, fp32 1e-4)."""
import numpy as np
import pytest

from paper_2407_08330_amd import inputs
from gpu_common import GuardedWorkspace, busy, from_dev, say, to_dev_bf16, to_dev_i32

pytestmark = pytest.mark.gpu

SEC, SENT, TOK = 1 << 1, 1 << 2, 1 << 3


def _encoder_levels(n_enc, seeds):
    """Encoder documents with the benchmark's structure, padded to n_enc."""
    lv = []
    for s in seeds:
        l, _ = inputs.tree_document([(2, 6), (2, 9), (4, 30)], np.random.default_rng(s), max_nodes=n_enc - s % 7)
        lv.append(np.concatenate([l, np.full(n_enc - l.shape[0], -1, np.int32)]))
    return np.stack(lv)


def _long_encoder_levels(n_enc, seeds, fill=1.0):
    """Documents of sections of 3..10 sentences of 5..60 tokens that fill about `fill` of n_enc positions."""
    lv = []
    for s in seeds:
        rng = np.random.default_rng(s)
        sections, used = [], 1
        while True:
            sec = [int(x) for x in rng.integers(5, 61, size=int(rng.integers(3, 11)))]
            need = 1 + sum(1 + l for l in sec)
            if used + need > int(n_enc * fill):
                break
            sections.append(sec)
            used += need
        lv.append(inputs.document_from_sections(sections, n_enc)[0])
    return np.stack(lv)


def _compare_schedule(got_layout, ref, b, what):
    got = got_layout.export(b)
    assert "kperm" not in got
    np.testing.assert_array_equal(got["q_rowptr"], ref.q_rowptr, err_msg=f"{what} q_rowptr sample {b}")
    np.testing.assert_array_equal(got["q_keys"], ref.q_keys, err_msg=f"{what} q_keys sample {b}")
    np.testing.assert_array_equal(got["q_sub"], ref.q_sub, err_msg=f"{what} q_sub sample {b}")
    np.testing.assert_array_equal(got["bits"], ref.bits, err_msg=f"{what} bits sample {b}")
    ordinal = np.arange(ref.q_keys.shape[0]) - np.repeat(ref.q_rowptr[:-1], np.diff(ref.q_rowptr))
    np.testing.assert_array_equal(got["q_cols"], ordinal)
    assert got_layout.sample_info(b) == (ref.q_keys.shape[0], ref.nnz)


@pytest.mark.parametrize("bm,bn", [(128, 64), (64, 32), (32, 32), (96, 64)])
@pytest.mark.parametrize("level_mask", [SEC, SEC | SENT, SEC | SENT | TOK, 1 | SEC, 1 << 7])
def test_cross_schedules_bit_exact(oracle, bm, bn, level_mask):
    import paper_2407_08330_amd as hdt
    n_enc, n_dec = 1000, 333
    level = _encoder_levels(n_enc, (3, 4, 5))
    level[2, :] = -1 if level_mask == SEC else level[2, :]   # one sample without any visible position
    say(f"[cross layout] {bm}x{bn} level_mask={level_mask} visible {[int(oracle.cross_select(l, level_mask).size) for l in level]}")
    lay = hdt.hdt_build_cross_layout(to_dev_i32(level), n_dec, level_mask, tile_m=bm, tile_n=bn)
    info = lay.info()
    assert (info["n_pos"], info["n_kv"], info["cross"], info["cross_level_mask"]) == (n_dec, n_enc, 1, level_mask)
    tr = lay.transposed()
    assert tr is not None
    tinfo = tr.info()
    assert (tinfo["n_pos"], tinfo["n_kv"]) == (n_enc, n_dec)
    for b in range(level.shape[0]):
        f_ref, t_ref = oracle.cross_schedule(level[b], n_dec, level_mask, bm, bn)
        _compare_schedule(lay, f_ref, b, "forward")
        _compare_schedule(tr, t_ref, b, "transposed")
        assert lay.sample_info(b)[1] == tr.sample_info(b)[1]
    # a cross layout has no key order to export
    import ctypes
    buf = np.zeros(max(n_dec, n_enc), np.int32)
    status = hdt.load_library().hdt_layout_export(lay.handle, 0, ctypes.c_void_p(buf.ctypes.data), None, None, None,
                                                  None, None, None, None, None, 0)
    assert hdt.load_library().hdt_status_string(status) == b"HDT_ERR_UNSUPPORTED"


@pytest.mark.parametrize("B,n_enc,n_dec,share", [
    (1, 63, 1, 0.5), (2, 64, 33, 1.0),           # one group of 64 positions, ragged and whole
    (1, 4097, 65, 0.9), (2, 4160, 40, 0.02),     # 65 groups: the search for a key's group takes two steps
    (3, 9001, 130, 0.3),                         # keys of an entry in more than four groups, and in up to four
    (300, 70, 65, 0.4),                          # a workgroup per sample
    (129, 700, 1100, 0.3),                       # three per sample, in two rounds
    (1, 340001, 20, 0.004),                      # more LDS than a launch gets by default, groups without a key
])
def test_cross_build_of_one_launch_at_its_edges(oracle, B, n_enc, n_dec, share):
    import paper_2407_08330_amd as hdt
    level = np.where(np.random.default_rng(n_enc).random((B, n_enc)) < share, 1, 3).astype(np.int32)
    level[0, -1] = 1                              # the last position is visible
    lay = hdt.hdt_build_cross_layout(to_dev_i32(level), n_dec, SEC)
    for b in sorted({0, B // 2, B - 1}):
        f_ref, t_ref = oracle.cross_schedule(level[b], n_dec, SEC, 128, 64)
        _compare_schedule(lay, f_ref, b, "forward")
        _compare_schedule(lay.transposed(), t_ref, b, "transposed")


@pytest.mark.parametrize("tile", [(128, 64), (64, 32)])
def test_cross_backward_of_samples_with_different_counts(oracle, tile):
    """The schedule over the visible positions has room for a quarter of the encoder's rows per sample; its tiles keep their
    places whatever the largest sample takes: none, two and up to the quarter visible, and beyond it in one sample.  (Not one: P is
    1 then and dK zero in the oracle, where run_cross_case takes a row for a hidden one.)"""
    level = np.full((4, 2000), 3, np.int32)
    for b, visible in enumerate((0, 2, 129, 300)):
        level[b, np.random.default_rng(b).choice(2000, visible, replace=False)] = 1
    run_cross_case(oracle, level, 70, SEC, 2, 64, "bf16", 61, tile=tile, poison_invisible=True)
    level[3, :501] = 1
    run_cross_case(oracle, level, 70, SEC, 2, 64, "bf16", 62, tile=tile)


def test_cross_build_of_one_more_sample_than_fits():
    """129 samples have 256 compute units to be built on, as 128 have: 1.2 times as long, 1.8 with a workgroup per sample."""
    import torch
    import paper_2407_08330_amd as hdt

    def us(batch):
        level = to_dev_i32(np.where(np.random.default_rng(1).random((batch, 8192)) < 0.03, 1, 3))
        begin, end = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        times = []
        for _ in range(6):
            begin.record()
            for _ in range(20):
                hdt.hdt_build_cross_layout(level, 512, SEC).destroy()
            end.record()
            end.synchronize()
            times.append(begin.elapsed_time(end) * 50)
        return min(times)

    assert us(129) < 1.5 * us(128)


def _tensors(B, H, n_dec, n_enc, D, seed, dtype):
    import torch
    rng = np.random.default_rng(seed)
    xs = [rng.standard_normal((B, H, n, D)).astype(np.float32) for n in (n_dec, n_enc, n_enc, n_dec)]
    if dtype == "bf16":
        xs = [inputs.round_to_bf16(x) for x in xs]
        dev = [to_dev_bf16(x) for x in xs]
    else:
        dev = [torch.from_numpy(x).cuda() for x in xs]
    return xs, dev


def pieces_of(hdt, lay, H, D, tile_m):
    """Into how many pieces the library cuts the key lists of this layout for H heads (from the size of the
    forward workspace: partial O rows of D bf16 and a partial LSE per row)."""
    need = hdt.hdt_attn_fwd_workspace_bytes(lay, H, D, 0)
    if need == 0:
        return 1
    rows_per_piece = lay.batch * H * ((lay.n_pos + tile_m - 1) // tile_m) * tile_m
    for p in (2, 4, 8):
        rows = rows_per_piece * p
        if need == ((rows * D * 2 + 255) // 256 + (rows * 4 + 255) // 256) * 256:
            return p
    raise AssertionError(f"unexpected workspace size {need}")


def run_cross_case(oracle, level, n_dec, level_mask, H, D, dtype, seed, tile=(0, 0), backward=True, want_pieces=None,
                   poison_invisible=False):
    import torch
    import paper_2407_08330_amd as hdt
    B, n_enc = level.shape
    scale = 1.0 / np.sqrt(D)
    (q, k, v, d_o), (q_, k_, v_, do_) = _tensors(B, H, n_dec, n_enc, D, seed, dtype)
    if poison_invisible:
        # K, V rows of the encoder positions the decoder does not see (pads and levels outside the mask) hold NaN and
        # infinities on the device; the oracle keeps the finite values (it never reads those rows)
        hidden = np.stack([~np.isin(np.arange(n_enc), oracle.cross_select(l, level_mask)) for l in level])
        junk = np.random.default_rng(seed).choice(np.array([np.nan, np.inf, -np.inf], np.float32), size=(B, H, n_enc, D))
        w = np.broadcast_to(hidden[:, None, :, None], k.shape)
        kd, vd = np.where(w, junk, k), np.where(w, junk[..., ::-1], v)
        k_, v_ = (to_dev_bf16(x) if dtype == "bf16" else torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in (kd, vd))
    lay = hdt.hdt_build_cross_layout(to_dev_i32(level), n_dec, level_mask, tile_m=tile[0], tile_n=tile[1])
    # the dK/dV pass tiles the visible positions alone iff at most a quarter of the positions are visible
    c_max = max(int(oracle.cross_select(l, level_mask).size) for l in level)
    compact_rows = lay.info()["compact_rows"]
    say(f"    visible at most {c_max} of {n_enc}: compact rows {compact_rows}")
    assert (compact_rows > 0) == (0 < c_max and 4 * c_max <= n_enc) and (compact_rows == 0 or c_max <= compact_rows < c_max + 32)
    o_ = torch.full_like(q_, float("nan"))
    lse_ = torch.full((B, H, n_dec), float("nan"), dtype=torch.float32, device="cuda")
    # with a workspace the forward cuts long key lists into pieces (none for short lists or fp32)
    ws_bytes = hdt.hdt_attn_fwd_workspace_bytes(lay, H, D, 0 if dtype == "bf16" else 1)
    pieces = pieces_of(hdt, lay, H, D, tile[0] or 128) if dtype == "bf16" else 1
    say(f"    key lists in {pieces} piece(s), forward workspace {ws_bytes} bytes")
    assert want_pieces is None or pieces == want_pieces
    gws = GuardedWorkspace(ws_bytes) if ws_bytes else None   # exactly what the library asks for, a guard behind it
    ws = gws.view if gws else None
    hdt.hdt_attn_fwd(lay, q_, k_, v_, scale, o=o_, lse=lse_, workspace=ws)
    torch.cuda.synchronize()
    if gws:
        gws.check()
    if ws is not None:   # the same call without a workspace walks the whole lists: same result up to rounding
        o1, lse1 = hdt.hdt_attn_fwd(lay, q_, k_, v_, scale)
        torch.cuda.synchronize()
        assert np.abs(from_dev(o1) - from_dev(o_)).max() <= 2e-2
        fin = np.isfinite(lse1.cpu().numpy())
        assert np.array_equal(fin, np.isfinite(lse_.cpu().numpy()))
        assert np.abs(lse1.cpu().numpy()[fin] - lse_.cpu().numpy()[fin]).max() <= 1e-3
    o_ref, lse_ref = oracle.cross_attn_fwd(q, k, v, level, level_mask, scale)
    o_g, lse_g = from_dev(o_), lse_.cpu().numpy()
    tol_o, tol_l, tol_g = {"bf16": (2e-2, 1e-2, 5e-2), "f32": (1e-4, 1e-4, 1e-4)}[dtype]
    assert not np.isnan(o_g).any() and not np.isnan(lse_g).any()
    blind = np.array([oracle.cross_select(l, level_mask).size == 0 for l in level])
    assert (o_g[blind] == 0).all() and np.isneginf(lse_g[blind]).all()
    err_o = np.abs(o_g - o_ref).max()
    err_l = np.abs(lse_g[~blind] - lse_ref[~blind]).max() if (~blind).any() else 0.0
    say(f"    max|dO|={err_o:.3e} (tol {tol_o})  max|dLSE|={err_l:.3e} (tol {tol_l})")
    assert err_o <= tol_o and err_l <= tol_l
    if not backward:
        return
    dq_ = torch.full_like(q_, float("nan"))
    dk_ = torch.full_like(k_, float("nan"))
    dv_ = torch.full_like(k_, float("nan"))
    bws = GuardedWorkspace(hdt.hdt_attn_bwd_workspace_bytes(lay, H, D, 0 if dtype == "bf16" else 1))
    hdt.hdt_attn_bwd(lay, q_, k_, v_, o_, lse_, do_, scale, dq=dq_, dk=dk_, dv=dv_, workspace=bws.view)
    torch.cuda.synchronize()
    bws.check()
    ref = oracle.cross_attn_bwd(q, k, v, d_o, level, level_mask, scale)
    for name, g_dev, g_ref in zip(("dq", "dk", "dv"), (dq_, dk_, dv_), ref):
        g = from_dev(g_dev)
        assert not np.isnan(g).any(), f"{name}: unwritten or NaN rows"
        assert (g[g_ref == 0] == 0).all() or name == "dq", f"{name}: rows of invisible positions must be 0"
        denom = np.abs(g_ref).max()
        rel = np.abs(g - g_ref).max() / denom if denom > 0 else np.abs(g).max()
        say(f"    {name}: max-rel {rel:.3e} (tol {tol_g})")
        assert rel <= tol_g


@pytest.mark.parametrize("dtype,D", [("bf16", 64), ("bf16", 128), ("f32", 64)])
@pytest.mark.parametrize("level_mask", [SEC, SEC | SENT, SEC | SENT | TOK], ids=["sec", "sec+sent", "sec+sent+tokens"])
def test_cross_attention_ragged(oracle, dtype, D, level_mask):
    level = _encoder_levels(1000, (13, 14))
    say(f"[cross] n_enc=1000 n_dec=333 {dtype} d={D} level_mask={level_mask}")
    run_cross_case(oracle, level, 333, level_mask, 3, D, dtype, 700 + level_mask)


@pytest.mark.parametrize("tile", [(64, 32), (128, 64)], ids=["64x32", "128x64"])
def test_cross_attention_both_tile_shapes_and_blind_sample(oracle, tile):
    level = _encoder_levels(777, (23, 24, 25))
    level[1, :] = -1   # all pads: nothing visible for sample 1
    say(f"[cross] tile {tile}: n_enc=777 n_dec=130, a sample without visible positions")
    run_cross_case(oracle, level, 130, SEC | SENT, 2, 64, "bf16", 801, tile=tile)
    run_cross_case(oracle, level, 1, SEC | SENT | TOK, 2, 128, "bf16", 802, tile=tile)


@pytest.mark.parametrize("D", [64, 128])
def test_cross_attention_more_decoder_rows_than_encoder_positions(oracle, D):
    # more row tiles on the decoder side than on the encoder side: the backward's leftover workgroups are dQ roles
    level = _encoder_levels(150, (33, 34))
    say(f"[cross] n_enc=150 n_dec=1000 d={D}")
    run_cross_case(oracle, level, 1000, SEC | SENT | TOK, 2, D, "bf16", 850 + D)
    run_cross_case(oracle, level, 1000, SEC, 2, D, "bf16", 860 + D, tile=(64, 32))


def test_cross_attention_benchmark_documents(oracle):
    # the encoder side of the benchmark's 8192-position batch; 512 decoder rows (section-level summaries)
    wl = inputs.make_workload(4)
    for level_mask in (SEC, SEC | SENT, SEC | SENT | TOK):
        say(f"[cross] config 4 documents, n_dec=512, level_mask={level_mask}: visible "
            f"{[int(oracle.cross_select(l, level_mask).size) for l in wl.level]}")
        run_cross_case(oracle, wl.level, 512, level_mask, 4, 64, "bf16", 900 + level_mask)


@pytest.mark.parametrize("D", [64, 128])
def test_cross_attention_long_key_lists_cut_into_pieces(oracle, D):
    # the regular tokens visible and few decoder rows: a handful of row tiles with lists of dozens of entries, which
    # the library cuts into pieces walked by separate workgroups (forward with a workspace; dQ role of the backward)
    level = _long_encoder_levels(5000, (43,))
    say(f"[cross] n_enc=5000 n_dec=100, tokens visible, d={D}: 8 pieces")
    run_cross_case(oracle, level, 100, SEC | SENT | TOK, 2, D, "bf16", 950 + D, want_pieces=8)
    level = _long_encoder_levels(3000, (44, 45))
    level[1, 1500:] = -1   # the second sample sees half as much: its later pieces are empty
    say(f"[cross] n_enc=3000 n_dec=333 (a ragged last row tile), tokens visible, d={D}: 4 pieces")
    run_cross_case(oracle, level, 333, SEC | SENT | TOK, 3, D, "bf16", 960 + D, want_pieces=4)
    say(f"[cross] the same at 64x32 tiles")
    run_cross_case(oracle, level, 333, SEC | SENT | TOK, 3, D, "bf16", 970 + D, tile=(64, 32))
    # short lists, and fp32: nothing to cut
    run_cross_case(oracle, _encoder_levels(600, (46,)), 100, SEC | SENT | TOK, 2, D, "bf16", 980 + D, want_pieces=1)
    run_cross_case(oracle, _long_encoder_levels(3000, (47,)), 64, SEC | SENT | TOK, 1, D, "f32", 990 + D, want_pieces=1, backward=False)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_cross_attention_ignores_what_invisible_rows_hold(oracle, dtype):
    # pads in front and behind, NaN / Inf in every K, V row the level mask hides: anchors only (the dK/dV pass tiles the
    # visible rows alone), and everything but [DOC] (it tiles the encoder rows, hidden ones among them)
    level = _long_encoder_levels(1536, (51, 52), fill=0.8)
    level = np.concatenate([np.full((2, 40), -1, np.int32), level[:, :-40]], axis=1)
    for level_mask in (SEC | SENT, SEC | SENT | TOK):
        say(f"[cross] NaN/Inf in hidden K, V rows, level_mask={level_mask}, {dtype}")
        run_cross_case(oracle, level, 200, level_mask, 2, 64, dtype, 1000 + level_mask, poison_invisible=True)


@pytest.mark.parametrize("n_enc", [3, 4, 1000, 2000])
@pytest.mark.parametrize("level_mask", [SEC, SEC | SENT | TOK, 1 << 7], ids=["sec", "tokens", "nothing"])
def test_cross_build_waits_for_nothing(n_enc, level_mask):
    """Build, forward and backward enqueued behind tens of milliseconds of other work: the build and a forward without a workspace
    come back while that still runs, and whichever call is the first to depend on the number of visible positions, the results
    are the same, bit for bit, as with a layout whose count has been read (few positions visible and a schedule over those alone,
    many, none; lengths with room for such a schedule and without)."""
    import torch
    import paper_2407_08330_amd as hdt
    B, H, n_dec, D = 2, 3, 70, 64
    level = np.full((B, n_enc), 3, np.int32)
    level[:, ::17] = 1
    level[1, n_enc - 1] = -1
    lv = to_dev_i32(level)
    g = torch.Generator(device="cuda")
    g.manual_seed(n_enc)
    q, d_o = (torch.randn((B, H, n_dec, D), device="cuda", generator=g).to(torch.bfloat16) for _ in range(2))
    k, v = (torch.randn((B, H, n_enc, D), device="cuda", generator=g).to(torch.bfloat16) for _ in range(2))
    lay = hdt.hdt_build_cross_layout(lv, n_dec, level_mask)
    rows = lay.info()["compact_rows"]
    visible = int((((level >= 0) & ((level_mask >> np.maximum(level, 0)) & 1 == 1)).sum(axis=1)).max())
    assert (rows > 0) == (0 < visible and 4 * visible <= n_enc)
    room = [hdt.hdt_attn_fwd_workspace_bytes(lay, H, D, 0), hdt.hdt_attn_bwd_workspace_bytes(lay, H, D, 0)]
    assert (room[0] > 0) == (n_enc >= 1000 and level_mask == SEC | SENT | TOK)     # lists of 16 entries and more are cut
    ws = torch.empty(max(room[0], 1 << 20), dtype=torch.uint8, device="cuda")
    o, lse = hdt.hdt_attn_fwd(lay, q, k, v, 0.125)
    want = [o, lse, *hdt.hdt_attn_fwd(lay, q, k, v, 0.125, workspace=ws), *hdt.hdt_attn_bwd(lay, q, k, v, o, lse, d_o, 0.125)]
    for first in ("backward", "forward with a workspace", "forward's query", "backward's query", "status"):
        running = busy()
        late = hdt.hdt_build_cross_layout(lv, n_dec, level_mask)
        got = [*hdt.hdt_attn_fwd(late, q, k, v, 0.125)]
        assert not running.query(), "the build or the forward waited for its number of visible positions"
        grads = hdt.hdt_attn_bwd(late, q, k, v, *got, d_o, 0.125) if first == "backward" else None
        if first == "forward's query":
            assert hdt.hdt_attn_fwd_workspace_bytes(late, H, D, 0) == room[0]
        if first == "backward's query":
            assert hdt.hdt_attn_bwd_workspace_bytes(late, H, D, 0) == room[1]
        if first == "status":
            assert late.status() == 0
        got += hdt.hdt_attn_fwd(late, q, k, v, 0.125, workspace=ws)
        assert running.query(), "the first call that depends on it had not waited"
        got += grads or hdt.hdt_attn_bwd(late, q, k, v, got[0], got[1], d_o, 0.125)
        late.destroy()
        torch.cuda.synchronize()
        for x, y in zip(got, want):
            assert torch.equal(x.view(torch.int16), y.view(torch.int16))


@pytest.mark.parametrize("tile,n_enc,n_dec,every,heads", [
    ((128, 64), 8192, 500, 1, 4), ((64, 32), 8192, 250, 1, 3),      # long lists of keys, cut into pieces
    ((128, 64), 2048, 500, 4, 65), ((64, 32), 2048, 250, 4, 48),    # a schedule over the visible positions
    ((128, 64), 1000, 300, 2, 84), ((64, 32), 500, 100, 2, 193)])    # neither
def test_cross_bwd_is_the_same_on_both_sides_of_the_line_where_the_roles_compute_d(tile, n_enc, n_dec, every, heads):
    """With `heads` heads the roles compute D, with one more a pass of its own does: the heads that both calls have come out the
    same, bit for bit."""
    import torch
    import paper_2407_08330_amd as hdt
    level = np.full((1, n_enc), 3, np.int32)
    level[:, ::every] = 1
    level[0, -5:] = -1
    lay = hdt.hdt_build_cross_layout(to_dev_i32(level), n_dec, SEC, tile_m=tile[0], tile_n=tile[1])
    g = torch.Generator(device="cuda")
    g.manual_seed(n_enc + n_dec)
    more = heads + 1
    q, d_o = (torch.randn((1, more, n_dec, 64), device="cuda", generator=g).to(torch.bfloat16) for _ in range(2))
    k, v = (torch.randn((1, more, n_enc, 64), device="cuda", generator=g).to(torch.bfloat16) for _ in range(2))
    o, lse = hdt.hdt_attn_fwd(lay, q, k, v, 0.125)
    results = []
    hdt.hdt_timing_enable(True)
    try:
        for h, d_pass in ((heads, False), (more, True)):
            hdt.hdt_timing_reset()
            results.append(hdt.hdt_attn_bwd(lay, *(x[:, :h].contiguous() for x in (q, k, v, o, lse, d_o)), 0.125))
            torch.cuda.synchronize()
            assert ("hdt_bwd_delta_d64" in hdt.hdt_timing_read()) == d_pass
    finally:
        hdt.hdt_timing_enable(False)
    for x, y in zip(*results):
        assert torch.equal(x.view(torch.int16), y[:, :heads].contiguous().view(torch.int16))


@pytest.mark.parametrize("tile", [(128, 64), (64, 32)], ids=["128x64", "64x32"])
def test_cross_bwd_has_a_d_pass_where_lists_are_longer_than_eight_entries(tile):
    import torch
    import paper_2407_08330_amd as hdt
    for n_dec, d_pass in ((8 * tile[1], False), (8 * tile[1] + 1, True)):
        lay = hdt.hdt_build_cross_layout(to_dev_i32(np.ones((1, 300), np.int32)), n_dec, SEC, tile_m=tile[0], tile_n=tile[1])
        q, d_o = (torch.randn((1, 2, n_dec, 64), device="cuda").to(torch.bfloat16) for _ in range(2))
        k, v = (torch.randn((1, 2, 300, 64), device="cuda").to(torch.bfloat16) for _ in range(2))
        o, lse = hdt.hdt_attn_fwd(lay, q, k, v, 0.125)
        hdt.hdt_timing_enable(True)
        try:
            hdt.hdt_timing_reset()
            hdt.hdt_attn_bwd(lay, q, k, v, o, lse, d_o, 0.125)
            assert ("hdt_bwd_delta_d64" in hdt.hdt_timing_read()) == d_pass
        finally:
            hdt.hdt_timing_enable(False)


def test_cross_calls_captured_on_a_layout_that_many_builds_have_followed():
    """The number of visible positions is asked for while a graph is being captured, where nothing may be waited for on the
    device, and more than a thousand builds after the one that reported it."""
    import torch
    import paper_2407_08330_amd as hdt
    level = to_dev_i32(_long_encoder_levels(2048, (7,)))
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    q, d_o = (torch.randn((1, 2, 100, 64), device="cuda", generator=g).to(torch.bfloat16) for _ in range(2))
    k, v = (torch.randn((1, 2, 2048, 64), device="cuda", generator=g).to(torch.bfloat16) for _ in range(2))
    for level_mask in (SEC, SEC | SENT | TOK):
        known = hdt.hdt_build_cross_layout(level, 100, level_mask)
        room = [torch.empty(max(need, 16), dtype=torch.uint8, device="cuda")
                for need in (hdt.hdt_attn_fwd_workspace_bytes(known, 2, 64, 0), hdt.hdt_attn_bwd_workspace_bytes(known, 2, 64, 0))]
        o, lse = hdt.hdt_attn_fwd(known, q, k, v, 0.125, workspace=room[0])
        want = [o, lse, *hdt.hdt_attn_bwd(known, q, k, v, o, lse, d_o, 0.125, workspace=room[1])]
        lay = hdt.hdt_build_cross_layout(level, 100, level_mask)
        for _ in range(1030):
            hdt.hdt_build_cross_layout(level, 100, SEC).destroy()
        got = [torch.empty_like(x) for x in want]
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            hdt.hdt_attn_fwd(lay, q, k, v, 0.125, o=got[0], lse=got[1], workspace=room[0])
            hdt.hdt_attn_bwd(lay, q, k, v, got[0], got[1], d_o, 0.125, *got[2:], workspace=room[1])
        for _ in range(3):
            for x in got:
                x.fill_(float("nan"))
            graph.replay()
            torch.cuda.synchronize()
            for x, y in zip(got, want):
                assert torch.equal(x.view(torch.int16), y.view(torch.int16))


def test_cross_builds_in_flight_by_the_hundreds_keep_their_reports_apart():
    """More builds than report words are made at a time, none of which has run when the last one is enqueued, some destroyed before
    that, on two streams: every layout gets its own number of visible positions, and so do those that take the words next."""
    import torch
    import paper_2407_08330_amd as hdt
    n_enc = 1024
    level = np.full((600, 1, n_enc), 3, np.int32)
    for i in range(600):
        level[i, 0, :1 + i % 250] = 1
    lv = to_dev_i32(level.reshape(600, n_enc)).view(600, 1, n_enc)
    other = torch.cuda.Stream()
    torch.cuda.synchronize()
    for _ in range(2):
        running = busy()
        other.wait_event(running)
        lays = []
        for i in range(600):
            lay = hdt.hdt_build_cross_layout(lv[i], 64, SEC, stream=other if i % 3 == 1 else None)
            lays.append(None if i % 3 == 2 else lay)     # (a third of them is destroyed here)
            del lay
        assert not running.query(), "the builds had reported: nothing was tested"
        for i, lay in enumerate(lays):
            if lay is not None:
                assert lay.status() == 0
        for i, lay in enumerate(lays):
            if lay is not None:
                assert lay.info()["compact_rows"] == (1 + i % 250 + 31) // 32 * 32
                lay.destroy()


def test_cross_layouts_of_a_decoder_stay_in_the_buffer_cache():
    """Four layouts at a time, built and destroyed step by step (a decoder with several settings of what it sees): the cache
    holds the buffers of all four, and none goes back to the system, which would wait for the device."""
    import torch
    import paper_2407_08330_amd as hdt
    level = to_dev_i32(_long_encoder_levels(8192, (1, 2)))
    torch.cuda.synchronize()
    hdt.hdt_release_cached_memory()
    free = []
    for _ in range(3):
        lays = [hdt.hdt_build_cross_layout(level, 512, m) for m in (SEC, SENT, SEC | SENT, SEC | SENT | TOK)]
        torch.cuda.synchronize()
        free.append(torch.cuda.mem_get_info()[0])
        for lay in lays:
            lay.destroy()
        free.append(torch.cuda.mem_get_info()[0])
    hdt.hdt_release_cached_memory()
    assert torch.cuda.mem_get_info()[0] > free[0]
    assert len(set(free)) == 1, free


def test_cross_argument_errors():
    import torch
    import paper_2407_08330_amd as hdt
    level = to_dev_i32(_encoder_levels(256, (1,)))
    with pytest.raises(hdt.HdtError) as e:
        hdt.hdt_build_cross_layout(level, 64, SEC, tile_m=48)
    assert e.value.name == "HDT_ERR_UNSUPPORTED"
    with pytest.raises(hdt.HdtError) as e:
        hdt.hdt_build_cross_layout(level, -1, SEC)
    assert e.value.name == "HDT_ERR_INVALID_ARG"
    lay = hdt.hdt_build_cross_layout(level, 64, SEC)
    q = torch.zeros((1, 2, 64, 64), dtype=torch.bfloat16, device="cuda")
    with pytest.raises(ValueError):
        hdt.hdt_attn_fwd(lay, q, q.clone(), q.clone(), 0.1)   # k, v must have the encoder's length
    for n_enc, n_dec in ((0, 64), (256, 0)):   # both sides need rows
        lv = torch.zeros((1, n_enc), dtype=torch.int32, device="cuda")
        with pytest.raises(hdt.HdtError) as e:
            hdt.hdt_build_cross_layout(lv, n_dec, 1)
        assert e.value.name == "HDT_ERR_SHAPE"
    lay0 = hdt.hdt_build_cross_layout(torch.zeros((0, 256), dtype=torch.int32, device="cuda"), 64, 1)
    assert lay0.info()["n_tiles"] == 0 and lay0.transposed().info()["n_tiles"] == 0
