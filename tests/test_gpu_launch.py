"""GPU checks of what changes the render kernel's speed but never its result:
the tile order (stripes of tiles per XCD), the early-termination path (rays
evaluated front to back in rounds, stopped rays dropped), the 16-byte block
gathers of x-neighbour corner pairs on the finest levels, the profiling
builds that time the kernel's phases, and the gather-replay microbenchmark
that measures the floor of its gather stream.

  - every tile order renders the same frame bit for bit, and every pixel;
  - the work counters are back at zero after every launch, whatever the
    kernel and grid size of the next one, and two contexts (each with its
    own counters) render on two streams at once;
  - the early-termination path renders the tile path's frame bit for bit
    (the same samples composited in the same order), at every round size,
    and evaluates fewer samples on opaque content;
  - block gathers on any set of finest levels render the same frame bit for
    bit as single-entry gathers;
  - the phase-timer build renders the same frame as the library, and its
    counters cover every tile of every launch;
  - the replay loads exactly the table entries of the oracle's corner
    indices for the frame's own sample positions (the XOR of everything it
    loads equals the XOR of those entries, which does not depend on which
    lane loaded what).
"""
import numpy as np
import pytest

import oracle
from paper_2312_11841_amd import mixrt, synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)


def _render(ds, **kw):
    r = mixrt.Renderer(0, sync_check=True, **kw)
    out = torch.full((ds.rays, 4), float("nan"), dtype=torch.float32, device="cuda:0")
    r.render(ds, out)
    shape = r.launch_shape(ds)
    r.sync()
    r.close()
    return out.cpu().numpy(), shape


ORDER_CFGS = [
    synth.VIEW720P_DENSE,
    synth.PAPER720P,
    synth.TINY64_DENSE.replace(name="ragged_views", H=37, W=53, views=3, K=8, gbuf="iid"),
    synth.TINY64_DENSE.replace(name="ragged_k1", H=29, W=71, views=2, K=1, gbuf="iid"),
    synth.TINY64_DENSE.replace(name="ragged_k3", H=23, W=37, views=2, K=3, gbuf="iid"),
]


@pytest.mark.parametrize("cfg", ORDER_CFGS, ids=lambda c: c.name)
def test_tile_order_never_changes_a_pixel(cfg):
    say("tile order", cfg.name)
    sc = synth.make_scene(cfg)
    ds = mixrt.DeviceScene.from_scene(sc, "cuda:0")
    ref, (_, default_stripe) = _render(ds, tile_stripe=-1)
    assert np.all(np.isfinite(ref))
    R = 64 // cfg.K
    seen = {default_stripe}
    for stripe in (1, 2, 3, 8, 16, 37, 1 << 20, 0):
        got, (blocks, st) = _render(ds, tile_stripe=stripe)
        seen.add(st)
        assert np.array_equal(got, ref), (stripe, st)
        for b in ("two", "full"):
            got, _ = _render(ds, tile_stripe=stripe, blocks=b)
            assert np.array_equal(got, ref), (stripe, b)
    say(f"  stripes launched: {sorted(seen)} (tiles of {R} rays)")


def test_work_counters_are_ready_for_every_launch():
    """One context renders frames of different kernels and grid sizes in turn
    (a queue-kernel frame, a ragged frame, a one-sample frame on the tile
    kernel, a frame of 25 tiles on 7 blocks, so in one pool, and a frame
    whose plan takes every unit in the fixed order), twice over: the pools'
    counters, left at zero by each launch's last blocks, give every later
    launch the same frame as a fresh context's first launch."""
    cfgs = [synth.VIEW720P, ORDER_CFGS[4], synth.PAPER720P,
            synth.TINY64_DENSE.replace(name="one_pool", H=5, W=37, views=1, K=8, gbuf="iid"),
            _table3("tab3_L1_T17")]
    scenes = [mixrt.DeviceScene.from_scene(synth.make_scene(c), "cuda:0") for c in cfgs]
    refs = [_render(ds)[0] for ds in scenes]
    r = mixrt.Renderer(0, sync_check=True)
    try:
        for rep in range(2):
            for cfg, ds, ref in zip(cfgs, scenes, refs):
                plan = r.launch_plan(ds)
                say("counters", rep, cfg.name, plan)
                if cfg.name == "one_pool":
                    assert plan["blocks"] == 7
                assert plan["claims"] == (0 if cfg.name == "tab3_L1_T17" else 1)
                out = torch.full((ds.rays, 4), float("nan"), dtype=torch.float32,
                                 device="cuda:0")
                r.render(ds, out)
                r.sync()
                assert np.array_equal(out.cpu().numpy(), ref), (rep, cfg.name)
    finally:
        r.close()


def test_contexts_on_two_streams_render_at_once():
    """Two contexts, each with its own work counters, render on two streams
    at the same time (launches alternate between the streams with no wait in
    between): every frame equals a lone context's."""
    cfgs = [synth.VIEW720P, synth.PAPER720P]
    scenes = [mixrt.DeviceScene.from_scene(synth.make_scene(c), "cuda:0") for c in cfgs]
    refs = [_render(ds)[0] for ds in scenes]
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    rs = [mixrt.Renderer(0, stream=st) for st in streams]
    outs = [[torch.full((ds.rays, 4), float("nan"), dtype=torch.float32, device="cuda:0")
             for _ in range(3)] for ds in scenes]
    try:
        torch.cuda.synchronize()
        for rep in range(3):
            for r, ds, o in zip(rs, scenes, outs):
                r.render(ds, o[rep])
        torch.cuda.synchronize()
        for cfg, ref, o in zip(cfgs, refs, outs):
            for rep in range(3):
                say("two streams", cfg.name, rep)
                assert np.array_equal(o[rep].cpu().numpy(), ref), (cfg.name, rep)
    finally:
        for r in rs:
            r.close()


def test_tile_order_spot_check_against_the_oracle():
    cfg = ORDER_CFGS[2]
    sc = synth.make_scene(cfg)
    ds = mixrt.DeviceScene.from_scene(sc, "cuda:0")
    got, _ = _render(ds, tile_stripe=3)
    ref = oracle.OracleScene(sc).render_pixels(np.arange(cfg.rays), threads=oracle.max_threads())
    assert np.abs(got - ref).max() <= 2e-3


@pytest.mark.parametrize("cfg", [synth.VIEW720P, synth.PAPER720P], ids=lambda c: c.name)
def test_phase_timer_build_renders_the_same_frame(cfg):
    say("timer build", cfg.name)
    sc = synth.make_scene(cfg)
    ds = mixrt.DeviceScene.from_scene(sc, "cuda:0")
    ref, (blocks, stripe) = _render(ds)
    r = mixrt.Renderer(0, sync_check=True, variant="timer")
    r.phase_cycles(reset=True)
    out = torch.full((ds.rays, 4), float("nan"), dtype=torch.float32, device="cuda:0")
    for _ in range(3):
        r.render(ds, out)
    ph = r.phase_cycles(reset=True)
    assert r.launch_shape(ds) == (blocks, stripe)
    r.close()
    assert np.array_equal(out.cpu().numpy(), ref)
    R = 64 // cfg.K
    say("  ", ph)
    assert ph["waves"] == 3 * blocks * 4
    assert ph["tiles"] == 3 * ds.rays // R   # whole tiles: W and H are multiples of the tile's
    assert all(ph[k] > 0 for k in ("setup", "hash", "mlp", "composite"))


def test_default_library_has_no_phase_timer():
    r = mixrt.Renderer(0)
    with pytest.raises(mixrt.MixrtError) as e:
        r.phase_cycles()
    assert e.value.status == mixrt.MIXRT_EUNSUPPORTED
    r.close()


@pytest.mark.parametrize("cfg", [synth.TINY64_DENSE.replace(name="replay_tiny", H=40, W=56),
                                 synth.VIEW720P.replace(name="replay_720p_rows", rows=48),
                                 synth.DEPLOYED720P.replace(name="replay_f4", rows=64),
                                 synth.TABLE3[0].replace(name="replay_f4_L8", rows=48),
                                 synth.TABLE3[0].replace(name="replay_f4_ragged", H=23, W=37,
                                                         views=2, K=3, gbuf="iid", delta=0.5,
                                                         log2_T=12)],
                         ids=lambda c: c.name)
def test_gather_replay_loads_exactly_the_corner_entries(cfg):
    from paper_2312_11841_amd import microbench as mb
    say("gather replay", cfg.name)
    sc = synth.make_scene(cfg)
    ds = mixrt.DeviceScene.from_scene(sc, "cuda:0")
    r = mixrt.Renderer(0, sync_check=True)
    x, hit = r.ray_setup(ds)
    blocks, stripe = r.launch_shape(ds)
    r.sync()
    N = np.ascontiguousarray(mixrt.level_resolutions(ds.grid), np.int32)
    # the XOR over every lane's fold is the XOR over all loaded words,
    # whichever lane loaded them
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    for grid in (blocks, 2 * cus):
        for st in (stripe, 1):
            res = mb.gather_replay(x, hit, cfg.views, cfg.W, cfg.rows_kept, cfg.K, ds.table, N,
                                   st, [grid], reps=1)
            assert res["best"]["ms"] > 0
    xs = x.cpu().numpy().reshape(-1, cfg.K, 3)[hit.cpu().numpy() != 0].reshape(-1, 3)
    _, idx, _, _ = oracle.hash_encode(xs, sc.table, cfg.N_min, cfg.N_max)
    words = sc.table.view(np.uint32).reshape(cfg.L, cfg.T, -1)      # an entry's 32-bit words
    acc = np.uint32(0)
    for l in range(cfg.L):
        w = words[l][idx[:, l, :].reshape(-1)]
        acc ^= np.bitwise_xor.reduce(w.reshape(-1))
    # the tile path's order and every rounds order the render can take, with
    # the render's 16-byte block gathers on none, the library's choice, all
    # hashed levels (4- and 8-byte entries; 16-byte ones ignore it)
    plan = r.launch_plan(ds)
    n_dense = int(sum((N.astype(np.int64) + 1) ** 3 <= cfg.T))
    # one work buffer for every call: each call leaves its counters at zero
    work = torch.zeros(mb.WORK_WORDS, dtype=torch.int32, device="cuda:0")
    for block_from in sorted({cfg.L, plan["block_from"], n_dense, 0, max(cfg.L - 3, 0)}):
        for batch in (2, 4):
            # rounds of a power of two samples, as the render takes them
            for chunk in sorted({c for c in (0, 1, cfg.K // 2, cfg.K) if c & (c - 1) == 0}):
              for claims in (True, False):
                sink = torch.zeros(blocks * 256, dtype=torch.int32, device="cuda:0")
                rc = mb.lib().mixrt_mb_gather_replay(
                    x.data_ptr(), hit.data_ptr(), cfg.views, cfg.W, cfg.rows_kept, cfg.K,
                    ds.table.data_ptr(), cfg.L, cfg.log2_T, ds.table.element_size() * cfg.F,
                    N.ctypes.data, stripe, chunk, block_from, batch, 0, blocks,
                    work.data_ptr() if claims else None, sink.data_ptr(), None)
                assert rc == 0
                torch.cuda.synchronize()
                got = np.bitwise_xor.reduce(sink.cpu().numpy().view(np.uint32))
                assert got == acc, (block_from, batch, chunk, claims)
    assert not work.any().item()
    r.close()


def _table3(name):
    return synth.CONFIGS[name]


BLOCK_CFGS = [
    synth.VIEW720P.replace(name="blk_720p_rows", rows=64),
    synth.VIEW720P_DENSE.replace(name="blk_dense_rows", rows=64),
    synth.OPAQUE720P.replace(name="blk_opaque_rows", rows=64),
    synth.VIEW720P.replace(name="blk_k1", K=1, rows=96),
    synth.VIEW720P.replace(name="blk_ragged", H=23, W=37, views=2, K=3, gbuf="iid",
                           delta=0.5, log2_T=12, N_max=2048),
    # 8-byte entries (fp16, F = 4): one query per pixel with the MLP, 8
    # samples per ray (the rounds path), and a ragged frame
    synth.TABLE3[0].replace(name="blk_f4_L8", rows=64),
    synth.TABLE3[0].replace(name="blk_f4_k8", K=8, delta=0.05, rows=32),
    synth.TABLE3[0].replace(name="blk_f4_ragged", H=23, W=37, views=2, K=3, gbuf="iid",
                            delta=0.5, log2_T=12),
]


@pytest.mark.parametrize("cfg", BLOCK_CFGS, ids=lambda c: c.name)
def test_block_gathers_give_the_same_frame(cfg):
    """16-byte block gathers of x-neighbour corner pairs read the same two
    entries as single gathers: every choice of levels renders the same bits,
    on the tile path, in the library's rounds and in rounds of one (where the
    entries of straddling voxels are loaded each with its block)."""
    say("block gathers", cfg.name)
    sc = synth.make_scene(cfg)
    ds = mixrt.DeviceScene.from_scene(sc, "cuda:0")
    ref = None
    seen = set()
    for chunk in (-1, 0, 1):
        for levels in (-1, 0, 1, 3, cfg.L):
            r = mixrt.Renderer(0, sync_check=True, early_stop_chunk=chunk, block_levels=levels)
            seen.add(r.launch_plan(ds)["block_from"])
            out = torch.full((ds.rays, 4), float("nan"), dtype=torch.float32, device="cuda:0")
            r.render(ds, out)
            r.sync()
            r.close()
            got = out.cpu().numpy()
            assert np.isfinite(got).all()
            if ref is None:
                ref = got
            assert np.array_equal(got, ref), (chunk, levels)
    say(f"  first block levels launched: {sorted(seen)}")
    assert len(seen) >= 3


@pytest.mark.parametrize("cfg", [BLOCK_CFGS[1], BLOCK_CFGS[5], BLOCK_CFGS[6]],
                         ids=lambda c: c.name)
def test_block_gathers_spot_check_against_the_oracle(cfg):
    say("block gathers against the oracle", cfg.name)
    sc = synth.make_scene(cfg)
    ds = mixrt.DeviceScene.from_scene(sc, "cuda:0")
    r = mixrt.Renderer(0, sync_check=True, block_levels=cfg.L)
    assert r.launch_plan(ds)["block_from"] < cfg.L
    got = r.render(ds).cpu().numpy()
    r.close()
    pix = np.random.default_rng(5).choice(cfg.rays, 2000, replace=False)
    ref = oracle.OracleScene(sc).render_pixels(pix, threads=oracle.max_threads())
    assert np.abs(got[pix] - ref).max() <= 2e-3


def _plan(cfg, W, H, views=1):
    """The launch plan of a frame of W x H x views pixels.  (A plan reads no
    device memory: the scene behind the descriptors is a small one.)"""
    ds = mixrt.DeviceScene.from_scene(synth.make_scene(cfg.replace(H=16, W=64, views=1)), "cuda:0")
    ds.gbuf = mixrt.GBuffer(views, W, H, ds.g0.data_ptr(), 0)
    ds.cams = type(ds.cams)._type_.__mul__(views)(*([ds.cams[0]] * views))
    r = mixrt.Renderer(0)
    plan = r.launch_plan(ds)
    r.close()
    return plan


def _frame_of(tiles, K):
    """(W, H) of a frame of exactly that many tiles, one above the other: 64 / K
    pixels each, four times as wide as high or more (K a power of two)."""
    R, rows = 64 // K, 1
    while rows * rows * 16 <= R:
        rows *= 2
    return R // rows, rows * tiles


@pytest.mark.parametrize("cfg", [synth.VIEW720P, synth.VIEW720P_DENSE,
                                 synth.VIEW720P_DENSE.replace(name="d05", delta=0.05),
                                 synth.VIEW720P.replace(name="k2", K=2),
                                 synth.VIEW720P.replace(name="k3", K=3),
                                 synth.BATCH8X1080P, synth.PAPER720P],
                         ids=lambda c: c.name)
def test_default_round_size_follows_the_rule(cfg):
    """The library's default samples per round (0 = the tile path) at the
    workload's own size: 4 when a ray's samples share the voxels of half the
    levels and a level fits one XCD's L2, 2 or 1 as they share fewer, the
    tile path for K < 4 or K not a power of two and for coherent samples on
    levels larger than the L2."""
    want = {"view720p": 4, "view720p_dense": 1, "d05": 2, "k2": 0, "k3": 0,
            "batch8x1080p": 0, "paper720p": 0}[cfg.name]
    assert _plan(cfg, cfg.W, cfg.H, cfg.views)["chunk"] == want


@pytest.mark.parametrize("K,delta,first", [(8, 0.25, 1), (8, 0.05, 2), (8, 0.01, 4), (4, 0.25, 1),
                                           (16, 0.25, 1)])
def test_default_round_size_of_small_frames(K, delta, first):
    """The plan names the round that is launched: doubled as often as it takes
    for half of 3 waves per SIMD to get a run of K / C tiles, on both sides of
    every step, up to the tile path."""
    cfg = synth.VIEW720P_DENSE.replace(name="small_plan", K=K, delta=delta)
    waves = 12 * torch.cuda.get_device_properties(0).multi_processor_count
    C = first
    while C < K:
        enough = K * waves // (2 * C)              # tiles from which rounds of C stay
        assert _plan(cfg, *_frame_of(enough, K))["chunk"] == C, (C, enough)
        if C > first:
            assert _plan(cfg, *_frame_of(2 * enough - 1, K))["chunk"] == C, (C, enough)
        C *= 2
    assert _plan(cfg, *_frame_of(enough - 1, K))["chunk"] == 0
    assert _plan(cfg, *_frame_of(1, K))["chunk"] == 0


_K1 = synth.VIEW720P.replace(name="k1", K=1)
_K2 = synth.VIEW720P.replace(name="k2", K=2)
_K3 = synth.VIEW720P.replace(name="k3", K=3)
_COARSE = synth.VIEW720P.replace(name="coarse_k1", K=1, N_max=1024)


@pytest.mark.parametrize("cfg,W,H,want", [
    (synth.VIEW720P, 0, 0, (13, 2)), (synth.VIEW720P_DENSE, 0, 0, (9, 2)),
    (synth.VIEW720P_DENSE.replace(name="dense_k4", K=4), 0, 0, (11, 2)),
    (_K1, 0, 0, (9, 2)), (_K1, 2560, 1440, (10, 2)), (_K1, 4096, 2160, (12, 2)),
    (_K1, 7680, 4320, (13, 2)), (_K1, 320, 180, (13, 2)), (_COARSE, 1280, 720, (11, 2)),
    (_COARSE, 2560, 1440, (13, 2)),
    (_K2, 0, 0, (10, 2)), (_K2, 2560, 1440, (12, 2)), (_K3, 0, 0, (10, 2)),
    (_K3, 2560, 1440, (12, 2)), (_K3, 4096, 2160, (13, 2)),
    (synth.VIEW720P.replace(name="fine_spacing", delta=1e-4), 0, 0, (16, 2)),
    (synth.BATCH8X1080P, 0, 0, (8, 2)), (synth.BATCH8X1080P.replace(name="batch_k4", K=4), 0, 0, (12, 2)),
    (synth.PAPER720P, 0, 0, (4, 4)), (synth.DEPLOYED720P, 0, 0, (4, 4)),
    (synth.TABLE3[0], 0, 0, (0, 2)), (_table3("tab3_L8_T5"), 0, 0, (8, 2)),
    (_table3("tab3_L16_T17").replace(name="tab3_L16"), 0, 0, (0, 2))],
    ids=lambda c: c.name if hasattr(c, "name") else str(c).replace(" ", ""))
def test_default_gather_plan_follows_the_rule(cfg, W, H, want):
    """4-byte entries, among hashed levels finer than the sample spacing: block
    gathers on the three finest levels; at K < 4 on the 3 to 7 whose cells are
    at most 4 (K = 1) or 2 far pixels wide; in rounds of one sample per ray on
    five, seven from K = 8 on; when a level's table exceeds one XCD's L2 on
    four, and eight at K >= 8.  8-byte (fp16 F = 4) entries: on every hashed
    level when there are 8 or more of them in tables of 2^10 or more entries.
    Batches of 4 hashed levels only for entries of 8+ bytes when that covers
    every hashed level.  W, H: the frame (0: the workload's own)."""
    plan = _plan(cfg, W or cfg.W, H or cfg.H, 1 if W else cfg.views)
    assert (plan["block_from"], plan["hash_batch"]) == want, plan


@pytest.mark.parametrize("cfg,filled,less", [(_K1, 9, 13), (_K3, 9, 13), (synth.VIEW720P_DENSE, 9, 11)],
                         ids=lambda c: c.name if hasattr(c, "name") else str(c))
def test_more_block_levels_only_where_the_card_is_full(cfg, filled, less):
    """The extra levels at K < 4 and in rounds of one take a tile for each of 3
    waves per SIMD."""
    waves = 12 * torch.cuda.get_device_properties(0).multi_processor_count
    R = 64 // cfg.K
    RH = 2 if R == 16 else 4 if R == 64 else 1
    for tiles, want in ((waves, filled), (waves - 1, less)):
        assert _plan(cfg, R // RH * tiles, RH)["block_from"] == want, (tiles, want)


@pytest.mark.parametrize("cfg", [synth.VIEW720P, synth.PAPER720P, synth.BATCH8X1080P,
                                 _table3("tab3_L8_T17_mlp"), _table3("tab3_L1_T17"),
                                 _table3("tab3_L4_T17"), _table3("tab3_L8_T5")],
                         ids=lambda c: c.name)
def test_default_claims_follow_the_rule(cfg):
    """The last units are claimed from the work counters when a unit's work
    hides a claim's latency: with an MLP, or with 8 or more levels."""
    want = {"view720p": 1, "paper720p": 1, "batch8x1080p": 1, "tab3_L8_T17_mlp": 1,
            "tab3_L1_T17": 0, "tab3_L4_T17": 0, "tab3_L8_T5": 1}[cfg.name]
    sc = synth.make_scene(cfg.replace(H=16, W=64, views=1))
    ds = mixrt.DeviceScene.from_scene(sc, "cuda:0")
    r = mixrt.Renderer(0)
    plan = r.launch_plan(ds)
    r.close()
    assert plan["claims"] == want, plan


QUEUE_CFGS = [
    synth.TINY64_DENSE.replace(name="q_tiny_dense", t_term=1e-2),
    synth.TINY64_DENSE.replace(name="q_ragged_k3", H=23, W=37, views=2, K=3, gbuf="iid",
                               t_term=1e-2),
    synth.TINY64_DENSE.replace(name="q_ragged_k7", H=19, W=21, views=3, K=7, gbuf="iid",
                               t_term=1e-3),
    synth.TINY64_DENSE.replace(name="q_k64", H=9, W=11, K=64, gbuf="iid", t_term=0.0),
    synth.TINY64_DENSE.replace(name="q_k1", H=33, W=31, views=2, K=1, gbuf="iid"),
    synth.TINY64_DENSE.replace(name="q_nomlp", widths=(16,), seed=16, t_term=1e-2),
    synth.TINY64_VEC3, synth.TINY64_U8,
    synth.OPAQUE720P, synth.TRANSLUCENT720P, synth.VIEW720P_DENSE, synth.PAPER720P,
]


@pytest.mark.parametrize("cfg", QUEUE_CFGS, ids=lambda c: c.name)
def test_early_termination_path_renders_the_same_frame(cfg):
    """Every round size renders the tile path's frame bit for bit, misses
    included (5% of each kind on the small workloads)."""
    say("early termination", cfg.name)
    sc = synth.make_scene(cfg)
    if cfg.rays < 20000:
        flat = sc.g0.reshape(-1, 4)
        rng = np.random.default_rng(cfg.seed)
        miss = rng.choice(flat.shape[0], flat.shape[0] // 20, replace=False)
        flat[miss, 0] = rng.choice([0.0, -1.0, np.nan, np.inf], miss.size)
    ds = mixrt.DeviceScene.from_scene(sc, "cuda:0")
    ref, _ = _render(ds, early_stop_chunk=-1)
    assert np.all(np.isfinite(ref))
    for chunk in (1, 2, 4, 8, 64):
        got, _ = _render(ds, early_stop_chunk=chunk)
        assert np.array_equal(got, ref), chunk
    got, _ = _render(ds, early_stop_chunk=2, tile_stripe=-1, blocks="two")
    assert np.array_equal(got, ref)


@pytest.mark.parametrize("cfg", [synth.OPAQUE720P, synth.TRANSLUCENT720P],
                         ids=lambda c: c.name)
def test_early_termination_against_the_oracle(cfg):
    """The frame within 2e-3 + t_term of the oracle (which never stops a
    ray) on sampled pixels, and fewer samples evaluated than the tile path
    (counted by the phase-timer build)."""
    say("early termination vs oracle", cfg.name)
    sc = synth.make_scene(cfg)
    ds = mixrt.DeviceScene.from_scene(sc, "cuda:0")
    got, _ = _render(ds, early_stop_chunk=1)
    rng = np.random.default_rng(9)
    pix = np.unique(np.concatenate([rng.choice(cfg.rays, 3000, replace=False),
                                    np.arange(cfg.W)]))
    ref = oracle.OracleScene(sc).render_pixels(pix, threads=oracle.max_threads())
    err = np.abs(got[pix] - ref).max()
    say(f"  max |gpu - oracle| = {err:.3e}")
    assert err <= 2e-3 + cfg.t_term
    counts = {}
    for chunk in (-1, 1, 2, 4):
        r = mixrt.Renderer(0, sync_check=True, variant="timer", early_stop_chunk=chunk)
        r.phase_cycles(reset=True)
        r.render(ds)
        counts[chunk] = r.phase_cycles(reset=True)["samples"]
        r.close()
    say("  samples evaluated by round size:", counts)
    assert counts[-1] == cfg.rays * cfg.K            # every pixel hits
    assert counts[1] < counts[2] <= counts[4] < counts[-1]


def test_gather_lines_microbenchmark():
    """The L1 cost probe behind the block gathers: runs at every width and
    sharing pattern, refuses a line count that does not divide 64, and a
    gather touching 64 lines costs more than one touching 4."""
    from paper_2312_11841_amd import microbench as mb
    t = torch.zeros(16 * 1024 // 4, dtype=torch.int32, device="cuda:0")
    sink = torch.empty(256 * 256, dtype=torch.int32, device="cuda:0")
    assert mb.lib().mixrt_mb_gather_lines(t.data_ptr(), 16 * 1024, 4, 3, 1, 1, 256,
                                          sink.data_ptr(), None) != 0
    assert mb.lib().mixrt_mb_gather_lines(t.data_ptr(), 16 * 1024 + 128, 4, 4, 1, 1, 256,
                                          sink.data_ptr(), None) != 0
    few = mb.gather_lines(16 * 1024, 4, 4, True, iters=32)
    many = mb.gather_lines(16 * 1024, 4, 64, True, iters=32)
    for width in (8, 16):
        assert mb.gather_lines(2048 * 1024, width, 16, False, iters=16) > 0
    say(f"  cycles per gather: 4 lines {few:.1f}, 64 lines {many:.1f}")
    assert many > 2 * few
