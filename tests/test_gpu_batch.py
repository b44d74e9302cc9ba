"""Batched form on the GPU: every keyframe of a mixed batch ends bit-identical
to the same keyframe fused alone (same tiling, same arithmetic), with and
without graph replay, and when there are more solver teams than co-resident
workgroups so that workgroups run several teams in turn."""

import numpy as np
import pytest

import kfsynth
from gpu_util import dev, map_dtype, say, torch

pytestmark = pytest.mark.gpu

BATCH_KW = dict(precision="bf16", pattern="line5", n_samples=32, n_gn=10, solver_threads=512)


def _make(case, n_cg=20, tiles=(0, 0)):
    from paper_2207_12244_amd.kf import Keyframe
    t = torch()
    kf = Keyframe(case.W, case.H, K=case.K, n_cg=n_cg, tiles=tiles, **BATCH_KW)
    dt = map_dtype(BATCH_KW["precision"])
    kf.set_prior(dev(case.image0, t.uint8), *[dev(m, dt) for m in case.priors.maps()], case.T_wc0)
    return kf


def _state(kf):
    s = kf.export_state()
    return {k: (v.cpu().numpy() if hasattr(v, "cpu") else v) for k, v in s.items()}


def _assert_same(a, b, label):
    for k in ("x", "rho", "var", "match"):
        assert np.array_equal(a[k], b[k], equal_nan=True), f"{label}: {k} differs " \
            f"(max |d| {np.nanmax(np.abs(a[k].astype(np.float64) - b[k].astype(np.float64)))})"
    assert a["tau"] == b["tau"], label


def _run_pair(cases, settings, frames, mode):
    from paper_2207_12244_amd.kf import Batch
    t = torch()
    solo = [_make(c, **s) for c, s in zip(cases, settings)]
    members = [_make(c, **s) for c, s in zip(cases, settings)]
    batch = Batch(members, use_graph=mode != "direct")
    imgs = [[dev(c.images[f], t.uint8) for c in cases] for f in range(frames)]
    for f in range(frames):
        for i, (k, c) in enumerate(zip(solo, cases)):
            k.fuse_frame(imgs[f][i], c.poses[f])
        poses = [c.poses[f] for c in cases]
        if mode == "split":
            batch.stereo_update(imgs[f], poses)
            batch.solve()
        else:
            batch.fuse(imgs[f], poses)
    t.cuda.synchronize()
    return solo, members, batch


@pytest.mark.parametrize("mode", ["graph", "direct", "split"])
def test_batch_equals_solo_mixed_sizes(mode):
    # sizes of the batched workload plus a ragged one; one member with another CG count
    sizes = [0, 1, 2, 3, 0, 1]
    cases = [kfsynth.config_case(3, i, size_index=s, frames=2) for i, s in enumerate(sizes)]
    extra = kfsynth.make_case(kfsynth.seed_for(3, 99), 200, 130, 2, "single")
    cases.append(extra)
    settings = [dict() for _ in cases]
    settings[4] = dict(n_cg=7)
    say(f"batch mixed: sizes {[(c.W, c.H) for c in cases]}, mode={mode}")
    solo, members, batch = _run_pair(cases, settings, 2, mode)
    lay = batch.layout()
    say(f"batch layout {lay}")
    for i, (a, b) in enumerate(zip(solo, members)):
        sa, sb = _state(a), _state(b)
        assert b.stats().n_updated == a.stats().n_updated
        _assert_same(sa, sb, f"member {i} ({cases[i].W}x{cases[i].H})")
        assert np.isfinite(sa["x"]).all()
    batch.close()


def test_batch_queues_more_teams_than_resident_workgroups():
    # 256-workgroup teams (16 x 16 tiles of 320 x 240): more teams than fit at once
    n = 8
    cases = [kfsynth.config_case(3, 10 + i, size_index=1, frames=1) for i in range(n)]
    settings = [dict(tiles=(16, 16)) for _ in cases]
    say(f"batch queued: {n} x 320x240 with 16x16 tiles")
    solo, members, batch = _run_pair(cases, settings, 1, "graph")
    lay = batch.layout()
    say(f"batch layout {lay}")
    assert lay["max_queue"] >= 2, lay
    for i, (a, b) in enumerate(zip(solo, members)):
        _assert_same(_state(a), _state(b), f"member {i}")
    batch.close()


def test_batch_subset_calls_equal_solo():
    """kf_batch_fuse_subset: listed members advance exactly as alone; the rest stay untouched."""
    from paper_2207_12244_amd.kf import Batch
    t = torch()
    cases = [kfsynth.config_case(3, 60 + i, size_index=i % 4, frames=3) for i in range(5)]
    solo = [_make(c) for c in cases]
    members = [_make(c) for c in cases]
    batch = Batch(members)
    plan = [[0, 1, 2, 3, 4], [0, 2, 4], [3, 1]]
    say(f"batch subset: plan {plan}")
    for f, active in enumerate(plan):
        imgs = [dev(cases[i].images[f], t.uint8) for i in active]
        poses = [cases[i].poses[f] for i in active]
        for k, i in enumerate(active):
            solo[i].fuse_frame(imgs[k], poses[k])
        batch.fuse_subset(active, imgs, poses)
    t.cuda.synchronize()
    for i in range(len(cases)):
        _assert_same(_state(solo[i]), _state(members[i]), f"member {i}")
    batch.close()


def test_batch_schedule_fills_the_workgroups():
    """The batched workload's 64-keyframe mix at 512 threads x 10 px per thread
    (14 x 160x120, 22 x 320x240, 16 x 512x384, 12 x 640x480: 4 / 15 / 39 / 60
    tiles) puts 1,730 team members on 256 workgroups. The host places next the
    team that can start earliest, so small teams fill the workgroups that large
    ones would leave waiting, and the longest queue holds ceil(1730 / 256) = 7
    teams (placing the teams in order of decreasing cost left gaps: 8)."""
    from paper_2207_12244_amd.autotune import tiles_for
    from paper_2207_12244_amd.kf import Batch, Keyframe
    t = torch()
    if t.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the expected queue length is for a 256-CU device")
    mix = {(160, 120): 14, (320, 240): 22, (512, 384): 16, (640, 480): 12}
    members, total = [], 0
    for (W, H), n in mix.items():
        tx, ty = tiles_for(W, H, 512, 10)
        K = np.array([[0.8 * W, 0.0, W / 2.0], [0.0, 0.8 * W, H / 2.0], [0.0, 0.0, 1.0]])
        for _ in range(n):
            members.append(Keyframe(W, H, K=K, tiles=(tx, ty), **BATCH_KW))
        total += n * tx * ty
    batch = Batch(members, use_graph=False)
    lay = batch.layout()
    say(f"schedule of the 64-keyframe mix: {total} team members, layout {lay}")
    assert total == 1730
    assert lay["workgroups"] == 256 and lay["ppt"] == 10, lay
    assert lay["max_queue"] == -(-total // 256), lay
    batch.close()
    for m in members:
        m.close()


@pytest.mark.parametrize("kw,tiles,per_cu", [
    (dict(precision="f64", solver_threads=512, cg_variant="textbook"), (16, 16), 2),
    (dict(precision="f64", solver_threads=512, cg_variant="textbook", robust="tukey"), (16, 16), 2),
    (dict(precision="f64", solver_threads=256, cg_variant="textbook", robust="tukey"), (16, 12), 3),
    (dict(precision="f64", solver_threads=256, cg_variant="textbook"), (8, 8), 2),
    (dict(precision="f64", solver_threads=256, cg_variant="textbook", robust="tukey"), (8, 8), 2),
    (dict(precision="f32", solver_threads=256, cg_variant="pipelined"), (10, 8), 3),
    (dict(precision="f32", solver_threads=512, cg_variant="pipelined"), (7, 6), 2),
])
def test_batch_workgroups_share_a_compute_unit(kw, tiles, per_cu):
    """The instances whose registers are held to a step, at 1, 2, 4 and 6 pixels per
    thread: as many workgroups as that step lets a compute unit hold."""
    from paper_2207_12244_amd.kf import Batch, Keyframe
    t = torch()
    n = 3 * 256 * per_cu // (2 * tiles[0] * tiles[1]) + 1
    members = [Keyframe(320, 240, tiles=tiles, **kw) for _ in range(n)]
    batch = Batch(members, use_graph=False)
    lay = batch.layout()
    say(f"batch residency {kw} tiles {tiles}: {lay}")
    assert lay["workgroups"] == per_cu * t.cuda.get_device_properties(0).multi_processor_count, lay
    batch.close()
    for m in members:
        m.close()


def _auto(case, n_cg=20, tiles=(0, 0), **kw):
    """A member with the automatic workgroup size: s-step PCG unless kw asks for another."""
    from paper_2207_12244_amd.kf import Keyframe
    t = torch()
    kf = Keyframe(case.W, case.H, K=case.K, n_cg=n_cg, tiles=tiles, precision="f32", n_samples=32, **kw)
    kf.set_prior(dev(case.image0, t.uint8), *[dev(m, t.float32) for m in case.priors.maps()], case.T_wc0)
    return kf


# one member per strip length of either kernel (a single tile, short and long
# strips, 2 and 4 iterations per synchronisation), with iteration counts of their own
AUTO_MEMBERS = [
    ((64, 48), dict()),
    ((64, 48), dict(tiles=(1, 1), n_cg=9)),
    ((160, 120), dict()),
    ((160, 120), dict(tiles=(2, 2))),
    ((168, 120), dict(tiles=(2, 2), n_cg=7)),
    ((320, 240), dict()),
    ((320, 240), dict(tiles=(6, 4), n_cg=11)),
    ((320, 240), dict(tiles=(8, 6), n_cg=6)),
    ((96, 80), dict(tiles=(2, 2))),
    ((128, 120), dict(tiles=(2, 2), n_cg=5)),
    ((512, 384), dict()),
    ((333, 251), dict(n_gn=3)),
    ((640, 480), dict(n_gn=4)),
]


def _auto_cases(sizes, frames):
    return [kfsynth.make_case(kfsynth.seed_for(3, 200 + i), W, H, frames, "single") for i, (W, H) in enumerate(sizes)]


@pytest.mark.parametrize("mode", ["graph", "direct", "split"])
@pytest.mark.parametrize("var", [False, True])
def test_batch_of_sstep_members_equals_solo(mode, var):
    """Members with the automatic workgroup size, of every strip length, in one
    launch with more teams than workgroups; var: one of them with Tukey's cost, so
    that all run the instance that has the variants."""
    from paper_2207_12244_amd.kf import Batch
    t = torch()
    settings = [dict(s) for _, s in AUTO_MEMBERS]
    if var:
        settings[2]["robust"] = "tukey"
    cases = _auto_cases([size for size, _ in AUTO_MEMBERS], 2)
    solo = [_auto(c, **s) for c, s in zip(cases, settings)]
    members = [_auto(c, **s) for c, s in zip(cases, settings)]
    batch = Batch(members, use_graph=mode != "direct")
    lay = batch.layout()
    say(f"batch of s-step members, mode {mode} var {var}: {lay}")
    assert lay["max_queue"] >= 2 and lay["threads"] == 512, lay
    for f in range(2):
        imgs = [dev(c.images[f], t.uint8) for c in cases]
        poses = [c.poses[f] for c in cases]
        for k, im, p in zip(solo, imgs, poses):
            k.fuse_frame(im, p)
        if mode == "split":
            batch.stereo_update(imgs, poses)
            batch.solve()
        else:
            batch.fuse(imgs, poses)
        t.cuda.synchronize()
    for i, (a, b) in enumerate(zip(solo, members)):
        assert a.stats().team_syncs == b.stats().team_syncs
        _assert_same(_state(a), _state(b), f"member {i} {AUTO_MEMBERS[i]}")
        assert np.isfinite(_state(a)["x"]).all()
    batch.close()


def test_batch_of_both_solvers_equals_solo():
    """Members of both solvers in one batch (two solver launches): all of them, and
    subsets that leave one or the other without a member."""
    from paper_2207_12244_amd.kf import Batch
    t = torch()
    sizes = [(160, 120), (160, 120), (320, 240), (320, 240), (64, 48)]
    settings = [dict(), dict(cg_variant="pipelined"), dict(), dict(cg_variant="pipelined"), dict(n_cg=2)]
    cases = _auto_cases(sizes, 5)
    solo = [_auto(c, **s) for c, s in zip(cases, settings)]
    members = [_auto(c, **s) for c, s in zip(cases, settings)]
    threads = {m.solver_layout()["threads"] for m in members}
    batch = Batch(members)
    say(f"batch of both solvers: {batch.layout()}, workgroup sizes {threads}")
    plan = [[0, 1, 2, 3, 4], [0, 2], [4, 1, 3], [3, 2], [0, 1, 2, 3, 4]]
    for f, active in enumerate(plan):
        imgs = [dev(cases[i].images[f], t.uint8) for i in active]
        poses = [cases[i].poses[f] for i in active]
        for k, i in enumerate(active):
            solo[i].fuse_frame(imgs[k], poses[k])
        if f == 4:
            batch.stereo_update(imgs, poses)
            batch.solve()
        else:
            batch.fuse_subset(active, imgs, poses)
        t.cuda.synchronize()
    for i in range(len(cases)):
        assert solo[i].stats().team_syncs == members[i].stats().team_syncs
        _assert_same(_state(solo[i]), _state(members[i]), f"member {i} {sizes[i]} {settings[i]}")
    batch.close()
