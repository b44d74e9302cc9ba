"""Keyframe rule (Sec. II) on the GPU against the oracle keyframe: a frame whose
camera centre moved more than lambda_trans from the keyframe's, or whose
semi-dense update produced fewer than lambda_inliers measurements, updates the
filter but is not fused. Decisions are compared frame by frame over a walk, the
depth map must stay bit-identical on frames that ask for a new keyframe, and a
new prior (kf_set_prior) starts the next keyframe."""

import numpy as np
import pytest

import kfsynth
from oracle import OracleKeyframe, SolverParams, StereoParams
from oracle.pipeline import NEW_KF_INLIERS, NEW_KF_TRANSLATION, camera_translation

import gpu_util as gu

pytestmark = pytest.mark.gpu


def test_translation_rule_over_a_walk():
    case = kfsynth.config_case(1, 0, frames=10)
    dist = [camera_translation(case.T_wc0, T) for T in case.poses]
    # a threshold half way between two frames' distances, so both sides decide alike
    srt = sorted(dist)
    lam = 0.5 * (srt[4] + srt[5])
    gu.say(f"[lifecycle] 320x240 f32 walk, distances {np.round(dist, 4).tolist()}, lambda_trans {lam:.4f}")
    from paper_2207_12244_amd.kf import Keyframe
    t = gu.torch()
    kf = Keyframe(case.W, case.H, precision="f32", pattern="sq5x5", n_samples=64, n_gn=10, n_cg=20, K=case.K,
                  lambda_trans=lam)
    kf.set_prior(gu.dev(case.image0, t.uint8), *[gu.dev(m, t.float32) for m in case.priors.maps()], case.T_wc0)
    ok = OracleKeyframe(case.K, case.W, case.H, StereoParams(n_samples=64, pattern="sq5x5"),
                        SolverParams(n_gn=10, n_cg=20, linear_solver="pcg"), lambda_trans=lam)
    ok.set_prior(case.image0, *case.priors.maps(), case.T_wc0)
    fired = 0
    for f in range(len(case.images)):
        before = gu.np_state(kf)
        kf.fuse_frame(gu.dev(case.images[f], t.uint8), case.poses[f])
        st = gu.np_state(kf)
        s = kf.stats()
        rep = ok.fuse_frame(case.images[f], case.poses[f])
        gu.say(f"[lifecycle] frame {f + 1}: distance {dist[f]:.4f} gpu {s.new_keyframe} oracle {rep.new_keyframe} "
               f"syncs {s.team_syncs}")
        assert s.new_keyframe == rep.new_keyframe
        if rep.new_keyframe:
            fired += 1
            assert rep.new_keyframe == NEW_KF_TRANSLATION
            assert np.array_equal(st["x"], before["x"]) and st["tau"] == before["tau"]
            assert s.team_syncs == 0
            assert np.count_nonzero(st["var"] != before["var"]) > 0      # the filter was still updated
        else:
            assert s.team_syncs > 0
    assert 0 < fired < len(case.images)
    # the caller starts the next keyframe: the rule measures from the new keyframe's pose
    kf.set_prior(gu.dev(case.images[0], t.uint8), *[gu.dev(m, t.float32) for m in case.priors.maps()],
                 case.poses[0])
    kf.fuse_frame(gu.dev(case.images[1], t.uint8), case.poses[1])
    assert kf.stats().new_keyframe == (NEW_KF_TRANSLATION if camera_translation(case.poses[0], case.poses[1]) > lam
                                       else 0)
    kf.close()


@pytest.mark.parametrize("lam,expect", [(1, 0), (10 ** 9, NEW_KF_INLIERS)])
def test_inlier_rule(lam, expect):
    case = kfsynth.config_case(0, 0)
    gu.say(f"[lifecycle] 160x120 f64 lambda_inliers {lam}")
    from paper_2207_12244_amd.kf import Keyframe
    t = gu.torch()
    kf = Keyframe(case.W, case.H, precision="f64", pattern="line5", n_samples=32, n_gn=3, n_cg=15, K=case.K,
                  lambda_inliers=lam)
    kf.set_prior(gu.dev(case.image0, t.uint8), *[gu.dev(m, t.float64) for m in case.priors.maps()], case.T_wc0)
    kf.fuse_frame(gu.dev(case.images[0], t.uint8), case.poses[0])
    st = gu.np_state(kf)
    s = kf.stats()
    assert s.new_keyframe == expect and s.n_updated > 0
    if expect:
        assert np.array_equal(st["x"], case.priors.logdepth) and st["tau"] == 0.0
    else:
        assert not np.array_equal(st["x"], case.priors.logdepth)
    kf.close()


def test_rule_per_member_in_a_batch():
    """Batched members decide on their own: one member with an unreachable inlier
    threshold is left unfused, the others fuse as they would alone."""
    from paper_2207_12244_amd.kf import Batch, Keyframe
    t = gu.torch()
    cases = [kfsynth.config_case(3, i, size_index=i % 2) for i in range(3)]
    members, imgs, poses = [], [], []
    for i, c in enumerate(cases):
        kf = Keyframe(c.W, c.H, precision="f32", pattern="line5", n_samples=32, n_gn=10, n_cg=20, K=c.K,
                      solver_threads=512, lambda_inliers=10 ** 9 if i == 1 else 0)
        kf.set_prior(gu.dev(c.image0, t.uint8), *[gu.dev(m, t.float32) for m in c.priors.maps()], c.T_wc0)
        members.append(kf)
        imgs.append(gu.dev(c.images[0], t.uint8))
        poses.append(c.poses[0])
    batch = Batch(members)
    batch.fuse(imgs, poses)
    for i, (kf, c) in enumerate(zip(members, cases)):
        s = kf.stats()
        st = gu.np_state(kf)
        gu.say(f"[lifecycle-batch] member {i} {c.W}x{c.H} new_keyframe {s.new_keyframe}")
        if i == 1:
            assert s.new_keyframe == NEW_KF_INLIERS and np.array_equal(st["x"], c.priors.logdepth.astype(np.float32))
        else:
            assert s.new_keyframe == 0 and not np.array_equal(st["x"], c.priors.logdepth.astype(np.float32))
    batch.close()


@pytest.mark.parametrize("W,H", [(8, 8), (16, 16), (257, 9), (129, 131), (1280, 1024)])
def test_search_list_counts(W, H):
    """The search list at the edges of its chunks of 256 pixels (fewer than one,
    exactly one, a remainder) and at the largest keyframe: as many pixels as the
    oracle's texture mask has, and measurements at those pixels alone."""
    from oracle import stereo
    from paper_2207_12244_amd.kf import Keyframe
    t = gu.torch()
    rng = np.random.default_rng(W * 10000 + H)
    img = rng.integers(0, 256, (H, W)).astype(np.uint8)
    img[: H // 2, : W // 3] = 128   # flat: not searched
    mask = stereo.texture_mask(img)
    K = np.array([[0.8 * W, 0.0, W / 2.0], [0.0, 0.8 * W, H / 2.0], [0.0, 0.0, 1.0]])
    kf = Keyframe(W, H, precision="f32", pattern="line5", n_samples=4, K=K)
    one = np.ones((H, W))
    kf.set_prior(gu.dev(img, t.uint8), *[gu.dev(m, t.float32) for m in (0 * one, one, 0 * one, one, 0 * one, one)],
                 np.eye(4))
    pose = np.eye(4)
    pose[0, 3] = 0.05
    kf.stereo_update(gu.dev(img, t.uint8), pose)
    assert kf.stats().n_searched == int(mask.sum())
    match = kf.export_state()["match"].cpu().numpy()
    assert np.array_equal(match == -2, ~mask)
    kf.close()


@pytest.mark.parametrize("pipelined", [False, True])
def test_contexts_on_different_streams(pipelined):
    """Three keyframes whose solver teams do not fit on the device together, each
    on a stream of its own and enqueued without a wait: the results of the same
    calls one after the other, and no team times out. A batch on a fourth stream
    runs in between."""
    from paper_2207_12244_amd.kf import Batch, Keyframe
    t = gu.torch()
    cases = [kfsynth.config_case(3, 20 + i, size_index=s, frames=8) for i, s in enumerate((3, 3, 2, 1, 1))]

    def make(c, stream, **kw):
        kf = Keyframe(c.W, c.H, precision="f32", n_samples=32, K=c.K, stream=stream, **kw)
        maps = [gu.dev(c.image0, t.uint8), *[gu.dev(m, t.float32) for m in c.priors.maps()]]
        t.cuda.synchronize()
        kf.set_prior(*maps, c.T_wc0)
        return kf

    images = [[gu.dev(im, t.uint8) for im in c.images] for c in cases]

    def run(streams, wait):
        kfs = [make(c, s, pipeline_frames=pipelined and i < 3) for i, (c, s) in enumerate(zip(cases, streams))]
        batch = Batch(kfs[3:])
        t.cuda.synchronize()
        for f in range(8):
            for i in range(3):
                kfs[i].fuse_frame(images[i][f], cases[i].poses[f])
                if wait:
                    t.cuda.synchronize()
            batch.fuse([images[i][f] for i in (3, 4)], [cases[i].poses[f] for i in (3, 4)])
            if wait:
                t.cuda.synchronize()
        t.cuda.synchronize()
        states = [gu.np_state(kf) for kf in kfs]
        batch.close()
        for kf in kfs:
            kf.close()
        return states

    own = [t.cuda.Stream() for _ in range(4)]
    alone = run([t.cuda.current_stream()] * 5, True)
    mixed = run(own + own[3:], False)
    for i, (a, b) in enumerate(zip(alone, mixed)):
        for k in ("x", "rho", "var", "match"):
            assert np.array_equal(a[k], b[k]), (i, k)
        assert a["tau"] == b["tau"], i


@pytest.mark.parametrize("cg_variant", ["auto", "pipelined"])
def test_probe_starts_from_cleared_words(cg_variant):
    """The synchronisation probe waits for tagged words; none may be left from a
    solve, an earlier probe or another use of the workspace (here: a pattern),
    also where a new keyframe does not clear them."""
    from paper_2207_12244_amd.kf import Keyframe
    t = gu.torch()
    W, H = 160, 120
    K = np.array([[0.8 * W, 0.0, W / 2.0], [0.0, 0.8 * W, H / 2.0], [0.0, 0.0, 1.0]])
    kf = Keyframe(W, H, precision="f32", K=K, cg_variant=cg_variant)
    kf.workspace.fill_(0xA5)
    z = t.zeros((H, W), dtype=t.float32, device="cuda")
    img = t.zeros((H, W), dtype=t.uint8, device="cuda")
    for _ in range(2):
        kf.set_prior(img, z, z + 1, z, z + 1, z, z + 1, np.eye(4))
        kf.probe_sync(1, 1)
        t.cuda.synchronize()
        lay = kf.solver_layout()
        words = 2 * lay["tiles_x"] * lay["tiles_y"] * 2 * 2 * (lay["tile_w"] + lay["tile_h"]) * 2   # kf_solve.hip's boundary
        end = -kf.workspace.data_ptr() % 256 + kf.cfg.workspace_bytes
        tail = kf.workspace[end - 8 * words:end].view(t.int64).cpu().numpy()
        assert not (tail == np.frombuffer(b"\xa5" * 8, np.int64)[0]).any()
        assert kf.stats().team_syncs == 1
    kf.close()


def test_contexts_come_and_go_with_solves_in_flight():
    """Contexts on streams of their own (a frame-pipelined one with an internal
    stream) are destroyed right after their calls, while others go on: no call
    fails, and the last ones' results are those of the same calls alone."""
    from paper_2207_12244_amd.kf import Keyframe
    t = gu.torch()
    c = kfsynth.config_case(3, 30, size_index=3, frames=2)
    maps = [gu.dev(c.image0, t.uint8), *[gu.dev(m, t.float32) for m in c.priors.maps()]]
    images = [gu.dev(im, t.uint8) for im in c.images]
    streams = [t.cuda.Stream() for _ in range(3)]
    t.cuda.synchronize()

    def life(stream, pipelined):
        kf = Keyframe(c.W, c.H, precision="f32", n_samples=32, K=c.K, stream=stream, pipeline_frames=pipelined)
        kf.set_prior(*maps, c.T_wc0)
        for im, T in zip(images, c.poses):
            kf.fuse_frame(im, T)
        return kf

    alone = gu.np_state(life(t.cuda.current_stream(), False))
    gone = []   # their workspaces stay until the device has passed the calls
    for _ in range(12):
        kfs = [life(s, i == 0) for i, s in enumerate(streams)]
        for kf in kfs[:2]:
            kf.close()
        gone += kfs
    for kf in gone[2::3]:
        st = gu.np_state(kf)
        for k in ("x", "rho", "var", "match"):
            assert np.array_equal(alone[k], st[k]), k
        kf.close()
    t.cuda.synchronize()


def _plain(c, stream, maps):
    from paper_2207_12244_amd.kf import Keyframe
    kf = Keyframe(c.W, c.H, precision="f32", n_samples=32, K=c.K, stream=stream)
    kf.set_prior(*maps, c.T_wc0)
    return kf


def test_contexts_in_different_threads():
    """A thread per keyframe, each on a stream of its own: the results of the same
    calls in one thread."""
    import threading
    t = gu.torch()
    cases = [kfsynth.config_case(3, 40 + i, size_index=s, frames=6) for i, s in enumerate((3, 2, 3))]
    maps = [[gu.dev(c.image0, t.uint8), *[gu.dev(m, t.float32) for m in c.priors.maps()]] for c in cases]
    images = [[gu.dev(im, t.uint8) for im in c.images] for c in cases]
    t.cuda.synchronize()

    def life(i, stream, out):
        kf = _plain(cases[i], stream, maps[i])
        for im, T in zip(images[i], cases[i].poses):
            kf.fuse_frame(im, T)
        out[i] = gu.np_state(kf)
        kf.close()

    alone, mixed = {}, {}
    for i in range(3):
        life(i, t.cuda.current_stream(), alone)
    threads = [threading.Thread(target=life, args=(i, t.cuda.Stream(), mixed)) for i in range(3)]
    for th in threads:
        th.start()
    for th in threads:
        th.join()
    for i in range(3):
        for k in ("x", "rho", "var", "match"):
            assert np.array_equal(alone[i][k], mixed[i][k]), (i, k)


def test_captured_call_beside_another_stream():
    """A captured kf_fuse_frame_static, captured and replayed while a context on
    another stream has solves in flight: every replay is the eager call's result,
    and the other context's results are its own."""
    import ctypes
    from paper_2207_12244_amd import kf as K
    t = gu.torch()
    lib = K.load_library()
    c, o = kfsynth.config_case(3, 50, size_index=1, frames=1), kfsynth.config_case(3, 51, size_index=3, frames=1)
    maps, maps_o = ([gu.dev(v.image0, t.uint8), *[gu.dev(m, t.float32) for m in v.priors.maps()]] for v in (c, o))
    img, img_o = gu.dev(c.images[0], t.uint8), gu.dev(o.images[0], t.uint8)
    s, so = t.cuda.Stream(), t.cuda.Stream()
    t.cuda.synchronize()
    eager, captured, other, other_alone = (_plain(v, st, m) for v, st, m in (
        (c, s, maps), (c, s, maps), (o, so, maps_o), (o, so, maps_o)))

    def static(kf):
        assert lib.kf_fuse_frame_static(kf.ctx, ctypes.c_void_p(img.data_ptr()), K._pose(c.poses[0])) == K.KF_OK

    t.cuda.synchronize()
    graph = t.cuda.CUDAGraph()
    other.fuse_frame(img_o, o.poses[0])
    with t.cuda.graph(graph, stream=s):
        static(captured)
        other.solve()
    t.cuda.synchronize()
    for replay in range(4):
        other.solve()
        t.cuda.synchronize()   # what a graph replays is for the caller to order
        with t.cuda.stream(s):
            graph.replay()
        t.cuda.synchronize()
        static(eager)
        a, b = gu.np_state(eager), gu.np_state(captured)
        for k in ("x", "rho", "var", "match"):
            assert np.array_equal(a[k], b[k]), (replay, k)
        assert a["tau"] == b["tau"], replay
    other_alone.fuse_frame(img_o, o.poses[0])
    for _ in range(5):
        other_alone.solve()
    a, b = gu.np_state(other_alone), gu.np_state(other)
    assert np.array_equal(a["x"], b["x"]) and a["tau"] == b["tau"]
    for kf in (eager, captured, other, other_alone):
        kf.close()
