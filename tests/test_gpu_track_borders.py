"""The tracker's pixel windows against the oracle, which reads the images
directly: keypoints at the limits of where their patch fits, all along the four
borders and in the corners, starts some pixels off, odd and small sizes. Compared
where the oracle itself is sure (its FP32 and FP64 tracks agree to a tenth of the
tolerance); a keypoint whose patch does not fit at level 0 is lost as out of bounds."""
import numpy as np
import pytest

import oracle
from parity_util import TOL_PX, TOL_THETA

SIZES = [(33, 20, 2), (64, 48, 3), (161, 97, 4), (250, 190, 5), (1280, 720, 6), (97, 331, 1)]
N = 300
ITERS = 5


def _frames(rng, w, h):
    """A smooth random image and the same moved by (1.3, -0.8) px."""
    y, x = np.mgrid[0:h, 0:w].astype(np.float64)

    def at(x, y):
        v = np.full(x.shape, 128.0)
        for _ in range(24):
            f = rng2.uniform(-1.0, 1.0, 2) * rng2.choice([0.12, 0.35, 0.8])
            v += rng2.uniform(4.0, 16.0) * np.sin(f[0] * x + f[1] * y + rng2.uniform(0.0, 6.28))
        return np.clip(np.round(v), 0, 255).astype(np.uint8)
    seed = rng.integers(1 << 30)
    rng2 = np.random.default_rng(seed)
    a = at(x, y)
    rng2 = np.random.default_rng(seed)
    return a, at(x - 1.3, y + 0.8)


def _keypoints(rng, w, h):
    """Positions x, y and starts, float32: half of them within a pixel of a border's limit."""
    x = rng.uniform(3.0, w - 4.0, N)
    y = rng.uniform(3.0, h - 4.0, N)
    for i in range(N // 2):
        d = rng.choice([0.0, 0.0, 0.5, -0.25, rng.uniform(-0.5, 3.0)])
        side = rng.integers(4)
        if side < 2 or i % 3 == 0:  # (some in the corners)
            x[i] = 4.5 + d if rng.random() < 0.5 else w - 5.5 - d
        if side >= 2 or i % 3 == 0:
            y[i] = 4.5 + d if rng.random() < 0.5 else h - 5.5 - d
    x, y = x.astype(np.float32), y.astype(np.float32)
    px = (x - 1.3 + rng.normal(0, 1, N) * rng.choice([0.2, 1.0, 2.5], N)).astype(np.float32)
    py = (y + 0.8 + rng.normal(0, 1, N) * rng.choice([0.2, 1.0, 2.5], N)).astype(np.float32)
    return x, y, px, py


def _case(w, h, levels, cam):
    rng = np.random.default_rng(w * 7 + h + levels + 1000 * cam)
    a, b = _frames(rng, w, h)
    x, y, px, py = _keypoints(rng, w, h)
    pts, start = np.stack([x, y], 1), np.stack([x + (x - px), y + (y - py)], 1)
    r32, s32 = oracle.track(a, b, pts, start, levels, ITERS)
    r64, s64 = oracle.track(a, b, pts, start, levels, ITERS, double=True)
    near = np.abs(r32 - r64).max(1) < 0.1 * TOL_PX
    sure = (s32 == s64) & (s32 == oracle.TRACKED) & near & (r32[:, 3] < 0.25)
    outside = (x < 4.5) | (y < 4.5) | (x > w - 5.5) | (y > h - 5.5)
    assert (s32[outside] == oracle.LOST_OOB).all()
    return a, b, (x, y, px, py), r32, sure, outside


@pytest.mark.parametrize("w,h,levels", SIZES)
def test_the_cases_say_something(w, h, levels):
    x, y, _, _ = _case(w, h, levels, 0)[2]
    sure, outside = _case(w, h, levels, 0)[4:]
    edge = sure & ((x < 6) | (y < 6) | (x > w - 7) | (y > h - 7))
    assert sure.sum() >= 60 and edge.sum() >= 20 and outside.sum() >= 10, (sure.sum(), edge.sum(), outside.sum())


@pytest.mark.gpu
@pytest.mark.parametrize("launch", [dict(track_kp_per_wave=1), dict(track_kp_per_wave=2),
                                    dict(track_kp_per_wave=1, track_waves_per_cu=2),
                                    dict(track_kp_per_wave=2, track_waves_per_cu=2)])
@pytest.mark.parametrize("w,h,levels", SIZES)
def test_borders(w, h, levels, launch):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_30459_amd as vf
    cases = [_case(w, h, levels, c) for c in range(2)]
    with vf.Frontend([(2, w, h, N, 32)], vf.make_params(levels=levels, gn_iters=ITERS, max_keypoints=N, cell_size=32,
                                                        **launch)) as fe:
        fe.push_stereo_frame(0, 1, [c[0] for c in cases])
        for c, case in enumerate(cases):
            kps = np.zeros(N, vf.KEYPOINT_DTYPE)
            kps["id"] = 1000 * (c + 1) + np.arange(N)
            kps["x"], kps["y"], kps["px"], kps["py"] = case[2]
            fe.set_keypoints(0, c, kps)
        fe.push_stereo_frame(0, 2, [c[1] for c in cases])
        rec = fe.get_tracks(0)
    for c, (_, _, _, want, sure, outside) in enumerate(cases):
        got = rec[(rec["camera"] == c) & (rec["id"] >= 1000 * (c + 1)) & (rec["id"] < 1000 * (c + 1) + N)]
        assert len(got) == N
        assert (got["status"][sure] == vf.VIO_TRACKED).all(), np.nonzero(sure & (got["status"] != vf.VIO_TRACKED))
        assert (got["status"][outside] == oracle.LOST_OOB).all()
        for i, (f, tol) in enumerate((("x", TOL_PX), ("y", TOL_PX), ("theta", TOL_THETA), ("fb_err", TOL_PX))):
            err = np.abs(got[f].astype(np.float64) - want[:, i])[sure]
            assert err.max() <= tol, (f, err.max())
