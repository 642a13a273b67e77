"""The tracker's LDS windows: keypoints at and past the borders, starts far from
the truth (windows that move, samples outside them) and small or odd levels.
The kernels of one and of two keypoints per wave leave their windows at
different positions (each sample's, or any the patch could reach) and then read
global memory: their records have to be the same, bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _images(rng, w, h, n):
    base = rng.integers(0, 256, (h // 6 + 8, w // 6 + 8)).astype(np.float64)
    big = np.kron(base, np.ones((6, 6)))
    big += rng.normal(0, 3, big.shape)
    out = []
    for t in range(n):
        dy, dx = (t * 2) % 7, (t * 3) % 11
        out.append(np.clip(big[dy:dy + h, dx:dx + w], 0, 255).astype(np.uint8))
    return out


@pytest.mark.parametrize("w,h,levels,cams", [(16, 16, 3, 1), (33, 20, 2, 1), (161, 97, 4, 2), (64, 48, 3, 2),
                                             (250, 190, 5, 1), (1280, 720, 6, 2)])
@pytest.mark.parametrize("persistent", [0, 2])
def test_windows_equal_global_gathers(w, h, levels, cams, persistent):
    import paper_2609_30459_amd as vf
    rng = np.random.default_rng(w * 31 + h + levels)
    frames = [_images(rng, w, h, 4) for _ in range(cams)]
    n = 200
    p = dict(levels=levels, max_keypoints=n, cell_size=max(8, w // 12), disparity0=min(30.0, w / 5),
             track_waves_per_cu=persistent)
    with vf.Frontend([(cams, w, h)], vf.make_params(**p)) as a, \
            vf.Frontend([(cams, w, h)], vf.make_params(track_kp_per_wave=2, **p)) as b:
        for t in range(4):
            if t > 0:
                kps = np.zeros(n, vf.KEYPOINT_DTYPE)
                kps["id"] = np.arange(n) + 1000 * t
                kps["x"] = rng.uniform(-4, w + 4, n)
                kps["y"] = rng.uniform(-4, h + 4, n)
                kps["px"] = kps["x"] + rng.normal(0, 1, n) * rng.choice([0.5, 4.0, 30.0], n)
                kps["py"] = kps["y"] + rng.normal(0, 1, n) * rng.choice([0.5, 4.0, 30.0], n)
                # exactly on the limits of the domain, whole and half pixels, and no position at all
                kps["x"][:12] = [0, w - 1, w - 2, 4.5, w - 5.5, w - 6, 5, w - 5, 1e9, -1e9, np.nan, w / 2]
                kps["y"][:12] = [h - 1, 0, 4.5, h - 5.5, h - 2, 5, h - 6, h / 2, 5, 5, 5, np.nan]
                kps["px"][:12], kps["py"][:12] = kps["x"][:12], kps["y"][:12]
                for c in range(cams):
                    a.set_keypoints(0, c, kps)
                    b.set_keypoints(0, c, kps)
            images = [frames[c][t] for c in range(cams)]
            a.push_stereo_frame(0, t + 1, images)
            b.push_stereo_frame(0, t + 1, images)
            ra, rb = a.get_tracks(0), b.get_tracks(0)
            assert ra.tobytes() == rb.tobytes(), (t, np.nonzero(ra.view(np.uint8).reshape(len(ra), -1) !=
                                                                rb.view(np.uint8).reshape(len(rb), -1))[0][:5])
            if t > 0 and min(w, h) > 64:
                assert (ra["status"] == vf.VIO_TRACKED).sum() > 20
