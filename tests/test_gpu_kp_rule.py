"""Keypoints per wave left to the library: launches on both sides of the number
of items from which a wave takes two, with short budgets, predictions and
deferred matches, give the records of one keypoint per wave, bit for bit."""
import numpy as np
import pytest

import synthgen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,extra", [(4, {}), (8, {}), (12, dict(stereo_mode=1)), (8, dict(pred_levels=2, pred_iters=3)),
                                     (8, dict(levels=5, gn_iters=7)), (12, dict(levels=1)),
                                     (8, dict(track_waves_per_cu=4))])
def test_rule_keeps_records(n, extra):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_30459_amd as vf
    seq = synthgen.render(seed=11, width=400, height=305, n_frames=4, stereo=True, density=8.0, max_scale=0.02)
    p = dict(max_keypoints=400, cell_size=16, **extra)  # 2 x 400 tracks and 500 possible matches a stream
    with vf.Frontend([(2, 400, 305)] * n, vf.make_params(**p)) as a, \
            vf.Frontend([(2, 400, 305)] * n, vf.make_params(track_kp_per_wave=1, **p)) as b:
        for t in range(4):
            for fe in (a, b):
                for s in range(n):
                    fe.stage_frame(s, t + 1, list(seq.frames[(t + s) % 4]))
                fe.step()
            for s in range(n):
                ra, rb = a.get_tracks(s), b.get_tracks(s)
                assert len(ra) > 100 and ra.tobytes() == rb.tobytes(), (t, s)
