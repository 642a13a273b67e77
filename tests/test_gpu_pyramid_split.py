"""The pyramid launch in its two forms, and with each tile edge: detection and
levels of a tile in one workgroup (a step of many streams) or in two (the same
stream alone), the former with 1,024 or 512 threads to a 64-px tile, at sizes on both sides of the tile edges, with more than one key
per cell, a detection mask, and 1 to 6 levels. Levels and records are whole
numbers and float bits that must not change, so they are compared exactly."""
import numpy as np
import pytest

import synthgen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("w,h,levels,kcell", [(64, 64, 2, 1), (65, 63, 1, 1), (97, 130, 3, 2), (320, 240, 6, 1),
                                              (383, 257, 4, 3), (641, 479, 5, 1), (161, 140, 1, 1),
                                              (200, 150, 2, 1), (180, 170, 3, 2)])
def test_split_and_joined_launches_agree(w, h, levels, kcell):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_30459_amd as vf
    seq = synthgen.render(seed=w + h, width=w, height=h, n_frames=3, stereo=True, density=6.0, max_scale=0.01)
    mask = np.zeros((h, w), np.uint8)
    mask[h // 4:h // 2, w // 4:w // 2] = 1
    extra = dict(max_keypoints=128, cell_size=32, levels=levels, k_per_cell=kcell)
    many = 32  # cameras of 32 streams: no room for a second entry each in the launch's arguments
    want = None
    for n_streams, tile in ((1, 0), (1, 32), (1, 64), (many, 32), (many, 64)):
        with vf.Frontend([(2, w, h)] * n_streams, vf.make_params(pyr_tile=tile, **extra)) as fe:
            got = []
            for s in range(n_streams):
                fe.set_detection_mask(s, 0, mask)
            for t in range(3):
                for s in range(n_streams):
                    fe.stage_frame(s, t + 1, list(seq.frames[t]))
                fe.step()
                got.append(fe.get_tracks(0).tobytes())
                got += [fe.get_pyramid(0, c, l).tobytes() for c in range(2) for l in range(levels)]
        want = want or got
        assert got == want, (n_streams, tile)
