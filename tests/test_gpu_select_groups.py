"""The selection with a workgroup per camera group: a rig's pairs, each on a
workgroup of its own, against the same pairs as streams of their own. The
records have to be the same but for the identifiers, which a rig's groups take
from one sequence: group by group, in cell order, without gaps. Sizes below and
above one pass of a workgroup (1,024 rows or cells), and rooms that fill up."""
import numpy as np
import pytest

import synthgen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("w,h,cell,cap,k", [(320, 240, 16, 40, 1), (641, 479, 12, 1100, 1), (500, 333, 32, 300, 3)])
@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("plain", [False, True])
def test_groups_of_a_rig_equal_streams(w, h, cell, cap, k, mode, plain):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_30459_amd as vf
    seqs = [synthgen.render(seed=s, width=w, height=h, n_frames=6, stereo=True, density=8.0, max_scale=0.03)
            for s in (3, 4)]
    p = vf.make_params(max_keypoints=cap, cell_size=cell, k_per_cell=k, stereo_mode=mode, plain=plain)
    with vf.Frontend([(4, w, h)], p) as rig, vf.Frontend([(2, w, h)], p) as a, vf.Frontend([(2, w, h)], p) as b:
        nxt = None
        for t in range(6):
            rig.push_stereo_frame(0, t + 1, [im for s in seqs for im in s.frames[t]])
            got = rig.get_tracks(0)
            for g, fe in enumerate((a, b)):
                fe.push_stereo_frame(0, t + 1, list(seqs[g].frames[t]))
                want = fe.get_tracks(0)
                mine = got[got["camera"] // 2 == g].copy()
                assert len(mine) == len(want) > 0, (t, g)
                # order-preserving renaming of the identifiers
                assert (np.unique(mine["id"], return_inverse=True)[1] ==
                        np.unique(want["id"], return_inverse=True)[1]).all(), (t, g)
                mine["camera"] -= 2 * g
                mine["id"] = want["id"]
                assert mine.tobytes() == want.tobytes(), (t, g)
                new = got["id"][(got["camera"] == 2 * g) & (got["status"] == vf.VIO_DETECTED)]
                if len(new):
                    assert (np.diff(new) == 1).all() and (nxt is None or new[0] == nxt), (t, g)
                    nxt = new[-1] + 1
