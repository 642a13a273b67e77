"""The tracker's persistent grid: a wave starts with the items of its number and
takes the rest from the queue counter. Grids with more and with fewer waves than
items, workgroups whose last waves have none, odd item counts and the second queue
of deferred matches give the records of one launch per item, bit for bit."""
import pytest

import oracle
import synthgen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kpw", [1, 2])
@pytest.mark.parametrize("extra", [{}, dict(stereo_mode=1), dict(levels=6), dict(levels=1, stereo_init=1, stereo_levels=1),
                                   dict(init_mode=1, learned_levels=2, learned_iters=3)])
@pytest.mark.parametrize("streams", [[(1, 161, 97, 5, 32)], [(2, 752, 480, 301, 32)],
                                     [(2, 321, 243, 333, 16)] * 5 + [(1, 161, 97, 7, 24)]])
def test_grids_equal_one_launch_per_item(streams, extra, kpw):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_30459_amd as vf
    seqs = {s[1:3]: synthgen.render(seed=9, width=s[1], height=s[2], n_frames=3, stereo=True, density=8.0,
                                    max_scale=0.02) for s in streams}
    P = oracle.mlp_init(13) * 0.05
    P[-3:] = 0.0
    want = None
    for waves, block in ((0, 4), (1, 4), (1, 1), (2, 2), (64, 4)):
        got = []
        p = vf.make_params(track_kp_per_wave=kpw, track_waves_per_cu=waves, track_block_waves=block, **extra)
        with vf.Frontend(streams, p) as fe:
            if "init_mode" in extra:
                fe.set_mlp(P, 0.03)
            for t in range(3):
                for i, s in enumerate(streams):
                    fe.stage_frame(i, t + 1, list(seqs[s[1:3]].frames[t][:s[0]]))
                fe.step()
                got += [fe.get_tracks(i).tobytes() for i in range(len(streams))]
        want = want or got
        assert any(got) and got == want, (waves, block)
