"""The launch shapes the library chooses by itself (csrc/launch_rules.h): the rules
built for the CPU, and on the GPU the kernels that launches on both sides of them
take, by name, with the records of the other choice."""
import os
import re
import subprocess

import pytest

import synthgen

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2609_30459_amd", "csrc")


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    """rule(expression): a list of ints printed by a C++ expression over the header."""
    d = tmp_path_factory.mktemp("rules")

    def run(body):
        src = d / "rules.cpp"
        src.write_text('#include <cstdio>\n#include <initializer_list>\n#include "launch_rules.h"\nusing namespace vio;\nint main() {\n' + body +
                       "\n}\n")
        subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, str(src), "-o", str(d / "rules")],
                       check=True)
        return [int(v) for v in subprocess.run([str(d / "rules")], check=True, capture_output=True,
                                               text=True).stdout.split()]
    return run


def test_keypoints_per_wave_rule(rule):
    got = rule("for (int l = 1; l <= 6; ++l) for (int n : {1, 3072, 3073, 6144, 6145, 100000}) "
               "printf(\"%d \", two_keypoints_a_wave(n, 256, l));")
    assert got == 4 * [0, 0, 0, 0, 1, 1] + 2 * [0, 0, 1, 1, 1, 1]


def test_pyramid_rules(rule):
    got = rule("for (int l = 1; l <= 6; ++l) for (int n : {1, 128, 129, 4000}) printf(\"%d \", default_pyr_tile(n, l));")
    assert got == 4 * [32, 32, 64, 64] + 2 * [64, 64, 64, 64]
    # the largest split launch whose joined one has 300 workgroups, and 200
    body = ("for (int j : {300, 200}) for (int t : {32, 64}) for (int l = 1; l <= 6; ++l) { int m = 0;"
            "for (int s = 1; s < 5000; ++s) if (split_pyramid(s, j, t, l, 256)) m = s; printf(\"%d \", m); }")
    small = [1024] * 4 + [768, 512]
    assert rule(body) == small + [512] * 4 + [256] * 2 + small + [384] * 4 + [256] * 2


def test_upload_rule(rule):
    got = rule("for (bool among : {false, true}) for (int c : {1, 2, 4}) for (int b : {262143, 262144, 393215, 393216, 786432})"
               " printf(\"%d \", split_upload(b, c, among));")
    assert got == 3 * [0, 1, 1, 1, 1] + [0, 0, 0, 0, 0] + [0, 0, 0, 0, 1] + [0, 0, 0, 1, 1]


def kernels_of(step):
    """Names of the library's kernels that step() launches."""
    import torch
    from torch.profiler import ProfilerActivity, profile
    with profile(activities=[ProfilerActivity.CUDA]) as p:
        step()
        torch.cuda.synchronize()
    return [m.group(1) for e in p.events() for m in [re.search(r"(k_\w+(?:<[^>]*>)?)\(", e.name)] if m]


@pytest.mark.gpu
@pytest.mark.parametrize("n,extra,name", [
    (1, {}, "k_track<4, false>"), (4, {}, "k_track<4, false>"), (5, {}, "k_track2<4>"),
    (2, dict(levels=5), "k_track<5, false>"), (3, dict(levels=5), "k_track2<5>"), (3, dict(levels=6), "k_track2<6>"),
    (3, dict(levels=5, track_kp_per_wave=1), "k_track<5, false>"),
    (5, dict(track_kp_per_wave=1), "k_track<4, false>"), (1, dict(track_kp_per_wave=2), "k_track2<4>"),
    (5, dict(track_waves_per_cu=4), "k_track_persistent<4, false>"),
    (1, dict(track_waves_per_cu=4, track_kp_per_wave=2), "k_track2_persistent<4>")])
def test_keypoints_per_wave_taken(n, extra, name):
    """Streams of 1,300 items (2 x 400 tracks, 500 possible matches)."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_30459_amd as vf
    seq = synthgen.render(seed=11, width=400, height=305, n_frames=3, stereo=True, density=8.0, max_scale=0.02)
    p = dict(max_keypoints=400, cell_size=16)
    other = dict(extra, track_kp_per_wave=1 if "track2" in name else 2)
    with vf.Frontend([(2, 400, 305)] * n, vf.make_params(**p, **extra)) as a, \
            vf.Frontend([(2, 400, 305)] * n, vf.make_params(**p, **other)) as b:
        for t in range(3):
            ks = []
            for fe in (a, b):
                for s in range(n):
                    fe.stage_frame(s, t + 1, list(seq.frames[(t + s) % 3]))
                if t == 1:
                    ks.append([k for k in kernels_of(fe.step) if k.startswith("k_track")])
                else:
                    fe.step()
            if t == 1:
                assert ks[0] == [name] and ks[1] != [name], ks
            for s in range(n):
                ra, rb = a.get_tracks(s), b.get_tracks(s)
                assert len(ra) > 100 and ra.tobytes() == rb.tobytes(), (t, s)


@pytest.mark.gpu
@pytest.mark.parametrize("cams,w,h,levels,name", [
    (1, 320, 240, 4, "k_pyr_detect<4, 32, 256>"), (1, 320, 240, 5, "k_pyr_detect<5, 64, 1024>"),
    (1, 320, 240, 6, "k_pyr_detect<6, 64, 1024>"), (2, 1280, 720, 4, "k_pyr_detect<4, 64, 1024>"),
    (2, 1920, 1080, 4, "k_pyr_detect<4, 64, 512>"), (2, 1920, 1080, 6, "k_pyr_detect<6, 64, 1024>")])
def test_pyramid_taken(cams, w, h, levels, name):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_30459_amd as vf
    dev = torch.randint(0, 256, (cams, h, w), dtype=torch.uint8, device="cuda")
    with vf.Frontend([(cams, w, h, 300, 48)], vf.make_params(levels=levels)) as fe:
        ks = kernels_of(lambda: fe.push_stereo_frame_device(0, 1, list(dev)))
    assert [k for k in ks if k.startswith("k_pyr")] == [name], ks
