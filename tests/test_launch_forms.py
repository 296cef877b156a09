"""The form that a call's launch takes, asked from the library's rules on the CPU (tests/host/launch_forms.hip): what a rule
must not do, and that the GPU tests written for a form have shapes that take it."""
import os
import shutil
import subprocess

import pytest

import paper_2605_11744_amd as sa
from conftest import ROOT


@pytest.fixture(scope="module")
def forms(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not found")
    sa.lib()  # built, and says so if not
    pkg = os.path.join(ROOT, "paper_2605_11744_amd")
    exe = tmp_path_factory.mktemp("forms") / "launch_forms"
    subprocess.run([hipcc, "--offload-arch=gfx950", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(pkg, "csrc"), os.path.join(ROOT, "tests", "host", "launch_forms.hip"),
                    "-L", pkg, "-lsegattn", "-Wl,-rpath," + pkg, "-o", str(exe)], check=True, capture_output=True, timeout=600)

    def ask(lines):
        out = subprocess.run([str(exe)], input="\n".join(lines) + "\n", capture_output=True, text=True, timeout=600)
        assert out.returncode == 0, out.stdout + out.stderr
        got = out.stdout.splitlines()
        assert len(got) == len(lines)
        return got

    return ask


def decode_line(D, Hq, Hkv, policy, S, T, closed, fill):
    fill = [fill] * len(closed) if isinstance(fill, int) else fill
    text = lambda xs: ",".join(str(x) for x in xs)
    return f"decode {D} {Hq} {Hkv} {''.join(map(str, policy))} {S} {T} {S * (max(closed) + 1)} 512 {text(closed)} {text(fill)}"


def test_numbering_the_slices_of_a_decode_step_costs_no_second_round(forms):
    """Slices that have a compute unit each are not numbered where the numbers (with the empty ones of shorter windows) are more
    than there are compute units: two slices then share one while another idles."""
    uneven = [decode_line(128, 32, 8, (3, 3, 3, 3, 1, 1, 1, 1), 2048, 512, (5, 6), (1139, 1663)),
              decode_line(128, 32, 8, (2, 2, 1, 1, 1, 1, 1, 1), 4096, 1024, (4, 4), (2374, 3909))]
    assert [x.split()[1:] for x in forms(uneven)] == [["240", "264"], ["256", "280"]]
    assert [x.split()[0] for x in forms(uneven)] == ["searched"] * 2
    # two sequences of every pair of lengths: never from one round of workgroups to two
    pairs = [decode_line(D, 32, 8, (3, 3, 3, 3, 1, 1, 1, 1), 2048, 512, (a, b), (700, 1500))
             for D in (64, 128) for a in range(12) for b in range(12)]
    kinds = set()
    for answer in forms(pairs):
        form, slices, numbers = answer.split()
        kinds.add(form)
        assert form != "numbered" or int(numbers) <= 256 or int(slices) > 256, answer
    assert kinds >= {"numbered", "searched"}


def chunk_line(D, Hq, Hkv, policy, S, T, closed, fill, m):
    text = lambda xs: ",".join(str(x) for x in xs)
    return (f"chunk {D} {Hq} {Hkv} {''.join(map(str, policy))} {S} {T} {S * (max(closed) + 1)} {m} {text(closed)} "
            f"{text([fill] * len(closed))}")


def test_pieces_in_the_key_split_form_only_where_memory_lets_them(forms):
    """Chunks whose 32-column workgroups would read the same keys over and over from beyond the L2s keep the pipelined pieces;
    short ones, and few heads' worth of keys, take the key-split ones."""
    bound = [chunk_line(128, 16, 2, (3, 1), 4096, 1024, (14,), 2085, 25),
             chunk_line(128, 8, 8, (3, 3, 1, 1, 1, 1, 1, 1), 4096, 512, (14,), 234, 137),
             chunk_line(128, 4, 1, (3,), 2048, 512, (13, 13, 13), 1019, 34),
             chunk_line(128, 8, 1, (3,), 4096, 1024, (15,), 273, 29),
             chunk_line(128, 4, 1, (3,), 4096, 512, (23, 23), 1634, 29),
             chunk_line(64, 32, 8, (3, 3, 3, 3, 3, 1, 1, 1), 1024, 128, (29,) * 6, 616, 17),
             chunk_line(64, 24, 4, (2, 2, 2, 1), 1024, 128, (62,) * 3, 625, 21),
             chunk_line(64, 16, 4, (3, 3, 3, 1), 1024, 128, (59,) * 6, 678, 57)]
    assert [x.split()[0] for x in forms(bound)] == ["piped"] * len(bound)
    assert all(int(x.split()[2]) > 1 for x in forms(bound))
    short = [chunk_line(128, 16, 2, (3, 1), 4096, 1024, (7,), 2085, 8),
             chunk_line(128, 16, 4, (3, 1, 1, 1), 4096, 1024, (10, 10, 10), 2085, 34),
             chunk_line(64, 16, 4, (3, 1, 1, 1), 4096, 1024, (6,), 300, 26),
             chunk_line(128, 8, 8, (3, 3, 1, 1, 1, 1, 1, 1), 4096, 512, (9,), 670, 76),  # 35 us, pipelined 40
             chunk_line(128, 4, 1, (3,), 2048, 256, (11,) * 3, 903, 22),                 # 33, 36
             chunk_line(128, 32, 8, (3, 3, 3, 3, 1, 1, 1, 1), 4096, 1024, (6,), 300, 1)]
    assert [x.split()[0] for x in forms(short)] == ["keysplit"] * len(short)
    assert all(int(x.split()[2]) > 1 for x in forms(short))


def test_short_prefixes_are_not_cut_where_the_uncut_launch_is_shorter(forms):
    """Chunks behind less than a segment: the uncut launch's own estimate counts, not the one for long prefixes."""
    short = [chunk_line(128, 8, 8, (3, 1, 1, 1, 1, 1, 1, 1), 2048, 512, (0,), 556, 9),
             chunk_line(128, 8, 8, (3, 3, 3, 3, 1, 1, 1, 1), 2048, 256, (0, 0), 403, 184)]
    assert [x.split()[2:] for x in forms(short)] == [["1", "1"]] * 2
    few = [chunk_line(64, 3, 3, (1, 1, 1), 1024, 128, (51,), 641, 3), chunk_line(64, 2, 1, (0,), 2048, 256, (10,) * 4, 749, 4)]
    assert [x.split()[2:] for x in forms(few)] == [["1", "1"]] * 2
    assert forms([chunk_line(128, 24, 8, (3,) * 8, 1024, 256, (50,) * 6, 269, 5)]) == ["keysplit 8 1 1"]  # two rounds of pieces


def test_longer_prefixes_are_cut_where_the_uncut_launch_only_seems_shorter(forms):
    """A workspace that holds too few pieces for the pipelined form, some for the key-split one."""
    longer = [chunk_line(128, 32, 8, (3, 3, 3, 3, 1, 1, 1, 1), 4096, 1024, (1, 1, 1), 2811, 14),
              chunk_line(128, 32, 8, (3, 3, 1, 1, 1, 1, 1, 1), 4096, 1024, (1, 1, 1), 3188, 11),
              chunk_line(128, 16, 2, (3, 1), 2048, 512, (1, 1, 1), 1180, 5),
              chunk_line(128, 32, 8, (3, 1, 3, 1, 1, 1, 1, 1), 4096, 1024, (2,) * 4, 300, 19),
              chunk_line(128, 40, 8, (2,) * 7 + (1,), 512, 64, (46,) * 6, 503, 3)]
    assert [(x.split()[0], int(x.split()[2]) > 1) for x in forms(longer)] == [("keysplit", True)] * len(longer)


def window_line(D, Hq, Hkv, policy, S, T, B, n, total=0):
    return f"window {D} {Hq} {Hkv} {''.join(map(str, policy))} {S} {T} {B} {n} {total}"


def test_one_launch_backward_only_where_two_launches_are_not_faster(forms):
    """Head dimension 64, one or two KV heads: windows whose longest chain the eight waves of the two split launches share out."""
    faster_in_two = [window_line(64, 4, 1, (3,), 128, 32, 1, 3678),         # 35 us, 69 in one launch
                     window_line(64, 4, 1, (3,), 512, 0, 1, 2964),          # 36, 58
                     window_line(64, 8, 2, (3, 3), 128, 16, 1, 1616),       # 27, 35
                     window_line(64, 12, 1, (1,), 1024, 256, 1, 677),       # 52, 60
                     window_line(64, 16, 1, (3,), 512, 128, 1, 1013),
                     window_line(64, 16, 1, (1,), 2048, 256, 1, 4096),
                     window_line(64, 16, 1, (1,), 512, 128, 1, 1024),
                     window_line(64, 8, 1, (1,), 512, 128, 1, 1024),
                     window_line(64, 8, 1, (3,), 2048, 256, 1, 1024)]
    assert [x.split()[0] == "both" for x in forms(faster_in_two)] == [False] * len(faster_in_two)
    faster_in_one = [window_line(64, 16, 4, (3, 3, 1, 1), 512, 128, 8, 2100, 6547),
                     window_line(64, 32, 8, (3, 1) * 4, 1024, 256, 1, 1500),
                     window_line(64, 16, 4, (3, 1, 1, 1), 2048, 512, 1, 3000),
                     window_line(64, 4, 1, (1,), 1024, 128, 1, 1500),
                     window_line(64, 8, 1, (3,), 512, 128, 1, 4096),
                     window_line(64, 16, 1, (3,), 512, 128, 1, 4096),
                     window_line(128, 16, 4, (3, 1, 1, 1), 512, 128, 1, 747),
                     window_line(128, 16, 2, (3, 1), 2048, 512, 2, 1402)]
    assert [x.split()[0] for x in forms(faster_in_one)] == ["both"] * len(faster_in_one)


def test_long_uncut_chains_of_head_dimension_64_have_sixteen_waves(forms):
    from test_gpu_keysplit import LONG
    from test_gpu_turn import CASES
    sixteen = [c for c in CASES if c[0] == 64 and c[6] in ((8,), (4,)) and c[8] in (33, 40, 68)]
    assert [c[1] // c[2] for c in sixteen] == [4, 1, 2]  # every number of query heads of a workgroup
    assert forms([chunk_line(*c) for c in sixteen]) == ["keysplit 16 1 1"] * 3
    assert forms([f"prompt 64 {g} 1 1 {S} {T} 1 {n}" for n, S, T, g in LONG]) == ["keysplit 16"] * len(LONG)
    others = [chunk_line(64, 16, 4, (1, 1, 1, 1), 2048, 512, (8,), 11, 68),          # a short chain
              chunk_line(64, 16, 4, (3, 1, 1, 1), 2048, 512, (8,) * 8, 11, 68)]      # more workgroups than compute units
    assert [x.split()[:2] for x in forms(others)] == [["keysplit", "8"]] * 2


def test_backward_shapes_take_the_forms_they_were_written_for(forms):
    """Every split form of dQ, and the split dK/dV form by itself, with each number of query heads a workgroup can have."""
    from test_gpu_backward_split import ONE_LAUNCH_PACKED, TWO_LAUNCHES, TWO_LAUNCHES_PACKED
    dense = forms([window_line(D, len(policy) * g, len(policy), policy, S, T, B, n) for D, g, S, T, policy, B, n, _ in TWO_LAUNCHES])
    assert dense == [case[-1] + " dense" for case in TWO_LAUNCHES]
    packed = forms([window_line(D, len(policy) * g, len(policy), policy, S, T, len(lens), max(lens), sum(lens))
                    for D, g, S, T, policy, lens, _ in TWO_LAUNCHES_PACKED + ONE_LAUNCH_PACKED])
    assert packed == [case[-1] + " packed" for case in TWO_LAUNCHES_PACKED + ONE_LAUNCH_PACKED]
    split = {(case[0], x.split()[0], x.split()[2], x.split()[3]) for cases, got in ((TWO_LAUNCHES, dense), (TWO_LAUNCHES_PACKED, packed))
             for case, x in zip(cases, got)}
    assert split >= {(D, "split", hs, how) for D in (64, 128) for hs in "124" for how in ("dense", "packed")}
    both = [window_line(D, g, 1, (3,), S, T, 2, n) for D, g in ((64, 8), (128, 2), (128, 8)) for n, S, T in ((31, 64, 8), (129, 128, 128), (430, 200, 64))]
    assert {x.split()[0] for x in forms(both)} == {"both"}


def test_decode_shapes_find_their_slices_in_every_way(forms):
    from test_gpu_decode_partials import CASES
    got = [x.split()[0] for x in forms([decode_line(*c) for c in CASES])]
    assert got == ["even"] * 4 + ["numbered"] * 3 + ["searched"] * 3


def test_turn_shapes_take_the_forms_they_were_written_for(forms):
    from test_gpu_turn import CASES
    got = [x.split() for x in forms([chunk_line(*c) for c in CASES])]
    for case, (form, waves, first, other) in zip(CASES, got):
        if case[8] <= 9 and max(case[6]) >= 20:  # the short chunks
            assert form == "keysplit" and waves == "8" and int(first) > 1, case
    pieces = {(c[0], c[1] // c[2]) for c, x in zip(CASES, got) if x[0] == "keysplit" and int(x[2]) > 1}
    assert pieces >= {(D, g) for D in (64, 128) for g in (1, 2, 4)}
    assert ["keysplit", "8", "1", "1"] in [x for c, x in zip(CASES, got) if c[0] == 64]
    assert any(x[0] == "piped" and int(x[2]) > 1 for x in got)
