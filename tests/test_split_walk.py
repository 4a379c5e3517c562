"""How a pass over K shares the keys out and where its requests lie, walked on the CPU: the header that the kernels take both from
also compiles for the host.  Every quad of 128 keys is taken once, every set of statistics has one writer, both passes visit
the same shares, and no request starts outside the sequence it reads."""
import os
import random
import subprocess

import pytest

import paper_2509_10798_amd as jq
from conftest import ROOT


def _compiled(tmp_path_factory, name):
    exe = str(tmp_path_factory.mktemp(name) / name)
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-Wall", "-Wno-unknown-pragmas", "-I" + os.path.join(ROOT, "include"),
                           "-I" + os.path.join(ROOT, "paper_2509_10798_amd", "csrc"), os.path.join(ROOT, "tests", name + ".cpp"), "-o", exe])
    return exe


@pytest.fixture(scope="module")
def walk(tmp_path_factory):
    exe = _compiled(tmp_path_factory, "split_walk")

    def run(calls):
        """calls: (n_layers, lens, h_kv, rows, rows2, chunk, every quad); returns (workgroups, sets, longest, quads) of each."""
        text = "".join("%d %d %d %d %d %d %d %s\n" % (nl, len(lens), h_kv, rows, rows2, chunk, full, " ".join(map(str, lens)))
                       for nl, lens, h_kv, rows, rows2, chunk, full in calls)
        r = subprocess.run([exe], input=text, capture_output=True, text=True, timeout=300)
        lines = r.stdout.splitlines()
        at = calls[len(lines)] if len(lines) < len(calls) else None
        assert r.returncode == 0 and at is None, "ended (%d) at %s" % (r.returncode, str(at)[:200])
        for call, line in zip(calls, lines):
            assert line.startswith("ok"), (line, str(call)[:200])
        return [tuple(map(int, line.split()[1:])) for line in lines]
    return run


def _call(rng):
    log = lambda lo, hi: int(round(lo * (hi / lo) ** rng.random()))
    nl, n_seq = log(1, 64), log(1, 128)
    top = max(2, min(300000, 40000000 // (nl * n_seq)))
    lens = [log(1, top) for _ in range(n_seq)] if rng.random() < 0.7 else [log(1, top)] * n_seq
    rows, rows2 = rng.choice(((16, 0), (128, 0), (128, 0), (500, 0), (128, 512), (32, 32)))
    return nl, lens, log(1, 256), rows, rows2, rng.choice((0, 0, 0, 0, 64, 2048)), 1


def test_every_key_is_taken_once(walk):
    rng = random.Random(12)
    walk([_call(rng) for _ in range(3000)])


# A paged cache may have its sequences share pages, so the keys of a call can be many times those in memory.
HUGE = [
    (3, [16000000] * 128, 1, 128, 0),   # 48 million quads: workgroup number times quads exceeds 32 bits
    (5, [8000000] * 127, 2, 128, 0),
    (1, [16777088] * 128, 1, 128, 0),   # 2^24 quads
    (128, [1000, 16000000], 1, 64, 0),
    (7, [16000000] * 33 + [1], 1, 128, 512),
]


def test_every_key_is_taken_once_in_the_largest_calls(walk):
    for (nl, lens, h_kv, rows, rows2), (n_wg, n_sets, longest, quads) in zip(HUGE, walk([c + (0, 0) for c in HUGE])):
        groups = ((rows + 31) // 32 + (rows2 + 31) // 32 + 3) // 4
        assert n_wg * h_kv * groups >= 250 and longest * 100 <= quads  # and the whole chip takes part


def test_the_chip_has_work_whatever_the_number_of_heads(walk):
    calls = [(1, [131072 if h_kv < 120 else 32768], h_kv, 64, 0, 0, 0) for h_kv in range(1, 257)]
    for (_, _, h_kv, _, _, _, _), (n_wg, n_sets, longest, quads) in zip(calls, walk(calls)):
        assert n_wg * h_kv >= 170, (h_kv, n_wg)  # of 256 CUs


def test_many_short_sequences_do_not_queue_in_one_workgroup_per_cu(walk):
    # several of them one after the other in one workgroup per CU leave the chip waiting for query rows and statistics
    calls = [(nl, [L] * n, h_kv, 128, 0, 0, 1) for nl, n, L, h_kv in ((32, 32, 512, 8), (1, 128, 1000, 8), (32, 8, 300, 8), (32, 1, 2048, 96), (100, 1, 700, 8))]
    for (nl, lens, h_kv, _, _, _, _), (n_wg, n_sets, longest, quads) in zip(calls, walk(calls)):
        assert n_wg * h_kv > 256, (nl, len(lens), h_kv, n_wg)


def test_long_sequences_of_few_heads_leave_sets_that_need_no_merge_launch(walk):
    calls = [(1, [L], h_kv, 128, 0, 0, 1) for L, h_kv in ((16384, 1), (24000, 2), (40000, 3))]
    for _, n_sets, _, _ in walk(calls):
        assert n_sets <= 64


def test_workspace_of_a_call_that_no_card_holds():
    # 2^32 quads: what a portion is divided by used to come out as zero
    sh = jq.Shape(n_layers=32768, seq_lens=[131072] * 128, n_q=32, h_q=4, h_kv=1)
    assert jq.workspace_bytes(sh) > 32768 * 128 * 131072 * 8


def test_no_request_starts_outside_what_it_reads(tmp_path_factory):
    r = subprocess.run([_compiled(tmp_path_factory, "request_walk")], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout == "ok\n", r.stdout
