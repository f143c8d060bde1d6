"""Launch-plan invariants checked on the host: the plan header is plain C++,
compiled here with g++, and every workgroup's decoded work item is checked
for range, uniqueness and workspace/LDS bounds."""
import os
import shutil
import subprocess

import pytest

from paper_2606_18394_amd import synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2606_18394_amd", "csrc")


def shapes():
    out = []
    for name in synth.WORKLOAD_ORDER:
        w = synth.WORKLOADS[name]
        out.append((w.B, w.N, w.Hq, w.Hkv, w.D, w.L, w.V))
    for B in [1, 3, 16]:
        for N in [1, 2, 17, 64, 65, 129, 512, 2048]:
            for Hq, Hkv in [(4, 4), (8, 2), (32, 8), (64, 8), (24, 8), (2, 1)]:
                for D in [64, 128]:
                    for L in [0, 1, 64, 1000, 32768]:
                        out.append((B, N, Hq, Hkv, D, L, 151936 if N < 100 else 1001))
    # around one, four and sixteen sequences per lane of the even split, and past it
    for B in [63, 64, 65, 200, 256, 257, 1000, 1024, 1025]:
        for Hq, Hkv in [(4, 1), (8, 2), (16, 8), (3, 3)]:
            for L in [64, 3000, 20000]:
                out.append((B, 3, Hq, Hkv, 128 if B % 2 else 64, L, 1001))
    # more key tiles than the even split takes
    out += [(1, 8, 4, 1, 64, 1 << 25, 1001), (3, 8, 4, 1, 64, (1 << 25) - 9, 1001)]
    # more row blocks than the split-KV sync region holds: no split
    out += [(64, 512, 64, 8, 128, 1000, 1001), (512, 64, 32, 8, 128, 32768, 1001)]
    return out


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_plans(tmp_path):
    exe = tmp_path / "plan_check"
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", CSRC,
                    os.path.join(ROOT, "tests", "native", "plan_check.cpp"), "-o", str(exe)],
                   check=True)
    data = "\n".join(" ".join(map(str, s)) for s in shapes()) + "\n"
    res = subprocess.run([str(exe)], input=data, capture_output=True, text=True)
    fails = [l for l in res.stdout.splitlines() if l.startswith("FAIL")]
    assert res.returncode == 0 and not fails, "\n".join(fails[:20]) + res.stdout[-300:]


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_plans_under_host_sanitizers(tmp_path):
    """The same checks with AddressSanitizer and UndefinedBehaviorSanitizer on
    the host planner (integer overflow in sizes, out-of-range indexing)."""
    exe = tmp_path / "plan_check_san"
    build = subprocess.run(["g++", "-O1", "-g", "-std=c++17", "-fsanitize=address,undefined",
                            "-fno-sanitize-recover=undefined", "-I", CSRC,
                            os.path.join(ROOT, "tests", "native", "plan_check.cpp"), "-o", str(exe)],
                           capture_output=True, text=True)
    if build.returncode != 0:
        pytest.skip("host sanitizer runtime not available: " + build.stderr[-200:])
    data = "\n".join(" ".join(map(str, s)) for s in shapes()) + "\n"
    res = subprocess.run([str(exe)], input=data, capture_output=True, text=True)
    fails = [l for l in res.stdout.splitlines() if l.startswith("FAIL")]
    assert res.returncode == 0 and not fails, "\n".join(fails[:20]) + res.stderr[-1000:]


def plans(tmp_path, cases):
    """The plan of each (B, N, Hq, Hkv, D, Lmax) as a dict of its numbers."""
    exe = tmp_path / "plan_check"
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", CSRC,
                    os.path.join(ROOT, "tests", "native", "plan_check.cpp"), "-o", str(exe)],
                   check=True)
    res = subprocess.run([str(exe)], input="".join(" ".join(map(str, c)) + " 1001\n" for c in cases),
                         capture_output=True, text=True, check=True)
    return [{k: int(v) for k, v in (f.split("=") for f in l.split()[1:])}
            for l in res.stdout.splitlines() if l.startswith("OK")]


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_few_rows_take_few_chunks(tmp_path):
    """With one 16-row tile per KV head one wave folds a whole fused merge, at 33
    to 44 KB/us: 383 chunks took 108 us where 42 take 23.  Few rows on a long
    cache keep enough workgroups to ask for its bytes all the same."""
    for p in plans(tmp_path, [(1, 1, 3, 3, 128, 24503), (1, 1, 3, 3, 128, 5618),
                              (3, 1, 6, 3, 64, 5495), (4, 1, 12, 3, 64, 24499),
                              (1, 2, 12, 3, 64, 3594), (2, 4, 4, 1, 128, 15042)]):
        assert p["S"] <= 64, p
    for p in plans(tmp_path, [(2, 4, 16, 8, 64, 80754), (1, 2, 64, 32, 64, 99422)]):
        assert p["slots"] * p["Hkv"] * p["nRB"] >= 256, p


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_few_more_chunks_than_sequences(tmp_path):
    """Ragged batches whose row blocks fill the GPU once only with a few chunks more
    than there are sequences: left whole they took 8 to 26% longer (3 x 433 nodes
    over 1121 rows 40.8 us in 4 chunks, 51.7 whole)."""
    for p in plans(tmp_path, [(3, 433, 32, 8, 128, 1600), (4, 389, 32, 8, 128, 2037),
                              (4, 391, 32, 8, 128, 2776), (6, 31, 64, 8, 128, 761),
                              (19, 12, 8, 8, 128, 454), (27, 22, 8, 8, 128, 777),
                              (52, 32, 32, 4, 128, 1746), (7, 86, 16, 8, 64, 896)]):
        assert p["slots"] > p["B"], p


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_batches_beyond_a_wave_still_split(tmp_path):
    """Long sequences of few KV heads are split on both sides of 64 sequences
    (one to a lane below, several above), up to 1024; those whose row blocks fill
    the GPU are not above 64."""
    split = [(B, N, Hq, Hkv, 128, L) for B in (63, 64, 65, 80, 200)
             for N, Hq, Hkv, L in ((33, 4, 1, 16384), (9, 4, 1, 3776), (3, 8, 1, 8192))
             if B * Hkv < 256]
    for p in plans(tmp_path, split):
        assert p["slots"] >= 2 * p["B"] and p["S"] > 1, p
    for p in plans(tmp_path, [(100, 1, 32, 8, 64, 7273), (1025, 1, 1, 1, 64, 4000)]):
        assert p["slots"] == 0 and p["S"] == 1, p


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_pack_rule(tmp_path):
    """Where the training mask packs several blocks into a workgroup, on both
    sides of the line: by blocks x KV heads, later for blocks of few rows and for
    many blocks of one example."""
    exe = tmp_path / "pack_check"
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", CSRC,
                    os.path.join(ROOT, "tests", "native", "pack_check.cpp"), "-o", str(exe)],
                   check=True)
    cases = [((1, 160, 16, 32, 8), 2), ((1, 159, 16, 32, 8), 0), ((1, 80, 16, 16, 16), 8),
             ((3, 559, 1, 8, 1), 0), ((1, 224, 2, 32, 8), 0), ((1, 226, 2, 32, 8), 16),
             ((1, 1584, 16, 1, 1), 0), ((1, 1863, 2, 2, 2), 16), ((1, 512, 16, 32, 8), 2),
             ((1, 2049, 16, 32, 8), 0), ((1, 512, 17, 32, 8), 0)]
    res = subprocess.run([str(exe)], input="".join(" ".join(map(str, c)) + "\n" for c, _ in cases),
                         capture_output=True, text=True, check=True)
    for (c, nb), line in zip(cases, res.stdout.splitlines()):
        got, packs, ws = map(int, line.split())
        assert got == nb, (c, got)
        if nb:
            assert packs == -(-c[1] // nb) and ws == 32768 + 4 * c[0] * c[1], (c, line)


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_accept_split_rule(tmp_path):
    """The acceptance scan's split count: the ~2048-workgroup target (at most
    16 splits, at least one full round of loads each), then down to half of
    it the count whose load slots are best used.  Checked against a plain
    re-derivation of that rule, and at the measured shapes: 512 rows of
    151936 bf16 logits take 2 splits (4 leave 23% of the slots empty), 128
    and 64 rows keep 10."""
    exe = tmp_path / "accept_split_check"
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", CSRC,
                    os.path.join(ROOT, "tests", "native", "accept_split_check.cpp"), "-o", str(exe)],
                   check=True)
    cases = [(1, 512, 151936, 2), (1, 128, 151936, 2), (1, 64, 151936, 2), (16, 64, 151936, 2),
             (1, 16, 1024, 4), (3, 100, 50000, 2), (1, 2048, 151936, 4), (7, 33, 32000, 4)]
    res = subprocess.run([str(exe)], input="".join(f"{b} {n} {v} {e}\n" for b, n, v, e in cases),
                         capture_output=True, text=True, check=True)
    got = {tuple(map(int, l.split()[:4])): int(l.split()[4]) for l in res.stdout.splitlines()}

    def rule(b, n, v, esize):
        rows, per_round = b * n, 512 * 4
        chunks = -(-v // (16 // esize))
        ns = min(16, max(1, -(-2048 // rows)), -(-chunks // per_round))
        ns = max(ns, 1)

        def fill(k):
            c = -(-chunks // k)
            return c / (-(-c // per_round) * per_round)
        best = ns
        for k in range(ns - 1, 0, -1):
            if 2 * k < ns:
                break
            if fill(k) > fill(best) + 1e-9:
                best = k
        return best
    for c in cases:
        assert got[c] == rule(*c), (c, got[c], rule(*c))
    assert got[(1, 512, 151936, 2)] == 2
    assert got[(1, 128, 151936, 2)] == 10 and got[(1, 64, 151936, 2)] == 10
