"""The library's rounding of Phi0 + delta (compiled for the host), exact and as the
grid pass decides it from a float32 delta with an error bound, against exact
rational round-half-to-even, including .5 ties and tiny deltas."""
import math
import os
import shutil
import struct
import subprocess
from fractions import Fraction

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _rne(x: Fraction) -> int:
    fl = math.floor(x)
    d = x - fl
    if d != Fraction(1, 2):
        return fl + (1 if d > Fraction(1, 2) else 0)
    return fl if fl % 2 == 0 else fl + 1


def _compile(tmp_path_factory, name):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    exe = str(tmp_path_factory.mktemp("host") / name)
    src = os.path.join(ROOT, "tests", "host", name + ".hip")
    cmd = [hipcc, "--offload-arch=gfx950", "-O2", "-std=c++17", "-I", os.path.join(ROOT, "paper_2406_06385_amd", "csrc"),
           src, "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return exe


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    return _compile(tmp_path_factory, "grid_round_host")


def _cases():
    rng = np.random.default_rng(1)
    out = []
    for f in (0, 1, 4, 5, 6):
        codes = list(range(-128, 128)) if f else list(range(-8, 8))
        for code in codes:
            for d in (0.0, 1e-9, -1e-9, 2.0 ** -30, -(2.0 ** -30), 1e-6, -1e-6, 0.03, -0.03, 0.49, -0.51):
                out.append((code, f, np.float32(d)))
        # exact half-integer crossings and random deltas
        for _ in range(3000):
            code = int(rng.integers(-128, 128)) if f else int(rng.integers(-8, 8))
            d = np.float32(rng.normal(0, 0.3) if rng.random() < 0.5 else rng.normal(0, 1e-6))
            out.append((code, f, d))
        for code in (codes[0], codes[-1], 0, 1):
            for k in (-2, -1, 1, 2):
                # delta that lands exactly on a .5 point of u
                v = Fraction(code, 2 ** f)
                target = math.floor(v) + k + Fraction(1, 2)
                d = np.float32(float(target - v))
                if Fraction(float(d)) == target - v:
                    out.append((code, f, d))
    return out


def test_grid_round_matches_exact_rne(driver):
    cases = _cases()
    lines = "".join(f"{c} {f} {struct.unpack('<Q', struct.pack('<d', float(d)))[0]:x}\n" for c, f, d in cases)
    r = subprocess.run([driver], input=lines, capture_output=True, text=True)
    assert r.returncode == 0
    got = [int(line) for line in r.stdout.splitlines()]
    assert len(got) == len(cases)
    bad = [(c, f, float(d), g) for (c, f, d), g in zip(cases, got) if g != _rne(Fraction(c, 2 ** f) + Fraction(float(d)))]
    assert not bad, bad[:10]


@pytest.fixture(scope="module")
def decide_driver(tmp_path_factory):
    return _compile(tmp_path_factory, "grid_decide_host")


def _bits(x):
    return struct.unpack("<I", struct.pack("<f", float(np.float32(x))))[0]


def _decisions():
    """Four codes with their deltas, and the error bound of the deltas."""
    rng = np.random.default_rng(7)
    out = []
    for b, f in [(b, 8 - b) for b in (2, 3, 4, 5, 6, 7)] + [(2, 0), (3, 0), (4, 0)]:
        codes = list(range(-128, 128)) if f else list(range(-8, 8))
        pick = lambda: [int(c) for c in rng.choice(codes, 4)]
        for tz in (0.0, 1e-20, 3e-5, 0.01, 0.2):
            for code in codes:  # every code, in every byte, below and above its decision points
                for pos in range(4):
                    c, d = pick(), [float(x) for x in rng.normal(0, 0.1, 4)]
                    c[pos] = code
                    v = Fraction(code, 2 ** f)
                    point = math.floor(v) + Fraction(1, 2) + int(rng.integers(-1, 2))
                    d[pos] = float(point - v) + float(rng.choice([0.0, 1e-21, -1e-21, 1e-6, -1e-6, tz, -tz, 1.1 * tz, -1.1 * tz, 0.1]))
                    out.append((f, b, tz, c, d))
        for scale in (1e-30, 1e-5, 0.1, 0.4, 3.0, 60.0, 3e4, 1e6):
            for _ in range(200):
                tz = float(rng.choice([0.0, 1e-5, 1e-3])) * scale
                out.append((f, b, tz, pick(), [float(x) for x in rng.normal(0, scale, 4)]))
    return [(f, b, float(np.float32(tz)), c, [float(np.float32(x)) for x in d]) for f, b, tz, c, d in out]


def test_certain_decisions_hold_for_every_delta_within_the_bound(decide_driver):
    """What the grid pass decides from a float32 delta, on the byte-parallel path (where its regime holds and nothing
    clips) and on the rounding path, is round-half-even(code 2^-f + delta) for every delta within the error bound,
    unless it is marked for settling in float64; the clip marks are those of results past the grid."""
    cases = _decisions()
    lines = "".join(f"{f} {b} {_bits(tz):x} " + " ".join(f"{_bits(x):x} {c}" for x, c in zip(d, code)) + "\n"
                    for f, b, tz, code, d in cases)
    r = subprocess.run([decide_driver], input=lines, capture_output=True, text=True)
    assert r.returncode == 0
    rows = [line.split() for line in r.stdout.splitlines()]
    assert len(rows) == len(cases)
    sure = {"bytes": [0, 0], "rounding": [0, 0]}
    bad = []
    for (f, b, tz, codes, deltas), row in zip(cases, rows):
        lo, hi = -(1 << (b - 1)), (1 << (b - 1)) - 1
        regime, q, clip, sure1 = int(row[0]), int(row[1], 16), int(row[2], 16), int(row[3], 16)
        v2, sure2 = [int(x) for x in row[4:8]], int(row[8], 16)
        for j in range(4):
            u = Fraction(codes[j], 2 ** f) + Fraction(deltas[j])
            ends = {_rne(u - Fraction(tz)), _rne(u + Fraction(tz))}
            if regime:
                ok = sure1 >> j & 1
                sure["bytes"][ok] += 1
                got = q >> (8 * j) & (0xFF if b > 4 else 15)
                if ok and (clip >> (8 * j + 7) & 1) != int(max(ends) > hi):
                    bad.append(("clip", f, b, tz, codes[j], deltas[j], ends))
                elif ok and max(ends) <= hi and {e & (0xFF if b > 4 else 15) for e in ends} != {got}:
                    bad.append(("bytes", f, b, tz, codes[j], deltas[j], ends, got))
            ok = sure2 >> j & 1
            sure["rounding"][ok] += 1
            if ok and ends != {v2[j]}:
                bad.append(("rounding", f, b, tz, codes[j], deltas[j], ends, v2[j]))
    assert not bad, bad[:10]
    # both answers occur, and a bound that marked everything would pass for nothing
    assert all(min(n) > 1000 and n[1] > n[0] for n in sure.values()), sure


def test_an_exactly_zero_delta_rounds_phi0_half_to_even(decide_driver):
    """delta = 0 (B at its initialisation) is decided by the rounding path alone, ties and all."""
    cases = [(8 - b if fmt else 0, b, c) for b in range(2, 8) for fmt in ((1, 0) if b <= 4 else (1,))
             for c in (range(-128, 128) if fmt else range(-8, 8))]
    lines = "".join(f"{f} {b} 0 " + " ".join(f"0 {c}" for _ in range(4)) + "\n" for f, b, c in cases)
    r = subprocess.run([decide_driver], input=lines, capture_output=True, text=True)
    got = [[int(x) for x in line.split()[4:8]] for line in r.stdout.splitlines()]
    assert len(got) == len(cases)
    assert all(g == [_rne(Fraction(c, 2 ** f))] * 4 for (f, b, c), g in zip(cases, got))


def test_tile_cases_reach_their_tiles(tmp_path):
    """The GPU tests of the GEMM tiles run the tiles that they are meant to run."""
    tiles = pytest.importorskip("test_gpu_tiles")
    gxx = shutil.which("g++")
    if not gxx:
        pytest.skip("g++ not available")
    exe = str(tmp_path / "gemm_plan_host")
    cmd = [gxx, "-O1", "-std=c++17", "-I", os.path.join(ROOT, "paper_2406_06385_amd", "csrc"),
           os.path.join(ROOT, "tests", "host", "gemm_plan_host.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    run = {c[:3] + c[6:8] for c in tiles.CASES + tiles.LARGE} | {c[:3] + (c[6], 0) for c in tiles.DW}
    lines, want = [], []
    for (tm, tn, split), claims in tiles.REACHED.items():
        for gemm, m, k, T, group, act in claims:
            assert (m, k, T, group, act) in run
            kpad = -(-k // 256) * 256
            v, size, ld = {"fwd": (0, (T, m, k), (kpad if act else k, kpad // 2)), "dx": (1, (T, k, m), (m, kpad // 2)),
                           "dw": (2, (m, k, T), (m, kpad if act else k))}[gemm]
            lines.append(" ".join(str(x) for x in (v, int(bool(act) and v == 0), int(bool(group)), *size, *ld)))
            want.append(f"0 {tm} {tn} {split}")
    r = subprocess.run([exe], input="\n".join(lines) + "\n", capture_output=True, text=True)
    assert [(a, b) for a, b in zip(lines, r.stdout.splitlines())] == list(zip(lines, want))
