"""The rules that choose launches of several steps (mdf_internal.h) and the
kernel of a convolution (nn_rules.h), asked on the CPU through a small program
built from those headers."""
import os
import shutil
import subprocess

import pytest

from paper_2108_08591_amd import mdf

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM = "/opt/rocm"
STRIPS, SMALL, LARGE = 0, 1, 2
STORAGES = [mdf.F64, mdf.F32, mdf.F16DEV, mdf.BF16DEV]

pytestmark = pytest.mark.skipif(shutil.which("g++") is None or not os.path.exists(f"{ROCM}/include/hip"),
                                reason="g++ or the HIP headers not available")


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("rules") / "launch_rules")
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I", f"{ROCM}/include",
                    "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2108_08591_amd", "csrc"),
                    "-o", exe, os.path.join(ROOT, "tests", "native", "launch_rules.cpp")], check=True)

    def run(*questions):
        text = "\n".join(" ".join(str(int(w)) if not isinstance(w, str) else w for w in q) for q in questions)
        r = subprocess.run([exe], input=text, capture_output=True, text=True, check=True)
        return [[float(v) for v in line.split()] for line in r.stdout.splitlines()]
    return run


def test_five_steps_only_where_the_kernel_keeps_its_registers(ask):
    """Five steps per launch in FP32 strips of plain cases; four with obstacles,
    a force field or Scheme II, whose five-step kernels spill, and elsewhere."""
    qs = [(c, s, m, g) for c in (STRIPS, SMALL, LARGE) for s in STORAGES for m in (0, 1) for g in (0, 1)]
    got = ask(*[("most",) + q for q in qs])
    for (c, s, m, g), (most,) in zip(qs, got):
        assert most == (5 if (c, s, m, g) == (STRIPS, mdf.F32, 0, 0) else 4), (c, s, m, g)


def test_two_steps_in_plain_16_bit_launches_near_the_cache(ask):
    """Two steps per launch for all sets of the 16-bit formats in large tiles of
    more than 3.5 million nodes, without mask, walls, fields and force; tiles
    of up to four steps elsewhere."""
    for lattice_pops in ((3, 15), (3, 12), (2, 10), (2, 8)):
        for c in (STRIPS, SMALL, LARGE):
            for s in STORAGES:
                base = [lattice_pops[0], lattice_pops[1], 3500001, 0, 0, 0, 0]
                others = [base[:i] + [v] + base[i + 1:]
                          for i, v in ((2, 3500000), (3, 1), (4, 1), (5, 1), (6, mdf.FIELD_VORT))]
                got = ask(*[("two", c, s, *w) for w in [base] + others])
                assert got[0] == [c == LARGE and s in (mdf.F16DEV, mdf.BF16DEV) and lattice_pops[0] == 3], (c, s)
                assert not any(v[0] for v in got[1:]), (c, s)


def test_two_steps_where_fp64_accumulates_many_channels(ask):
    """Two steps per launch in FP64 large tiles where more than one and a half
    channels per population are accumulated, or ten and more on small grids."""
    channels = {mdf.FIELD_MOMENTS: 4, mdf.FIELD_GRAD: 4, mdf.FIELD_DIV: 1, mdf.FIELD_STRAIN: 3, mdf.FIELD_STRESS: 3,
                mdf.FIELD_VORT: 1}
    qs = [(c, s, sets, pops, nodes, m, g, wall, f | acc) for c in (STRIPS, SMALL, LARGE) for s in (mdf.F64, mdf.F32)
          for sets, pops in ((3, 15), (3, 12), (2, 10), (2, 8)) for m, g, wall in ((0, 0, 0), (1, 0, 1), (0, 1, 0))
          for nodes in (100000, 100001, 3200000 // pops, 3200000 // pops + 1, 2 ** 31)
          for f in range(mdf.FIELD_ALL + 1) for acc in (0, mdf.FIELD_ACCUMULATE)]
    for (c, s, sets, pops, nodes, m, g, wall, f), (two,) in zip(qs, ask(*[("two",) + q for q in qs])):
        n = sum(v for bit, v in channels.items() if f & bit)
        many = n > 1.5 * pops or (n >= 10 and 100000 < nodes <= 3200000 // pops)
        assert two == (c == LARGE and s == mdf.F64 and not g and bool(f & mdf.FIELD_ACCUMULATE) and many)


def test_steps_of_a_call(ask):
    """A call's launches take all of its steps, at most `most` each, the last
    one alone, and no others alone but in a call of two: the two steps before
    the last of three run as one launch."""
    ks = {}
    for most in (4, 5):
        nxt = [int(v[0]) for v in ask(*[("next", left, most) for left in range(1, 301)])]
        for n in range(1, 301):
            seq, left = [], n
            while left > 0:
                seq.append(nxt[left - 1])
                left -= seq[-1]
            assert left == 0 and seq[-1] == 1 and max(seq) <= most, (n, most, seq)
            assert seq[:-1].count(1) == (1 if n == 2 else 0), (n, most, seq)
            assert len(seq) - 1 == (n - 1 + most - 1) // most, (n, most, seq)
            ks[n, most] = seq
    assert ks[3, 4] == ks[3, 5] == [2, 1]
    assert ks[6, 4] == [3, 2, 1] and ks[6, 5] == [5, 1] and ks[5, 4] == [4, 1]


def test_units_of_a_batch(ask):
    """The grid of a batched launch covers the running cases' units, at most
    twice over and never more than all units; small cases run in small tiles
    whatever else the batch holds."""
    qs = [(a, b) for b in (1, 7, 93000, 2 ** 30 + 5) for a in (1, 2, 3, 5, 64, 46501, 92999, 93000, 2 ** 30 + 5) if a <= b]
    for (a, b), (g,) in zip(qs, ask(*[("grid",) + q for q in qs])):
        assert a <= g <= b and (g == b or g < 2 * a), (a, b, g)
    for st in STORAGES:
        for beyond in (0, 1):
            most = 73728 if st in (mdf.F64, mdf.F32) else 65536
            assert ask(("cover", 128 * 128, st, beyond), ("cover", most, st, beyond)) == [[SMALL], [SMALL]]
            assert ask(("cover", most + 1, st, beyond)) == [[STRIPS if beyond and st != mdf.F64 else LARGE]]


def test_accumulated_fields_are_not_emitted_from_strips(ask):
    for cover in (STRIPS, SMALL, LARGE):
        plain, acc = ask(("emit", cover, mdf.FIELD_ALL), ("emit", cover, mdf.FIELD_VORT | mdf.FIELD_ACCUMULATE))
        assert plain == [cover] and acc == [LARGE if cover == STRIPS else cover]


TILE, RUN32, RUN64, LDS = 0, 1, 2, 3


def test_kernel_of_a_convolution(ask):
    """Sizes whose fastest kernel is known by a wide margin (times in nn_rules.h),
    with a bias, with a mask and with neither, and either side of every line."""
    bias, mask, none, f32 = (1, 0, 0), (0, 1, 0), (0, 0, 0), (0, 0, 1)
    known = [((8, 512, 64, 256, 128), bias, LDS), ((8, 512, 64, 256, 128), mask, LDS), ((3, 512, 64, 256, 128), mask, LDS),
             ((16, 64, 64, 384, 128), bias, LDS), ((16, 32, 32, 256, 256), bias, RUN64),
             ((1, 32, 32, 256, 256), bias, RUN32), ((16, 64, 64, 64, 256), mask, RUN64), ((16, 128, 128, 64, 128), mask, RUN64),
             ((1, 1024, 64, 512, 64), bias, LDS), ((16, 128, 128, 192, 64), bias, LDS), ((16, 128, 128, 192, 64), mask, RUN64),
             ((16, 128, 128, 64, 64), mask, RUN64), ((16, 256, 256, 96, 32), bias, LDS), ((8, 128, 128, 128, 32), bias, RUN32),
             ((1, 32, 32, 64, 64), bias, RUN32), ((16, 256, 256, 32, 32), bias, TILE), ((16, 128, 128, 32, 64), mask, TILE),
             ((1, 8, 8, 32, 256), bias, TILE)]
    # inputs, outputs, runs of 128 pixels, options, kernels there and one run on
    lines = [(128, 128, 640, bias, RUN64, LDS), (128, 128, 768, bias, LDS, RUN64), (128, 128, 1279, mask, RUN64, LDS),
             (192, 128, 639, bias, RUN64, LDS), (192, 128, 1023, mask, RUN64, LDS), (256, 128, 639, mask, RUN64, LDS),
             (288, 128, 511, bias, RUN64, LDS), (128, 128, 511, none, RUN64, LDS), (384, 128, 383, none, RUN64, LDS),
             (64, 128, 640, bias, RUN64, LDS), (64, 128, 768, bias, LDS, RUN64), (64, 128, 1280, none, RUN64, LDS),
             (64, 128, 192, mask, RUN32, RUN64), (128, 64, 1280, bias, RUN64, LDS), (288, 64, 384, bias, RUN32, LDS),
             (288, 64, 512, bias, LDS, RUN64), (64, 64, 384, bias, RUN32, RUN64), (64, 64, 1280, f32, RUN64, LDS),
             (96, 32, 2047, bias, RUN32, LDS)]
    qs = [("conv",) + k + o for k, o, _ in known]
    for cin, cout, runs, o, _, _ in lines:
        qs += [("conv", 1, runs + more, 128, cin, cout) + o for more in (0, 1)]
    want = [w for _, _, w in known] + [w for line in lines for w in line[4:]]
    got = [int(v[0]) for v in ask(*qs)]
    assert got == want, [(q, g, w) for q, g, w in zip(qs, got, want) if g != w]


def test_default_form_in_3d(ask):
    """The grids that the rule's comment cites: their fill as the plan gives it
    and the form it chooses, which is the faster one but for the 64^3 cube."""
    cited = [(mdf.F64, 4, 0, (40, 40, 250), 0.51, 0), (mdf.F64, 4, 0, (72, 88, 120), 0.58, 1),
             (mdf.F64, 4, 0, (64, 64, 64), 0.67, 1), (mdf.F64, 3, 0, (138, 148, 60), 0.73, 1),
             (mdf.F64, 4, 1, (130, 97, 75), 0.69, 0), (mdf.F64, 4, 1, (150, 65, 150), 0.83, 1),
             (mdf.F32, 3, 0, (80, 80, 80), 0.43, 0), (mdf.F32, 3, 0, (39, 223, 123), 0.45, 1),
             (mdf.F32, 3, 1, (138, 148, 60), 0.62, 1), (mdf.F32, 4, 1, (130, 97, 75), 0.56, 0),
             (mdf.F32, 4, 1, (138, 148, 60), 0.67, 1), (mdf.F32, 4, 0, (256, 256, 256), 0.94, 1)]
    plans = ask(*[("plan", st, sets, 7) + dims for st, sets, _, dims, _, _ in cited])
    pays = ask(*[("pays", st, sets, 7, w) + dims for st, sets, w, dims, _, _ in cited])
    for (st, sets, w, dims, fill, two), (zc, f), (p,) in zip(cited, plans, pays):
        assert round(f, 2) == fill and p == two, (st, sets, w, dims, zc, f, p)
