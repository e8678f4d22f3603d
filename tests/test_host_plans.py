"""The host side's memory plans, without a GPU: the built library against a stand-in for the HIP
calls (fake_hip.cpp), in a process of its own, in which kernels do nothing and every solve ends at
once.  Checked is what the library allocates and what it does when that fails."""
import json
import os
import re
import subprocess
import sys

import pytest

from paper_2604_22625_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))

PRELUDE = """
import ctypes, json, os, sys
sys.path.insert(0, {root!r})
fake = ctypes.CDLL({fake!r}, mode=ctypes.RTLD_GLOBAL)
fake.fake_log.restype = ctypes.c_char_p
fake.fake_limit.argtypes = fake.fake_allow.argtypes = [ctypes.c_size_t]
READ = ctypes.CFUNCTYPE(None, ctypes.c_void_p, ctypes.c_size_t)
import paper_2604_22625_amd as ff
L, p, INFOS = ff.lib(), ctypes.c_void_p(0x1000), [None]      # p: device arrays, never read

def options(**kw):
    o = ff.default_options()
    for k, v in kw.items():
        setattr(o, k, v)
    return ctypes.byref(o)

def solve(n, m, T=0, **kw):
    return L.ffo_solve(n, 0, m, T, p, None, None, p, p, p, 1.5, p, p, p, p, 1e9, 1e-9, 1.0, 1.0, p if T else None,
                       options(verbose=1, **kw), None, p, None, ctypes.byref(ff._Info()))

def many(sizes, m, **kw):
    B, P = len(sizes), ctypes.c_void_p * len(sizes)
    a = P(*[0x1000] * B)
    return L.ffo_solve_many(B, (ctypes.c_int64 * B)(*sizes), 0, m, 0, a, None, None, a, a, a, a, a, a, a, None, 1.5, 1e9, 1e-9,
                            1.0, 1.0, options(verbose=1, **kw), None, a, (ff._Info * B)())

def batched(sizes, m, **kw):
    B = len(sizes)
    INFOS[0], W = (ff._Info * B)(), ctypes.create_string_buffer(8 * sum(sizes))
    nb, offs = (ctypes.c_int64 * B)(*sizes), (ctypes.c_int64 * (B + 1))(0)
    for b in range(B):
        offs[b + 1] = offs[b] + nb[b]
    return L.ffo_solve_batched(B, nb, max(sizes), 0, m, None, None, p, p, offs, p, p, p, p, p, p, 1.5, 1e9, 1e-9, 1.0, 1.0,
                               options(verbose=1, **kw), None, W, INFOS[0]), [(i.status, i.iters) for i in INFOS[0]]

"""


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("fake") / "libfake_hip.so")
    subprocess.run([build.hipcc(), "-O1", "-fPIC", "-shared", "--offload-host-only", "-o", out, os.path.join(HERE, "fake_hip.cpp")],
                   check=True, capture_output=True)
    return out


def _run(fake, body):
    """The value of `out` that the body leaves, the stand-in's calls and the standard error."""
    code = (PRELUDE.format(root=os.path.dirname(HERE), fake=fake) + body +
            "\nprint(json.dumps([out, fake.fake_log().decode()]), flush=True)\nsys.stderr.flush()\nos._exit(0)\n")
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr
    out, log = json.loads(r.stdout.splitlines()[-1])
    return out, [(w, int(v)) for w, v in (line.split() for line in log.splitlines())], r.stderr


@pytest.mark.parametrize("precision,floats", [(0, 0), (1, 1)])
def test_solve_without_room_for_tiles(fake, precision, floats):
    """n = 400,000, 60 rows: 192 MB of rows, about fifteen vectors, and the rows again in tiles
    (80 of them, with the padding of a tile) or, in FP32 without tiles, as floats."""
    out, log, err = _run(fake, f"""
out = [solve(400_000, 60, precision={precision})]
L.ffo_release()
fake.fake_limit(350_000_000)
out.append(solve(400_000, 60, precision={precision}))
""")
    sizes = [v for w, v in log if w == "malloc"]
    assert out == [0, 0], err
    assert [s.split()[0] for s in err.split("kernel ")[1:]] == ["tiles", "general"]
    assert len(sizes) == 3 and sizes[0] == sizes[1] >= 350_000_000
    rows, vectors = 60 * 400_000 * 8, 16 * 400_000 * 8
    assert rows < sizes[2] < rows + vectors + floats * rows // 2 + 2_000_000


def test_batch_without_room_for_iterates(fake):
    """200 instances of 7500 assets: a dozen vectors of 1.5 million entries, and 32 copies of two
    vectors for the hand-off."""
    out, log, err = _run(fake, """
out = [batched([7500] * 200, 10)[0]]
L.ffo_release()
fake.fake_limit(600_000_000)
out.append(batched([7500] * 200, 10)[0])
""")
    sizes = [v for w, v in log if w == "malloc"]
    assert out == [0, 0], err
    assert len(sizes) == 3 and sizes[0] == sizes[1] > 64 * 1_500_000 * 8
    assert sizes[2] < 13 * 1_500_000 * 8


def test_iterates_beyond_a_gibibyte_are_not_kept(fake):
    out, log, err = _run(fake, "out = [batched([7500] * 270, 10)[0], batched([7500] * 300, 10)[0]]")
    assert out == [0, 0], err
    assert [v for w, v in log if w == "malloc"][0] > 64 * 270 * 7500 * 8
    out, log, err = _run(fake, "out = batched([7500] * 300, 10)[0]")
    assert [v for w, v in log if w == "malloc"][0] < 13 * 300 * 7500 * 8


HAND_OFF = """
import struct
B, LEN = 8, {len}
def read(dst, n):       # the teams' records: instance b ended after 64 (b + 1) iterations, converged
    if n == B * LEN * 8:
        for b in range(B):
            ctypes.memmove(dst + b * LEN * 8, struct.pack("d", 64.0 * (b + 1)), 8)
cb = READ(read)
fake.fake_on_read(cb)
"""


@pytest.mark.parametrize("mallocs", [2, 1])
def test_hand_off_without_room_for_a_solve(fake, mallocs):
    """The four longest of eight converged instances go on from their iterates at 256 iterations, in
    a workspace of their own; where there is none left, they keep what their teams found."""
    info_len = int(re.search(r"INFO_LEN = (\d+)", open(os.path.join(build.CSRC, "internal.h")).read())[1])
    out, log, err = _run(fake, HAND_OFF.format(len=info_len) + f"fake.fake_allow({mallocs})\nout = batched([50] * 8, 10)")
    assert out[0] == 0, (out, err)
    assert sum(w == "malloc" for w, v in log) == (2 if mallocs == 2 else 5)     # (each instance tries)
    ended = [64 * (b + 1) for b in range(8)] if mallocs == 1 else [64, 128, 192, 256, 256, 256, 256, 256]
    assert out[1] == [[0, i] for i in ended]


@pytest.mark.parametrize("call,B", [("batched", 65_536), ("batched", 131_072), ("many", 65_536)])
def test_staging_grows_with_the_batch(fake, call, B):
    """Pinned tables: a record of about 1 KB an instance, and two words for each of its workgroups."""
    out, log, err = _run(fake, f"out = {call}([3] * {B}, 10)")
    assert (out[0] if call == "batched" else out) == 0, err
    assert sum(v for w, v in log if w == "host") < 1200 * B


def test_barrier_counts_past_32_bits(tmp_path):
    """The team barrier's comparisons about the wrap of its exchange counter (some hours into a
    solve): a workgroup waits until the last of its team has arrived, and no longer."""
    src = tmp_path / "wrap.hip"
    src.write_text(r"""
#include "team_exchange.h"
#include <cstdio>
int main() {
  for (int members : {2, 3, 20, 256})
    for (uint64_t e = (1ull << 32) / members - 3; e < (1ull << 32) + 3; e += e == (1ull << 32) / members + 3 ? (1ull << 32) - 6 - e : 1) {
      const uint32_t want = ffo::arrivals((uint32_t)e, members);
      for (int a = 0; a < 2 * members; ++a)
        if (ffo::reached((uint32_t)(e * members + a), want) != (a >= members)) return printf("%d %llu %d\n", members, (unsigned long long)e, a), 1;
      if (ffo::reached((uint32_t)e, (uint32_t)e + 1) || !ffo::reached((uint32_t)(e + 1), (uint32_t)e + 1)) return 2;
    }
  return 0;
}
""")
    exe = str(tmp_path / "wrap")
    r = subprocess.run([build.hipcc()] + build.flags() + ["-I", build.CSRC, "-o", exe, str(src)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
