"""The text functions of the build by induced order, on the CPU: suffix types
and runs, preceding bases, later windows, compiled host-only from the kernels'
source and compared with a base-by-base reading of reads of every length
around the record and payload sizes.  And the vector registers of every
kernel: no 64-bit shift may take its amount from the last one allocated."""
import ctypes
import os
import re
import shutil
import subprocess

import numpy as np
import pytest

from conftest import ROOT
from paper_1401_7457_amd import build as pkg_build
from test_window_keys_cpu import _records

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
CSRC = os.path.join(ROOT, "paper_1401_7457_amd", "csrc")
needs_hipcc = pytest.mark.skipif(not (os.path.exists(HIPCC) or shutil.which(HIPCC)), reason="hipcc not available")


@pytest.fixture(scope="module")
def it(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("it") / "libit.so")
    subprocess.run([HIPCC, "-x", "hip", "--cuda-host-only", "-O2", "-std=c++17", "-fPIC", "-shared", "-I", CSRC,
                    "-I", os.path.join(ROOT, "include"), os.path.join(ROOT, "tests", "induced_types_host.cpp"),
                    "-o", so], check=True, capture_output=True)
    L = ctypes.CDLL(so)
    vp, u32, u64 = ctypes.c_void_p, ctypes.c_uint32, ctypes.c_uint64
    L.it_type.argtypes = [vp, u64, ctypes.POINTER(u32)]
    L.it_preceding.argtypes = [vp, u64, ctypes.c_int]
    L.it_preceding.restype = u32
    L.it_trim.argtypes = L.it_run.argtypes = [u32]
    L.it_trim.restype = L.it_run.restype = u32
    L.it_window.argtypes = [vp, u64, u32, ctypes.POINTER(u32)]
    L.it_window.restype = u64
    L.it_samples.argtypes = [vp, u64, u64, u64]
    L.it_samples.restype = u32
    L.it_masks.argtypes = [vp, u64, ctypes.POINTER(u32)]
    return L


def _payload(before, most, bits):
    """The nearest bases of `before` (nearest last) as a payload of at most `most` in `bits` bits."""
    n = min(len(before), most)
    v = 0
    for k in range(n):
        v |= int(before[len(before) - 1 - k]) << (2 * k)
    start = len(before) <= most
    if start and 2 * n + 1 >= bits:  # the start mark does not fit: one base fewer, more before it
        n, start = n - 1, False
        v &= (1 << (2 * n)) - 1
    return v | ((2 if start else 1) << (2 * n))


@needs_hipcc
@pytest.mark.parametrize("alphabet", ["ACGT", "AC", "A", "GT", "T"])
def test_types_payloads_and_windows(it, alphabet):
    rng = np.random.default_rng(ord(alphabet[-1]) + len(alphabet))
    lens = [int(x) for x in rng.choice([1, 2, 3, 7, 8, 14, 15, 16, 17, 25, 26, 27, 28, 29, 41, 42, 60, 90], size=60)]
    codes = rng.choice(["ACGT".index(c) for c in alphabet], size=sum(lens)).astype(np.uint8)
    ends = np.cumsum(lens)
    bounds = [(int(e) - n, int(e)) for e, n in zip(ends, lens)]
    recs = _records(codes, bounds)
    ptr = recs.ctypes.data_as(ctypes.c_void_p)
    out = (ctypes.c_uint32 * 4)()
    cl = ctypes.c_uint32()
    for a, b in bounds:
        r = codes[a:b]
        assert it.it_preceding(ptr, b, 1) == _payload(r, 15, 32)
        for p in range(a, b):
            run = 0
            while p + run + 1 < b and codes[p + run + 1] == codes[p]:
                run += 1
            s = p + run + 1 < b and codes[p + run + 1] > codes[p]
            it.it_type(ptr, p, out)
            assert (out[0], out[1], bool(out[2])) == (int(codes[p]), run, bool(s))
            if p > a:
                assert out[3] == codes[p - 1]
            pl = it.it_preceding(ptr, p, 0)
            assert pl == _payload(codes[a:p], 15, 32)
            assert it.it_trim(pl) == _payload(codes[a:p], 7, 15)
            if p > a:
                same = 1
                while same < min(p - a, 15) and codes[p - 1 - same] == codes[p - 1]:
                    same += 1
                assert it.it_run(pl) == same
            for depth in (0, 22, 47):
                if 0 < depth <= b - p:
                    for full in (22, 25):
                        w = it.it_window(ptr, p + depth, full, ctypes.byref(cl))
                        n = min(b - p - depth, full)
                        want = 0
                        for k in range(n):
                            want |= int(codes[p + depth + k]) << (62 - 2 * k)
                        assert (w, cl.value) == (want, n)


@needs_hipcc
@pytest.mark.parametrize("alphabet", ["ACGT", "AC", "A", "GT", "T"])
def test_samples_of_whole_records(it, alphabet):
    """Sixteen positions at once against one at a time, for every run of positions a tile may hold."""
    rng = np.random.default_rng(7 + ord(alphabet[-1]) + len(alphabet))
    lens = [int(x) for x in rng.choice([1, 2, 5, 15, 16, 17, 31, 32, 33, 40, 48, 70, 100], size=50)]
    codes = rng.choice(["ACGT".index(c) for c in alphabet], size=sum(lens)).astype(np.uint8)
    ends = np.cumsum(lens)
    bounds = [(int(e) - n, int(e)) for e, n in zip(ends, lens)]
    recs = _records(codes, bounds)
    ptr = recs.ctypes.data_as(ctypes.c_void_p)
    out = (ctypes.c_uint32 * 4)()
    n = codes.size
    s, sample, eq = np.zeros(n, bool), np.zeros(n, bool), np.zeros(n, bool)
    for a, b in bounds:
        for p in range(a, b):
            it.it_type(ptr, p, out)
            s[p], eq[p] = bool(out[2]), p + 1 < b and codes[p + 1] == codes[p]
            sample[p] = s[p] and p > a and codes[p - 1] > codes[p]
    slow = 0
    for w in range((n + 15) // 16):
        for a, e in ((0, n), (bounds[3][0], bounds[-4][1])):
            if 16 * w + 16 <= a:
                continue  # a tile begins at the record its collection begins in
            got = it.it_samples(ptr, w, a, e)
            want = sum(int(sample[p]) << (p - 16 * w) for p in range(16 * w, min(16 * w + 16, n)) if a <= p < e)
            assert got & 0xFFFF == want, (w, a, e)
        got = it.it_samples(ptr, w, 0, n)
        slow += got >> 16
        if not got >> 16:
            it.it_masks(ptr, w, out)
            for p in range(16 * w, min(16 * w + 16, n)):
                assert (out[0] >> (p - 16 * w)) & 1 == s[p] and (out[1] >> (p - 16 * w)) & 1 == eq[p]
    assert slow > 0 or len(alphabet) > 1  # long runs of one base take the slow way


@needs_hipcc
def test_no_shift_amount_in_the_last_register(tmp_path):
    # with the amount of a 64-bit shift in the last vector register of the
    # allocation (granules of 8), the shift has given wrong results on gfx950
    asm = tmp_path / "cxbwt.s"
    flags = [f for f in pkg_build.HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    r = subprocess.run([HIPCC, *flags, "--cuda-device-only", "-S", "-I", os.path.join(ROOT, "include"),
                        os.path.join(CSRC, "cxbwt.hip"), "-o", str(asm)], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-2000:]
    seen = 0
    for m in re.finditer(r"\n(_Z\w+):[^\n]*\n(.*?)\.end_amdhsa_kernel", asm.read_text(), re.S):
        last = int(re.search(r"\.amdhsa_next_free_vgpr (\d+)", m.group(2)).group(1)) - 1
        amounts = {int(v) for v in re.findall(r"\bv_(?:lshlrev_b64|lshrrev_b64|ashrrev_i64)\S*\s+v\[\d+:\d+\],\s*v(\d+),",
                                              m.group(2))}
        seen += 1
        assert not (last % 8 == 7 and last in amounts), f"{m.group(1)}: v{last}"
    assert seen > 30
