"""Host code of the attention launch (attend_split.hpp), compiled for the CPU: no GPU needed."""
import ctypes
import os
import random
import subprocess
import sys

import pytest

from paper_2602_10825_amd import build

DRIVER = r"""
#include "attend_split.hpp"
extern "C" {
__attribute__((visibility("default"))) int listed_chunk(const int32_t* rec, int n, int A, int i) {
    return fc_listed_chunk(rec, n, A, i);
}
__attribute__((visibility("default"))) int room(const void* ws, size_t bytes, int parts, int d) {
    return fc_room_for_partials(ws, bytes, parts, d);
}
// partials that the plans ask for, the most over key counts from 0 to 2^17
__attribute__((visibility("default"))) int parts(int A, int L_c, int H_q, int d) {
    int most = 0;
    for (int clean = 0; clean < 1 << 17; clean += 1 + clean / 7) {
        const int b = fc_attend_plan_bf16(A, L_c, clean, H_q, d, true).parts, f = fc_attend_plan_f32(A, L_c, clean, H_q, true).parts;
        most = most > b ? most : b;
        most = most > f ? most : f;
    }
    return most;
}
// what a bf16 launch of R chunks runs: 32-row blocks (0), 256-row units whole (1), all split (2), the last round split (3)
__attribute__((visibility("default"))) int form(int A, int L_c, int L_clean, int H_q, int d, int R) {
    const FcAttendPlan p = fc_attend_plan_bf16(A, L_c, L_clean, H_q, d, true);
    if (p.narrow[R - 1]) return 0;
    const int S = p.splits[R - 1];
    return S == 1 ? 1 : fc_wide_shape(R, H_q * ((L_c + kWideRows - 1) / kWideRows), S).full == 0 ? 2 : 3;
}
__attribute__((visibility("default"))) int bound(int A, int L_c, int H_q) { return (int)fc_split_parts_bound(A, L_c, H_q); }
}
"""


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    src, so = d / "plan.hip", d / "plan.so"
    src.write_text(DRIVER)
    subprocess.run([build.HIPCC, "--offload-host-only", *build.FLAGS, "-shared", str(src), "-o", str(so)], check=True)
    return str(so)


def read_lists(so):
    """Every list ends at the last byte before a page that must not be touched."""
    libc = ctypes.CDLL(None, use_errno=True)
    libc.mmap.restype = ctypes.c_void_p
    libc.mmap.argtypes = [ctypes.c_void_p, ctypes.c_size_t, ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.c_long]
    libc.mprotect.argtypes = [ctypes.c_void_p, ctypes.c_size_t, ctypes.c_int]
    page = os.sysconf("SC_PAGE_SIZE")
    base = libc.mmap(None, 2 * page, 3, 0x22, -1, 0)             # read | write, private | anonymous
    assert base and base != ctypes.c_void_p(-1).value
    assert libc.mprotect(base + page, page, 0) == 0
    f = ctypes.CDLL(so).listed_chunk
    f.argtypes = [ctypes.c_void_p, ctypes.c_int, ctypes.c_int, ctypes.c_int]
    for A in (1, 3, 16):
        for entries in ([], [0], [A - 1], [0, A, -1][:A], list(range(A))):
            at = base + page - 4 * len(entries)
            (ctypes.c_int32 * len(entries)).from_address(at)[:] = entries
            got = [f(at, len(entries), A, lane) for lane in range(64)]
            assert got == [c if 0 <= c < A else -1 for c in entries] + [-1] * (64 - len(entries))
    assert [f(base, -3, 4, lane) for lane in range(64)] == [-1] * 64
    full = (ctypes.c_int32 * 16)(*range(16))                     # a count above A is cut to A
    assert [f(ctypes.addressof(full), 99, 16, lane) for lane in range(64)] == list(range(16)) + [-1] * 48


def test_recompute_list_is_not_read_past_its_count(driver):
    """A list of exactly *n_rec entries: 64 lanes look at it, none touches what lies behind."""
    r = subprocess.run([sys.executable, "-c", "import sys; sys.path.insert(0, %r); "
                        "from tests.test_attend_plan import read_lists; read_lists(%r)" % (build.ROOT, driver)])
    assert r.returncode == 0


def test_room_for_partials(driver):
    f = ctypes.CDLL(driver).room
    f.argtypes = [ctypes.c_void_p, ctypes.c_size_t, ctypes.c_int, ctypes.c_int]
    need = 3 * 32 * 66 * 4
    assert f(None, 0, 0, 64) and f(0x1000, need, 3, 64)
    assert not f(None, need, 3, 64) and not f(0x1000, need - 1, 3, 64)
    assert not any(f(0x1000 + off, need, 3, 64) for off in range(1, 16)) and f(0x1010, need, 3, 64)


def test_workspace_holds_what_any_number_of_keys_can_ask_for(driver):
    so = ctypes.CDLL(driver)
    rng = random.Random(1)
    for _ in range(4000):
        A, H, d = rng.randint(1, 16), rng.choice((1, 2, 3, 8, 12, 24, 40, 64)), rng.choice((64, 128))
        L_c = int(2 ** rng.uniform(0, 14))
        assert so.parts(A, L_c, H, d) <= so.bound(A, L_c, H), (A, L_c, H, d)


@pytest.mark.parametrize("A,L_c,H,most", [(2, 10200, 12, 0),              # SkyReels-V2-1.3B-like layer: never split
                                          (4, 9360, 24, 8 * 8 * 15 * 2),  # MAGI-1-like: one chunk, the last round in two
                                          (3, 328, 8, 2048),
                                          (5, 2040, 24, 2048), (2, 1021, 12, 3840), (3, 5000, 12, 0), (4, 2500, 24, 0)])
def test_workspace_of_known_layers(driver, A, L_c, H, most):
    """No room for splits that no plan takes: 60 and 64 MB of them on the two layers."""
    assert ctypes.CDLL(driver).bound(A, L_c, H) == most
