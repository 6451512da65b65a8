"""The library's host paths against a stand-in for the HIP runtime (CPU only).

A small C library with the runtime calls that a path makes is preloaded in a
process of its own: it launches nothing, notes every call in order, hands out
the words that a read-back from the device would give and can let a wait fail.
"""
import os
import subprocess
import sys
import textwrap

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2502_01637_amd", "libscone.so")

STUB = r"""
#include <stddef.h>
#include <string.h>
typedef struct { unsigned x, y, z; } dim3;
char stub_log[65536];
static size_t used;
unsigned stub_words[16];      /* what a read-back gives, then zeros */
int stub_fail_sync, stub_syncs;
static void note(char c) { if (used + 1 < sizeof(stub_log)) stub_log[used++] = c; }
int hipMemsetAsync(void* p, int v, size_t n, void* s) { note('M'); return 0; }
int hipMemcpyAsync(void* d, const void* s, size_t n, int kind, void* st) {
    note(kind == 2 ? 'D' : 'U');
    if (kind == 2) {
        memset(d, 0, n);
        memcpy(d, stub_words, n < sizeof(stub_words) ? n : sizeof(stub_words));
    }
    return 0;
}
int hipStreamSynchronize(void* s) { note('S'); return ++stub_syncs == stub_fail_sync; }
int hipLaunchKernel(const void* f, dim3 g, dim3 b, void** a, size_t n, void* s) {
    note('K');
    return 0;
}
int __hipPushCallConfiguration(dim3 g, dim3 b, size_t n, void* s) { return 0; }
int __hipPopCallConfiguration(dim3* g, dim3* b, size_t* n, void** s) {
    dim3 one = {1, 1, 1};
    *g = *b = one;
    *n = 0;
    *s = 0;
    return 0;
}
int hipGetLastError(void) { return 0; }
int hipGetDevice(int* d) { *d = 0; return 0; }
"""

HEAD = textwrap.dedent("""
    import ctypes, struct, sys
    P, I64, I32, D = ctypes.c_void_p, ctypes.c_int64, ctypes.c_int32, ctypes.c_double
    stub = ctypes.CDLL(sys.argv[1])
    L = ctypes.CDLL(sys.argv[2])
    log = lambda: ctypes.c_char_p(ctypes.addressof(ctypes.c_char.in_dll(stub, "stub_log"))).value
    words = (ctypes.c_uint * 16).in_dll(stub, "stub_words")
    fail_sync = ctypes.c_int.in_dll(stub, "stub_fail_sync")
    A = 0x7f0000000000          # addresses that nothing touches
""")


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    d = tmp_path_factory.mktemp("stub")
    src, so = d / "stub.c", d / "stub.so"
    src.write_text(STUB)
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", str(src), "-o", str(so)], check=True)
    return str(so)


def run(stub, body):
    env = dict(os.environ)
    env["LD_PRELOAD"] = ":".join(p for p in (stub, os.environ.get("LD_PRELOAD", "")) if p)
    p = subprocess.run([sys.executable, "-c", HEAD + textwrap.dedent(body), stub, LIB], env=env,
                       capture_output=True, text=True, timeout=120)
    assert p.returncode == 0, p.stderr[-2000:]
    return p.stdout.split()


@pytest.mark.parametrize("max_len", [2, 3, 4, 7])
@pytest.mark.parametrize("n", [0, 1000])
def test_table_sizes_leave_nothing_queued(stub, max_len, n):
    """scone_fgram_table_bytes, and a build that is refused for a short
    memory, have nothing queued in the caller's memory when they return."""
    for call in ("L.scone_fgram_table_bytes(P(A), I64(n), I32(K), D(0.5), P(A + (1 << 20)), None,"
                 " ctypes.byref(b))",
                 "L.scone_build_fgram_table_in(P(A), P(A + (1 << 20)), P(A + (2 << 20)), I64(n),"
                 " I32(K), D(0.5), P(A + (3 << 20)), I64(300), None, ctypes.byref(h))"):
        out = run(stub, f"""
            n, K, b, h = {n}, {max_len}, I64(), P()
            print({call}, "log=" + log().decode())
        """)
        assert out[0] == ("0" if "bytes(" in call else "1")
        assert out[1] == "log=" or out[1].endswith("S"), out


@pytest.mark.parametrize("max_len,waits", [(3, 1), (5, 2)])
def test_lengths_are_counted_once(stub, max_len, waits):
    """The sizes and then the build, as the binding calls them: the host waits for
    the count of the longer lengths, where there can be any, and for the table."""
    slot = 16 if max_len <= 5 else 32
    out = run(stub, f"""
        b, h = I64(), P()
        a = lambda k: P(A + (k << 24))
        r0 = L.scone_fgram_table_bytes(a(0), I64(1000), I32({max_len}), D(0.25), a(1), None,
                                       ctypes.byref(b))
        rc = lambda nbytes: L.scone_build_fgram_table_sized(
            a(2), a(0), a(3), I64(1000), I32({max_len}), D(0.25), a(4), I64(nbytes), None,
            ctypes.byref(h))
        r1 = rc(b.value)
        print(r0, r1, b.value, log().decode().count("S"),
              *[rc(k) for k in (0, 256, b.value - 1, b.value + {slot}, b.value // 2 + 128)])
    """)
    assert out == ["0", "0", str(4096 * slot + 256), str(waits)] + ["1"] * 5


def test_discovery_tells_its_two_data_errors_apart(stub):
    """The status word's bits: a bad token, regions that disagree, and both."""
    for bits, want in [(1 << 8, "8"), (1 << 5, "5"), (1 << 8 | 1 << 5, "8")]:
        out = run(stub, f"""
            words[0], words[2], words[3] = {bits}, 5, 3
            found = I64(-1)
            a = lambda k: P(A + (k << 24))
            rc = L.scone_discover_fgrams(a(0), I64(10), I64(100), I32(3), I32(1), I64(20), a(1),
                                         a(2), a(3), ctypes.byref(found), a(4), I64(1 << 24),
                                         None)
            print(rc, found.value)
        """)
        assert out == [want, "0"], (bits, out)


def test_discovery_reports_a_failed_last_wait(stub):
    """The second selection (a cut above the histogram) is waited for at the
    end of the call; an error that this wait returns is the call's."""
    for fail, want in [(0, "0"), (2, "7")]:
        out = run(stub, f"""
            words[2], words[3] = 50, 4095               # candidates, the largest count
            words[8], words[9] = 4095, 1                # the cut is still to be found
            fail_sync.value = {fail}
            found = I64(-1)
            a = lambda k: P(A + (k << 24))
            rc = L.scone_discover_fgrams(a(0), I64(10), I64(100), I32(2), I32(1), I64(20), a(1),
                                         a(2), a(3), ctypes.byref(found), a(4), I64(1 << 24),
                                         None)
            print(rc, found.value, log().decode())
        """)
        assert out[0] == want and out[1] == ("20" if want == "0" else "0"), out
        assert out[2].endswith("DSUKS"), out


@pytest.mark.parametrize("n,layers,most", [(1, 0, 4), (8193, 0, 4), (1, 1, 11), (255, 1, 11),
                                           (8193, 1, 18), (20_000, 1, 40)])
def test_launches_of_small_precomputes(stub, n, layers, most):
    """K = 7: no tree without layers, one launch for the tree of a short list, and no
    radix passes (five launches for each of twelve) where counting ranks is faster."""
    out = run(stub, f"""
        a = lambda k: P(A + (k << 34))
        L.scone_fgram_model_workspace.restype = I64
        need = L.scone_fgram_model_workspace(I64({n}), 7, 512, 8, 128)
        rc = L.scone_fgram_model_forward_in(a(0), a(1), a(2), I64({n}), 7, a(3), I64(50257), a(4),
                                            512, 8, 128, {layers}, a(5), I64({n}), a(6), I64(need),
                                            None)
        print(rc, log().decode().count("K"))
    """)
    assert out[0] == "0" and int(out[1]) <= most, out
