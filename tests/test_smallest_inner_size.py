"""CPU test of the host side at inner sizes below one 16-byte vector: a problem
is valid from k = 1 on (only an encode or a product needs whole vectors), so
every entry point that sizes or checks a workspace has to answer.  A crash would
take the interpreter with it, so the calls run in a child process."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CODE = """
import ctypes as C
from paper_0806_3121_amd import abft
L = abft.lib()
one = C.c_void_p(256)          # never read: every call below is refused before a launch
for dt, ks in ((abft.ABFT_F64, (1,)), (abft.ABFT_F32, (1, 3)), (abft.ABFT_BF16, (1, 4, 7)),
               (abft.ABFT_FP8_E4M3, (1, 7, 8, 15))):
    for k in ks:
        for m, n, br, bc in ((1, 1, 1, 1), (32, 32, 1, 1), (64, 64, 1, 1), (6400, 34, 2, 1), (34, 6400, 1, 32),
                             (4096, 4096, 1024, 1024)):
            p = abft.problem(dt, m, n, k, br, bc)
            size = abft.workspace_size(p)
            assert size > 0, (dt, m, n, k)
            # a workspace one byte short
            host = C.create_string_buffer(C.sizeof(abft.abft_report))
            for f in (L.abft_verify, L.abft_verify_noalloc):
                st = f(C.byref(p), one, None, 0, one, size - 1, C.cast(host, C.c_void_p), None)
                assert st == abft.ABFT_E_WORKSPACE, (dt, m, n, k, st)
            assert L.abft_verify_fused(C.byref(p), one, one, size - 1, None, None) == abft.ABFT_E_WORKSPACE
            # an encode or a product needs whole vectors
            assert L.abft_encode(C.byref(p), one, one, one, size, None) == abft.ABFT_E_ARG
            assert L.abft_gemm(C.byref(p), one, one, one, one, size, 0, None) == abft.ABFT_E_ARG
print("answered")
"""


def test_every_sizing_entry_answers():
    r = subprocess.run([sys.executable, "-c", CODE], capture_output=True, text=True, cwd=ROOT, timeout=300)
    assert r.returncode == 0 and "answered" in r.stdout, (r.returncode, r.stderr[-2000:])
