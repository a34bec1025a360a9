"""Launch shapes of problems that are too large to run in a test: the library's launches are recorded instead of made, by functions
that take the place of the HIP runtime's in a process of their own.  No GPU."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

RECORDER = r"""
#include <stddef.h>
#include <stdint.h>
#include <stdio.h>
typedef struct { uint32_t x, y, z; } dim3_;
static dim3_ last_grid, last_block;
unsigned __hipPushCallConfiguration(dim3_ grid, dim3_ block, size_t shared, void *stream) {
    last_grid = grid;
    last_block = block;
    return 0;
}
int __hipPopCallConfiguration(dim3_ *grid, dim3_ *block, size_t *shared, void **stream) {
    *grid = last_grid;
    *block = last_block;
    *shared = 0;
    *stream = 0;
    return 0;
}
int hipLaunchKernel(const void *f, dim3_ grid, dim3_ block, void **args, size_t shared, void *stream) {
    printf("%u %u %u %u", grid.x, grid.y, grid.z, block.x);
    if (block.x == 256) {                             /* k_recall_logits(pv, Q, K, G, head, rows, L, ws, ..) */
        const int32_t *rows = args[5];
        printf(" %ld %ld %ld %d %d", *(long *)args[1], *(long *)args[2], *(long *)args[7], rows[1], rows[2]);
    }
    printf("\n");
    fflush(stdout);
    return 0;
}
int hipGetLastError(void) { return 0; }
"""

RECALL = """
import ctypes, sys
sys.modules["torch"] = None                           # not needed, and it would bring a runtime of its own
import numpy as np
ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)     # before the library and the runtime it is linked to
import paper_2510_24606_amd as dhsa
L = int(sys.argv[2])
B = np.array([0, L // 2, L], dtype=np.int32)
p = dhsa.dhsa_problem(L=L, H_q=1, H_kv=1, D=64, N_c=2, N_b=1000, dtype=dhsa.DHSA_F32)
rows = np.array([0, L - 1], dtype=np.int64)
at = 1 << 40                                          # an address that nothing reads
code = dhsa.lib().dhsa_recall_rows(p, at, at, B.ctypes.data, at, dhsa.dhsa_plan_bytes(p, B), 0,
                                   rows.ctypes.data_as(ctypes.POINTER(ctypes.c_int64)), 2, at, at, 16 * L, at, at, None)
assert code == 0, code
"""


def launches(code, tmp_path, *args):
    """(grid x, y, z, threads a block, ..) of every launch that the program makes."""
    source, stub = tmp_path / "recorder.c", tmp_path / "recorder.so"
    source.write_text(RECORDER)
    subprocess.run(["gcc", "-shared", "-fPIC", "-w", "-o", str(stub), str(source)], check=True)
    out = subprocess.run([sys.executable, "-c", code, str(stub), *map(str, args)], cwd=ROOT, check=True, timeout=300,
                         stdout=subprocess.PIPE, text=True).stdout
    return [tuple(map(int, line.split())) for line in out.splitlines()]


def test_recall_of_rows_beyond_2_to_the_30(tmp_path):
    """A grid has fewer than 2^32 threads along x; the logits' launches have every key of the last row (64 to a workgroup), and
    what a launch calls row or key j is row or key key0 + j, wherever it reads or writes."""
    at = 1 << 40
    for L in (100, 1 << 20, (1 << 29) + 1, (1 << 30) + 100):
        *logits, count = launches(RECALL, tmp_path, L)
        assert count[:2] == (2, 1)
        key0 = 0
        for x, y, z, threads, q, k, ws, *rows in logits:
            assert x * threads < 1 << 32 and (y, z) == (1, 1)
            assert (q, k, ws) == (at + 256 * key0, at + 256 * key0, at + 8 * key0) and rows == [0 - key0, L - 1 - key0]
            key0 += 64 * x
        assert key0 >= L > key0 - 64, logits
