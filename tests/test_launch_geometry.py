"""Launch geometry of the largest calls, on the CPU: the runtime refuses 2^32 threads or more in a dimension of a grid, after the call's earlier hops are on their
way.  A program of its own puts a recorder in the place of the runtime's launch function (made-up addresses, nothing runs) and makes the calls."""
import json
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CC = shutil.which("cc") or shutil.which("gcc")
RECORDER = """
#include <stddef.h>
typedef struct { unsigned x, y, z; } dim;
unsigned long long launches[64][6]; int launch_count;
int hipLaunchKernel(const void* f, dim g, dim b, void** a, size_t s, void* q) {
    const unsigned long long r[6] = {g.x, g.y, g.z, b.x, b.y, b.z};
    for (int i = 0; i < 6 && launch_count < 64; ++i) launches[launch_count][i] = r[i];
    ++launch_count;
    return 0;
}
static dim grid, block; static size_t lds; static void* stream;
int __hipPushCallConfiguration(dim g, dim b, size_t s, void* q) { grid = g; block = b; lds = s; stream = q; return 0; }
int __hipPopCallConfiguration(dim* g, dim* b, size_t* s, void** q) { *g = grid; *b = block; *s = lds; *q = stream; return 0; }
int hipGetLastError(void) { return 0; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipFuncSetAttribute(const void* f, int a, int v) { return 0; }
"""
PROGRAM = """
import ctypes as C, json, sys
recorder = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)     # ahead of the runtime in the order of symbols
sys.path.insert(0, sys.argv[2])
import paper_2410_20926_amd as ta
lib, out = ta.load_library(), []
for dims, B, Hq, Hkv, D, axis, vin in json.loads(sys.argv[3]):
    plan, at = ta.ta_plan_create(B, Hq, Hkv, D, dims, ta.TA_BF16, True), [(i + 1) << 40 for i in range(7)]
    C.c_int.in_dll(recorder, "launch_count").value = 0
    st = [lib.ta_axis_attn_forward(plan.handle, axis, at[0], at[1], at[2], vin, at[3], None),
          lib.ta_axis_attn_backward(plan.handle, axis, at[0], at[1], at[2], vin, at[3], at[4], at[5], at[6], 0, None)]
    n = C.c_int.in_dll(recorder, "launch_count").value
    out.append((st, plan.hop_function(axis, vin, True), [list(r) for r in (C.c_ulonglong * 6 * 64).in_dll(recorder, "launches")[:n]]))
print(json.dumps(out))
"""
CASES = [
    # dims, B, Hq, Hkv, D, axis, value input
    ((33, 8_000_000), 9, 1, 1, 8, 0, 1),                   # 72,000,000 fibres of two narrow tiles; shares of four take 18,000,000 workgroups of 256 threads
    ((4_000_000, 64), 17, 1, 1, 8, 1, 0),
    ((2_500_000, 50), 14, 2, 2, 8, 1, 1),
    ((2_000_000, 100), 40, 1, 1, 8, 1, 0),                 # four tiles
    ((8_000_000, 32), 16, 1, 1, 8, 1, 1),
    ((1_500_000, 160), 10, 1, 1, 8, 1, 1),
]


@pytest.mark.skipif(CC is None, reason="no C compiler")
def test_no_grid_passes_what_the_runtime_takes(tmp_path):
    source, recorder = tmp_path / "recorder.c", tmp_path / "recorder.so"
    source.write_text(RECORDER)
    subprocess.run([CC, "-shared", "-fPIC", str(source), "-o", str(recorder)], check=True)
    res = subprocess.run([sys.executable, "-c", PROGRAM, str(recorder), ROOT, json.dumps(CASES)], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stderr
    results = json.loads(res.stdout.splitlines()[-1])
    assert [r[1] for r in results[:4]] == ["mfma_bwd_resident_kernel"] * 4
    for case, (status, _, launches) in zip(CASES, results):
        assert status == [0, 0] and len(launches) >= 2, (case, status)
        for g in launches:
            assert all(g[i] * g[3 + i] < 1 << 32 for i in range(3)) and max(g[1:3]) <= 65535, (case, g)
