"""What launches ask of the runtime beside the launch itself, seen through a stand-in for the runtime's entry points (no GPU): a
kernel's grant of LDS is one for all its calls, whichever thread makes them."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

STAND_IN = r"""
#include <stddef.h>
#include <stdio.h>
struct dim3 { unsigned x, y, z; };
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipGetLastError(void) { return 0; }
int hipFuncSetAttribute(const void* f, int attribute, int value) { printf("grant %p %d %d\n", f, attribute, value); return 0; }
static struct { struct dim3 grid, block; size_t lds; void* stream; } at;
int __hipPushCallConfiguration(struct dim3 grid, struct dim3 block, size_t lds, void* stream)
{
    at.grid = grid; at.block = block; at.lds = lds; at.stream = stream;
    return 0;
}
int __hipPopCallConfiguration(struct dim3* grid, struct dim3* block, size_t* lds, void** stream)
{
    *grid = at.grid; *block = at.block; *lds = at.lds; *stream = at.stream;
    return 0;
}
int hipLaunchKernel(const void* f, struct dim3 grid, struct dim3 block, void** args, size_t lds, void* stream)
{
    printf("launch %p %zu\n", f, lds);
    return 0;
}
"""

CALLS = r"""
import ctypes, sys
lib = ctypes.CDLL(sys.argv[1])
i64, vp = ctypes.c_int64, ctypes.c_void_p
lib.pgk_conv1d.argtypes = [vp] * 4 + [i64] * 8 + [ctypes.c_int] * 2 + [vp, ctypes.c_size_t, vp]
for Kw in (7, 6, 7):
    rc = lib.pgk_conv1d(0x10000, 0x20000, None, 0x30000, 8, 384, 9000, 64, Kw, 1, 0, 1, 0, 1, 0x40000, 1 << 40, None)
    assert rc == 0, rc
"""


@pytest.fixture(scope="module")
def trace(tmp_path_factory):
    from paper_2511_06345_amd import binding
    if not os.path.exists(binding.LIB_PATH):
        pytest.skip("the library is not built")
    folder = tmp_path_factory.mktemp("stand_in")
    source, lib = folder / "hip.c", folder / "hip.so"
    source.write_text(STAND_IN)
    subprocess.run(["gcc", "-shared", "-fPIC", "-o", str(lib), str(source)], check=True)
    run = subprocess.run([sys.executable, "-c", CALLS, binding.LIB_PATH], capture_output=True, text=True, cwd=ROOT,
                         env=dict(os.environ, LD_PRELOAD=" ".join(filter(None, [str(lib), os.environ.get("LD_PRELOAD")]))))
    assert run.returncode == 0, run.stderr
    return [line.split() for line in run.stdout.splitlines()]


def test_a_call_does_not_lower_what_another_was_granted(trace):
    launches = [(line[1], int(line[2])) for line in trace if line[0] == "launch" and int(line[2]) > 65536]
    assert len(launches) == 3 and len({kernel for kernel, _ in launches}) == 1, trace
    assert launches[0][1] > launches[1][1], "the calls are meant to differ in what they take"
    granted = [int(line[3]) for line in trace if line[0] == "grant" and line[1] == launches[0][0]]
    assert granted and len(set(granted)) == 1 and granted[0] >= launches[0][1], granted
    # before the kernel's first launch, and not again
    assert len(granted) == 1 and trace.index(["launch", launches[0][0], str(launches[0][1])]) > [line[0] for line in trace].index("grant")
