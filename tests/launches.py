"""Which kernels calls of the library launch, without a GPU: the library runs in a process of its own under a stand-in for the
runtime's entry points that notes every launch and grant of LDS and launches nothing.

    traced([("conv1d", F32, B, Cin, L, Cout, Kw, stride, pad, dilation), ("reduce_max", F32, outer, red, inner)])

gives, per call, a list of Launch and Grant; the operands' addresses are made up (aligned, or one element off with
`x_off`), the workspace is as large as any call wants unless `workspace` says otherwise."""
import ctypes
import json
import os
import subprocess
import sys
import tempfile
from collections import namedtuple

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
Launch = namedtuple("Launch", "kernel grid block lds")           # kernel: demangled, without its parameters
Grant = namedtuple("Grant", "kernel bytes")

STAND_IN = r"""
#include <stddef.h>
#include <stdio.h>
typedef struct { unsigned x, y, z; } dim3;
static int handle;
static struct { dim3 grid, block; size_t lds; void* stream; } at;
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipGetLastError(void) { return 0; }
int hipGetSymbolAddress(void** p, const void* symbol) { *p = (void*)0x7000000; return 0; }
void** __hipRegisterFatBinary(const void* data) { static void* p = &handle; return &p; }
void __hipUnregisterFatBinary(void** modules) {}
void __hipRegisterVar(void** modules, void* var, char* host, char* device, int ext, size_t size, int constant, int global) {}
void __hipRegisterFunction(void** modules, const void* host, char* device, const char* name, unsigned limit, void* tid, void* bid,
                           dim3* block, dim3* grid, int* size)
{
    printf("kernel %p %s\n", host, name);
    fflush(stdout);
}
int __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, void* stream)
{
    at.grid = grid; at.block = block; at.lds = lds; at.stream = stream;
    return 0;
}
int __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, void** stream)
{
    *grid = at.grid; *block = at.block; *lds = at.lds; *stream = at.stream;
    return 0;
}
int hipFuncSetAttribute(const void* f, int attribute, int value) { printf("grant %p %d\n", f, value); fflush(stdout); return 0; }
int hipLaunchKernel(const void* f, dim3 grid, dim3 block, void** args, size_t lds, void* stream)
{
    printf("launch %p %u %u %zu\n", f, grid.x, block.x, lds);
    fflush(stdout);
    return 0;
}
"""


def _run():
    """The child: calls from stdin."""
    lib = ctypes.CDLL(sys.argv[1])
    i64, vp, ci, size = ctypes.c_int64, ctypes.c_void_p, ctypes.c_int, ctypes.c_size_t
    lib.pgk_conv1d.argtypes = [vp] * 4 + [i64] * 8 + [ci] * 2 + [vp, size, vp]
    lib.pgk_reduce_max.argtypes = [vp] * 3 + [i64] * 3 + [ci, vp, size, vp]
    for k, (op, dtype, *sizes, room, off) in enumerate(json.load(sys.stdin)):
        print("call", k, flush=True)
        x, rest = (1 << 40) + off * (2 if dtype else 4), [1 << 41, 1 << 42, 1 << 43]
        ws = (1 << 44, 1 << 42 if room is None else room) if room != 0 else (None, 0)
        if op == "conv1d":
            rc = lib.pgk_conv1d(x, rest[0], None, rest[1], *sizes, 0, dtype, *ws, None)
        else:
            rc = lib.pgk_reduce_max(x, rest[0], rest[1], *sizes, dtype, *ws, None)
        print("status", rc, flush=True)


def traced(calls, workspace=None, x_off=0):
    """Launches and grants of each call, in order; a call that is refused gives its status instead of the list.  workspace: bytes, of all
    calls or of each."""
    room = workspace if isinstance(workspace, list) else [workspace] * len(calls)
    from paper_2511_06345_amd import binding, build
    with tempfile.TemporaryDirectory() as folder:
        source, lib = os.path.join(folder, "hip.c"), os.path.join(folder, "hip.so")
        with open(source, "w") as f:
            f.write(STAND_IN)
        subprocess.run(["gcc", "-shared", "-fPIC", "-o", lib, source], check=True)
        env = dict(os.environ, LD_PRELOAD=" ".join(filter(None, [lib, os.environ.get("LD_PRELOAD")])))
        run = subprocess.run([sys.executable, os.path.abspath(__file__), binding.LIB_PATH], capture_output=True, text=True, cwd=ROOT, env=env,
                             input=json.dumps([[*map(lambda v: v if isinstance(v, str) else int(v), call), r, x_off] for call, r in zip(calls, room)]))
    assert run.returncode == 0, run.stderr
    names, out = {}, []
    for line in run.stdout.splitlines():
        what, *rest = line.split()
        if what == "kernel":
            names[rest[0]] = rest[1]
        elif what == "call":
            out.append([])
        elif what == "grant":
            out[-1].append(Grant(names[rest[0]], int(rest[1])))
        elif what == "launch":
            out[-1].append(Launch(names[rest[0]], *map(int, rest[1:])))
        elif what == "status" and rest[0] != "0":
            out[-1] = int(rest[0])
    mangled = sorted({step.kernel for call in out if isinstance(call, list) for step in call})
    plain = {m: p.replace("(anonymous namespace)::", "").replace("void ", "").replace("pgk::", "").split("(")[0] for m, p in zip(mangled, build._demangle(mangled))}
    return [call if isinstance(call, int) else [step._replace(kernel=plain[step.kernel]) for step in call] for call in out]


if __name__ == "__main__":
    _run()
