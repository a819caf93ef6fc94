"""Factorizations beside other work on the GPU: two wide ones on two streams,
and one during which another stream's kernel takes every CU of one die (XCD) for
longer than any launch of its own, so that the workgroups that build an inverse
Gram together start far apart.  All results as those of the same call alone.
"""
import ctypes
import os
import threading
import time

import numpy as np
import pytest

from paper_2607_13511_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

HOLD = b"""
extern "C" __global__ void hold(unsigned long long ticks) {  // of the 100 MHz wall clock
  extern __shared__ char whole[];
  if (ticks == 0) whole[threadIdx.x] = 0;
  if (blockIdx.x % 8 != 5) return;  // workgroups go to the 8 dies in turn
  const unsigned long long t0 = wall_clock64();
  while (wall_clock64() - t0 < ticks) __builtin_amdgcn_s_sleep(64);
}
"""
LDS_BYTES = 160 * 1024


def hold_code():
    """The hold kernel's code object, compiled for gfx950."""
    rtc = ctypes.CDLL(os.path.join(os.path.dirname(torch.__file__), "lib", "libhiprtc.so"))
    prog = ctypes.c_void_p()
    assert rtc.hiprtcCreateProgram(ctypes.byref(prog), HOLD, b"hold.hip", 0, None, None) == 0
    opts = (ctypes.c_char_p * 1)(b"--offload-arch=gfx950")
    assert rtc.hiprtcCompileProgram(prog, 1, opts) == 0
    size = ctypes.c_size_t()
    assert rtc.hiprtcGetCodeSize(prog, ctypes.byref(size)) == 0
    code = ctypes.create_string_buffer(size.value)
    assert rtc.hiprtcGetCode(prog, code) == 0
    return code


def hold_kernel():
    """hold(stream, ms): every CU (its whole LDS) of one die for ms milliseconds."""
    hip = ctypes.CDLL(os.path.join(os.path.dirname(torch.__file__), "lib", "libamdhip64.so"))
    code, module, fn = hold_code(), ctypes.c_void_p(), ctypes.c_void_p()
    assert hip.hipModuleLoadData(ctypes.byref(module), code) == 0
    assert hip.hipModuleGetFunction(ctypes.byref(fn), module, b"hold") == 0
    cus = torch.cuda.get_device_properties(0).multi_processor_count

    def hold(stream, ms):
        ticks = ctypes.c_ulonglong(int(ms * 1e5))
        args = (ctypes.c_void_p * 1)(ctypes.cast(ctypes.pointer(ticks), ctypes.c_void_p))
        assert hip.hipModuleLaunchKernel(fn, cus, 1, 1, 64, 1, 1, LDS_BYTES, ctypes.c_void_p(stream.cuda_stream),
                                         args, None) == 0
    return hold


def same(a, b):
    assert torch.equal(a.B_packed, b.B_packed) and torch.equal(a.C_packed, b.C_packed)
    assert torch.equal(a.D, b.D) and np.array_equal(a.curve, b.curve)


@pytest.mark.parametrize("block", [64, 128])
def test_beside_a_kernel_that_holds_a_die(block):
    from paper_2607_13511_amd import binding
    A = torch.from_numpy(synth.small("t4_rowscale", 1100, 1040, 3)).cuda()
    run = lambda s=None: binding.factorize(A, 1.0, 1.0, block, 8, stream=s)
    run()
    t0 = time.perf_counter()
    alone = run()
    took = time.perf_counter() - t0
    hold = hold_kernel()
    streams = [torch.cuda.Stream() for _ in range(4)]
    torch.cuda.synchronize()
    for i in range(12):
        # another stream's kernel starts somewhere in the middle
        other, mine = streams[i % 4], streams[(i + 1) % 4]
        t = threading.Timer(took * (0.1 + 0.05 * i), hold, (other, 30.0))
        t0 = time.perf_counter()
        t.start()
        beside = run(mine)
        print(f"[streams] block {block}: {1e3 * took:.1f} ms alone, "
              f"{1e3 * (time.perf_counter() - t0):.1f} ms beside", flush=True)
        t.join()
        torch.cuda.synchronize()
        same(alone, beside)


def test_two_wide_factorizations_on_two_streams():
    from paper_2607_13511_amd import binding
    As = [torch.from_numpy(synth.small("t4_rowscale", 2100, 2060, s)).cuda() for s in (1, 2)]
    alone = [binding.factorize(A, 0.5, 1.0, 256, 8) for A in As]
    streams = [torch.cuda.Stream() for _ in As]
    torch.cuda.synchronize()
    got = [None, None]

    def run(i):
        for _ in range(3):
            got[i] = binding.factorize(As[i], 0.5, 1.0, 256, 8, stream=streams[i])

    threads = [threading.Thread(target=run, args=(i,)) for i in range(2)]
    print("[streams] two wide factorizations", flush=True)
    for t in threads:
        t.start()
    for t in threads:
        t.join(60)
    torch.cuda.synchronize()
    for a, b in zip(alone, got):
        same(a, b)
