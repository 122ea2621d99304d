"""ss_bench_weight_stream launches the matrix kernels of a decode forward: the same ones in the same order on the same grids.

A process of its own, in which tests/launch_names_shim.cpp stands in front of the runtime's launch call and notes them."""
import ctypes as C
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def child(shim_path):
    shim = C.CDLL(shim_path, mode=C.RTLD_GLOBAL)   # before the library: its calls resolve to it
    shim.shim_launches.restype = C.c_size_t
    shim.shim_launches.argtypes = [C.c_char_p, C.c_size_t]
    sys.path.insert(0, ROOT)
    import numpy as np
    from paper_2305_13144_amd import binding as ss, synth

    def matrix_kernels():
        buf = C.create_string_buffer(1 << 20)
        n = shim.shim_launches(buf, len(buf))
        assert n <= len(buf)
        return [line for line in buf.raw[:n].decode().splitlines() if "k_gemm" in line]

    shape = synth.ModelShape("stream", 2, 1024, 8, 128, 2048, 4096)
    W = synth.make_weights(shape, seed=3, threads=8)
    other = list(W)
    other[3] = W[3].copy()
    other[3][5, 5] = synth.f32_to_bf16_bits(np.array([0.5], np.float32))[0]   # q|k|v of the first layer has no copy
    per = 4 * shape.n_layers + 1
    for tensors in (W, other):
        gw = ss.Weights(shape, tensors)
        for rows in (1, 2, 3, 4, 5, 16, 17, 64, 96, 200, 300):
            print("rows", rows, flush=True)
            toks = np.arange(rows * 8, dtype=np.int32) % shape.vocab
            ss.ss_bench_decode_step(gw, toks, rows, 8, 1)
            decode = matrix_kernels()[-per:]
            ms, launches = ss.ss_bench_weight_stream(gw, rows, 2)
            stream = matrix_kernels()
            assert launches == per and (ms > 0).all()
            assert stream == decode * 2, (rows, stream[:per], decode)
        gw.close()


@pytest.mark.gpu
def test_its_launches_are_those_of_a_decode_forward(tmp_path):
    so = tmp_path / "launch_names_shim.so"
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", os.path.join(ROOT, "tests", "launch_names_shim.cpp"), "-ldl", "-o", str(so)],
                   check=True, capture_output=True, text=True)
    r = subprocess.run([sys.executable, os.path.abspath(__file__), str(so)], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-4000:]


if __name__ == "__main__":
    child(sys.argv[1])
