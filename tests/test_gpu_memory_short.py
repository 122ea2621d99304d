"""What the library does when device memory ends: it gives the 12-bit weight copies back where that helps, and only there.

Each test is a process of its own, in which tests/memory_budget_shim.cpp stands in front of the runtime's allocation calls and
makes device memory end at a budget."""
import ctypes as C
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
MB = 1 << 20


# ------------------------------------------------------------------------------------------------ in the child
class Child:
    def __init__(self, shim):
        self.shim = C.CDLL(shim, mode=C.RTLD_GLOBAL)   # before the library: its calls resolve to these
        self.shim.shim_live.restype = C.c_size_t
        self.shim.shim_budget.argtypes = [C.c_size_t]
        sys.path.insert(0, ROOT)
        import numpy as np
        from paper_2305_13144_amd import binding, synth
        self.np, self.ss, self.synth = np, binding, synth
        self.shape = synth.ModelShape("short", 2, 1024, 16, 64, 2752, 8000)
        self.tensors = synth.make_weights(self.shape, seed=6, threads=8)

    def weights(self):
        return self.ss.Weights(self.shape, self.tensors)

    def live(self):
        return self.shim.shim_live()

    def budget(self, over_live):
        self.shim.shim_budget(0 if over_live is None else self.live() + over_live)

    def copies(self, w):
        """Bytes that the handle's copies hold (they are made again afterwards)."""
        self.budget(None)
        before = self.live()
        w.set_option(self.ss.SS_OPT_WEIGHT_COPIES, 0)
        held = before - self.live()
        w.set_option(self.ss.SS_OPT_WEIGHT_COPIES, 1)
        return held

    def given_back(self, w):
        self.budget(None)
        before = self.live()
        w.set_option(self.ss.SS_OPT_WEIGHT_COPIES, 0)
        return self.live() == before

    def request(self, rows, plen, seed=1):
        rng = self.np.random.default_rng(seed)
        toks = rng.integers(0, self.shape.vocab, rows * plen).astype(self.np.int32)
        return toks, (self.np.arange(rows + 1) * plen).astype(self.np.int32)

    def microbatch(self, w, rows, plen, new=4):
        toks, offs = self.request(rows, plen)
        return self.ss.ss_decode_microbatch(w, toks, offs, new, self.np.full(rows, new, self.np.int32))["tokens"]

    def out_of_memory(self, call):
        try:
            call()
        except self.ss.SsError as e:
            assert e.code == self.ss.SS_ENOMEM, e
            return
        raise AssertionError("the call had memory enough")


def child_a_call_that_is_short_of_what_the_copies_hold(c):
    w = c.weights()
    held = c.copies(w)
    assert held > 30 * MB, held
    w.set_option(c.ss.SS_OPT_WEIGHT_COPIES, 0)
    before = c.live()
    want = c.microbatch(w, 16, 40)
    need = c.live() - before
    w.close()
    w = c.weights()
    assert c.copies(w) == held
    c.budget(need - held // 2)
    got = c.microbatch(w, 16, 40)
    assert c.given_back(w)
    assert c.np.array_equal(got, want)       # run again from the start, with the halves
    w.set_option(c.ss.SS_OPT_WEIGHT_COPIES, 1)
    assert c.copies(w) == held               # made again on request


def child_a_call_that_the_copies_cannot_help_leaves_them(c):
    w = c.weights()
    held = c.copies(w)
    want = c.microbatch(w, 1, 4)
    c.budget(MB)
    c.out_of_memory(lambda: c.microbatch(w, 64, 1000))   # its first buffer alone is larger than they are
    assert c.copies(w) == held
    c.budget(MB)
    c.out_of_memory(lambda: c.microbatch(w, 24, 160))    # each of its buffers would fit in their place, all of them not
    assert c.copies(w) == held
    assert c.np.array_equal(c.microbatch(w, 1, 4), want)


def child_host_memory_is_not_device_memory(c):
    w = c.weights()
    toks, offs = c.request(2, 5)
    held = c.copies(w)
    c.shim.shim_host_fails(1)
    c.out_of_memory(lambda: c.ss.ss_forward_logits(w, toks, offs, c.np.full(2, 5, c.np.int32)))
    c.shim.shim_host_fails(0)
    before = c.live()
    w.set_option(c.ss.SS_OPT_WEIGHT_COPIES, 0)
    assert before - c.live() == held, "the copies went for memory that they are not made of"


def child_lanes(c):
    """Group passes and the in-flight measurement, whose allocations fail on a lane's thread."""
    rng = c.np.random.default_rng(2)
    n, L, plen = 64, 8, 10
    toks, offs = c.request(n, plen, seed=3)
    targets = rng.integers(1, L + 1, n).astype(c.np.int32)
    pol = c.ss.make_policy((), 16, L, 16)
    run = lambda w: c.ss.ss_run_group(w, toks, offs, targets, None, 0, pol)
    pt = rng.integers(0, c.shape.vocab, 16 * plen).astype(c.np.int32)
    w = c.weights()
    held = c.copies(w)
    w.set_option(c.ss.SS_OPT_WEIGHT_COPIES, 0)
    before = c.live()
    c.microbatch(w, 16, plen, L)
    lane = c.live() - before                     # what one lane takes
    want = run(w)["tokens"]
    w.close()
    w = c.weights()
    before = c.live()
    c.ss.ss_bench_decode_step(w, pt, 16, plen, 1)
    bench_lane = c.live() - before
    w.close()
    for what in ("group", "bench"):
        w = c.weights()
        assert c.copies(w) == held
        c.budget(4 * (lane if what == "group" else bench_lane) - held // 2)
        if what == "group":
            assert c.np.array_equal(run(w)["tokens"], want)
        else:
            assert (c.ss.ss_bench_decode_steps_in_flight(w, pt, 16, plen, 3, 4) > 0).all()
        assert c.given_back(w), what
        w.close()
        c.budget(None)


def child_shared_forwards(c):
    """A group whose micro-batches share their decode forwards, with memory for one micro-batch a lane but not for the joint ones
    beside others: it runs without sharing, and gives the same tokens."""
    shape = c.synth.ModelShape("share", 2, 2048, 32, 64, 5504, 8000)
    tensors = c.synth.make_weights(shape, seed=7, threads=8)
    rng = c.np.random.default_rng(4)
    plen, small, large = 10, 256, 128
    targets = c.np.repeat([small, large], [4 * 16, 12 * 32]).astype(c.np.int32)   # four micro-batches of 16, twelve of 32
    toks = rng.integers(0, shape.vocab, len(targets) * plen).astype(c.np.int32)
    offs = (c.np.arange(len(targets) + 1) * plen).astype(c.np.int32)
    pol = c.ss.make_policy(("SORT", "BIN", "FCR", "VBS"), 16, small, 32)

    def handle():
        w = c.ss.Weights(shape, tensors)
        w.set_option(c.ss.SS_OPT_WEIGHT_COPIES, 0)
        return w

    run = lambda w: c.ss.ss_run_group(w, toks, offs, targets, targets, 8, pol)
    w = handle()
    before = c.live()
    r = run(w)
    together, want = c.live() - before, r["tokens"]
    assert r["stats"]["n_mb_first"] == 16
    w.close()
    w = handle()
    before = c.live()
    for rows, new in ((16, small), (32, large)):
        c.ss.ss_decode_microbatch(w, toks[:rows * plen], offs[:rows + 1], new, c.np.full(rows, 2, c.np.int32))
    lane = c.live() - before                     # what one lane takes
    w.close()
    assert 4 * lane + 8 * MB < together, (lane, together)
    w = handle()
    c.budget(4 * lane + 8 * MB)
    assert c.np.array_equal(run(w)["tokens"], want)
    w.close()
    w = handle()
    c.budget(2 * lane)
    c.out_of_memory(lambda: run(w))
    c.budget(None)
    assert c.np.array_equal(run(w)["tokens"], want)
    w.close()


def child_other_handles(c):
    """A new handle, and a call on another one, take the copies of the handles that are there."""
    a = c.weights()
    held = c.copies(a)
    before = c.live()
    b = c.weights()
    whole = c.live() - before                    # a handle with copies
    want = c.microbatch(b, 16, 40)
    need = c.live() - before - whole             # what the call takes
    b.close()
    c.budget(whole - held // 2)                  # room for a handle without copies, not for the rule that grants them
    b = c.weights()
    assert c.copies(a) == held                   # there was room: nothing was taken
    b.close()
    c.budget(whole - held - held // 2)           # half of what the first one's copies hold is missing
    b = c.weights()
    assert c.given_back(a)
    a.set_option(c.ss.SS_OPT_WEIGHT_COPIES, 1)
    assert c.copies(a) == held
    c.microbatch(a, 4, 5)
    b.set_option(c.ss.SS_OPT_WEIGHT_COPIES, 0)
    halves = c.microbatch(a, 4, 5)
    c.budget(need - held // 2)
    got = c.microbatch(b, 16, 40)                # b has none of its own
    assert c.given_back(a)
    a.set_option(c.ss.SS_OPT_WEIGHT_COPIES, 1)
    assert (got == want).mean() > 0.9            # other rounding, the same model
    assert c.np.array_equal(c.microbatch(a, 4, 5), halves)
    # far too much for both: nobody loses anything
    c.budget(MB)
    c.out_of_memory(lambda: c.microbatch(b, 64, 1000))
    assert c.copies(a) == held
    b.close()
    # a handle that cannot be had: the first one keeps its copies
    c.budget(whole - 3 * held)
    c.out_of_memory(c.weights)
    assert c.copies(a) == held


def child_a_busy_handle_gives_back_when_its_call_ends(c):
    import threading
    a, b = c.weights(), c.weights()
    held = c.copies(a)
    b.set_option(c.ss.SS_OPT_WEIGHT_COPIES, 0)
    before = c.live()
    want = c.microbatch(b, 16, 40)
    need = c.live() - before
    b.close()
    b = c.weights()
    b.set_option(c.ss.SS_OPT_WEIGHT_COPIES, 0)
    toks, offs = c.request(8, 20, seed=5)
    long_call = lambda: c.ss.ss_decode_microbatch(a, toks, offs, 400, c.np.full(8, 400, c.np.int32))["tokens"]
    ref = long_call()
    out, started = [], threading.Event()

    def run():
        started.set()
        out.append(long_call())

    c.budget(need - held // 2)
    t = threading.Thread(target=run)
    t.start()
    started.wait()
    got = c.microbatch(b, 16, 40)                # waits for the long call where that is still running
    t.join()
    assert c.given_back(a)
    assert c.np.array_equal(got, want)
    assert (out[0] == ref).mean() > 0.9 and out[0].shape == ref.shape


# ------------------------------------------------------------------------------------------------ in pytest
@pytest.fixture(scope="module")
def shim(tmp_path_factory):
    so = tmp_path_factory.mktemp("shim") / "memory_budget_shim.so"
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", os.path.join(ROOT, "tests", "memory_budget_shim.cpp"), "-ldl",
                    "-o", str(so)], check=True, capture_output=True, text=True)
    return str(so)


@pytest.mark.gpu
@pytest.mark.parametrize("what", sorted(n for n in globals() if n.startswith("child_")))
def test_memory(what, shim):
    r = subprocess.run([sys.executable, os.path.abspath(__file__), what, shim], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-4000:]


if __name__ == "__main__":
    globals()[sys.argv[1]](Child(sys.argv[2]))
    print("ok", flush=True)
