"""The library's host code against a HIP runtime without a device
(stub_hip.cpp): what is launched, copied, waited for and kept, also after a
call of the runtime fails.  Each scenario runs in a process of its own, with
the stub loaded before the library.
"""
import ctypes as C
import os
import random
import subprocess
import sys
import types

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
USER = "0x77000"  # the caller's stream


class Host:
    """The library on the stub, with one context."""

    def __init__(self, stub):
        sys.path.insert(0, os.path.dirname(HERE))
        self.stub = C.CDLL(stub, mode=C.RTLD_GLOBAL)
        self.stub.stub_log.restype = C.c_char_p
        sys.modules["torch"] = types.ModuleType("torch")  # the binding only has it load the real runtime
        import paper_1103_4697_amd as snc
        self.snc, self.L = snc, snc.lib()
        self.ctx = C.c_void_p()
        assert self.L.snc_create(0, C.byref(self.ctx)) == 0
        self.stub.stub_loaded_bytes.restype = C.c_size_t
        self.loaded = self.stub.stub_loaded_bytes()
        self.stub.stub_clear()
        self.ws = C.c_void_p(0x10000000)  # never read on the host
        self.stream = C.c_void_p(int(USER, 16))

    def log(self):
        return self.stub.stub_log().decode().splitlines()

    def fail(self, name, nth):
        self.stub.stub_fail(name.encode(), nth)

    def pairs(self, ps):
        """Operand arrays, output array and plans of a batch."""
        snc, n, keep = self.snc, len(ps), []
        F = (snc.Bipoly * n)(*[snc._as_bipoly(f, keep) for f, g in ps])
        G = (snc.Bipoly * n)(*[snc._as_bipoly(g, keep) for f, g in ps])
        plans, total = (snc.Plan * n)(), snc.Plan()
        assert self.L.snc_resultant_y_batch_plan(n, F, G, plans, C.byref(total)) == 0
        outs = (snc.Upoly * n)(*[snc._out_upoly(p.deg_bound, p.out_nlimbs, keep)[0] for p in plans])
        self.keep = keep
        return F, G, outs, plans, total

    def batch(self, ps):
        F, G, outs, _, total = self.pairs(ps)
        return self.L.snc_resultant_y_batch(self.ctx, len(ps), F, G, self.ws, C.c_size_t(total.workspace_bytes),
                                            self.stream, outs)

    def prepare(self, ps):
        F, G, outs, _, total = self.pairs(ps)
        h = C.c_void_p()
        assert self.L.snc_resultant_y_prepare(self.ctx, len(ps), F, G, self.ws, C.c_size_t(total.workspace_bytes),
                                              self.stream, C.byref(h)) == 0
        return h, outs

    def prepare_run(self, ps):
        h, outs = self.prepare(ps)
        self.stub.stub_clear()
        assert self.L.snc_prepared_run(h, self.stream, outs) == 0


def dense(rnd, m, dx, bits):
    return [[rnd.randrange(1, 1 << bits) for _ in range(dx + 1)] for _ in range(m + 1)]


def two_class_batch():
    """More than 2^20 output words, of y-degree 1, and enough evaluation in another register class: two tails."""
    rnd = random.Random(3)
    return ([(dense(rnd, 1, 900, 1500), dense(rnd, 1, 900, 1500)) for _ in range(7)] +
            [(dense(rnd, 20, 20, 60), dense(rnd, 19, 20, 60)) for _ in range(9)])


# ---------------------------------------------------------------------------
# Scenarios: print the log of the calls under test
# ---------------------------------------------------------------------------
def failed_second_tail_single_call(H):
    H.fail("graph_launch", 2)
    assert H.batch(two_class_batch()) == H.snc.SNC_EDEVICE
    return H.log()


def failed_second_tail_handle(H):
    h, outs = H.prepare(two_class_batch())
    H.stub.stub_clear()
    H.fail("graph_launch", 2)
    assert H.L.snc_prepared_run(h, H.stream, outs) == H.snc.SNC_EDEVICE
    return H.log()


def failed_submit(H):
    h, outs = H.prepare(two_class_batch())
    need = H.L.snc_prepared_stage_bytes(h)
    H.stub.stub_clear()
    H.fail("event_record", 3)  # the slot's copy, the first chunk, the second
    t = C.c_int64()
    assert H.L.snc_prepared_submit(h, C.c_void_p(0x20000000), C.c_size_t(need), H.stream,
                                   C.byref(t)) == H.snc.SNC_EDEVICE
    return H.log()


def remaindering_kernels(H, ps):
    H.prepare_run(ps)
    return [line for line in H.log() if "k_crt" in line]


def few_small_beside_many_large(H):
    """Twenty thousand coefficients of 65..128 primes and ninety of four: the four-prime ones do not fill the chip."""
    rnd = random.Random(4)
    ps = [(dense(rnd, 1, 100, 1200), dense(rnd, 1, 100, 1200)) for _ in range(100)]
    ps += [(dense(rnd, 1, 15, 40), dense(rnd, 1, 15, 40)) for _ in range(3)]
    plans = H.pairs(ps)[3]
    assert {(p.nprimes > 64) for p in plans} == {True, False} and max(p.nprimes for p in plans) <= 128
    return remaindering_kernels(H, ps)


def many_small_beside_few_large(H):
    rnd = random.Random(5)
    ps = [(dense(rnd, 1, 100, 40), dense(rnd, 1, 100, 40)) for _ in range(90)]
    ps += [(dense(rnd, 1, 10, 1200), dense(rnd, 1, 10, 1200))]
    return remaindering_kernels(H, ps)


def pinned_blocks_of_single_calls(H):
    """Single calls with a small output, then 40, 48 and 80 MiB, then small again; the blocks held after each."""
    rnd = random.Random(6)
    big = [(dense(rnd, 40, 30, 80), dense(rnd, 40, 30, 80)) for _ in range(42)]
    out, held = [], {}
    for n in (0, 21, 25, 42, 0):
        ps = big[:n] or [(dense(rnd, 1, 3, 30), dense(rnd, 1, 3, 30))]
        H.stub.stub_clear()
        assert H.batch(ps) == 0
        words = sum((p.deg_bound + 1) * p.out_nlimbs for p in H.pairs(ps)[3])
        for e in map(str.split, H.log()):
            if e[0] == "host_malloc":
                held[e[1]] = int(e[2])
            elif e[0] == "host_free":
                held.pop(e[1], None)
        out.append(f"{4 * words} " + " ".join(str(v) for v in held.values()))
    return out


def general_first_batch(rnd):
    """Two tails whose first is the pairs above the register classes."""
    return ([(dense(rnd, 70, 8, 64), dense(rnd, 69, 8, 64)) for _ in range(4)] +
            [(dense(rnd, 60, 20, 24), dense(rnd, 59, 20, 24)) for _ in range(4)] +
            [(dense(rnd, 4, 4, 12), dense(rnd, 3, 4, 12))])


def two_tails_class_first(H):
    H.prepare_run(two_class_batch())
    return H.log()


def two_tails_general_first(H):
    H.prepare_run(general_first_batch(random.Random(8)))
    return H.log()


def one_tail_of_one_class(H):
    rnd = random.Random(9)
    H.prepare_run([(dense(rnd, 1, 900, 1500), dense(rnd, 1, 900, 1500)) for _ in range(7)])
    return H.log()


def one_tail_of_a_submitted_run(H):
    h, _ = H.prepare(two_class_batch())
    need = H.L.snc_prepared_stage_bytes(h)
    H.stub.stub_clear()
    assert H.L.snc_prepared_submit(h, C.c_void_p(0x20000000), C.c_size_t(need), H.stream, C.byref(C.c_int64())) == 0
    return H.log()


def static_memory(H):
    H.batch(two_class_batch())
    return [f"{H.loaded} {H.stub.stub_loaded_bytes()}"]


# ---------------------------------------------------------------------------
@pytest.fixture(scope="session")
def stub(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("stub") / "libstub_hip.so")
    subprocess.run(["g++", "-shared", "-fPIC", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include",
                    os.path.join(HERE, "stub_hip.cpp"), "-o", so], check=True)
    return so


def run(stub, scenario):
    r = subprocess.run([sys.executable, os.path.abspath(__file__), stub, scenario], capture_output=True, text=True,
                       timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    return [line.split() for line in r.stdout.splitlines()]


@pytest.mark.parametrize("scenario", ["failed_second_tail_single_call", "failed_second_tail_handle", "failed_submit"])
def test_failed_call_leaves_no_copy_in_flight(stub, scenario):
    log = run(stub, scenario)
    downs = [i for i, e in enumerate(log) if e[0] == "download"]
    side = log[downs[-1]][3]
    assert side != USER and all(log[i][3] == side for i in downs)
    for stream in (side, USER):
        waits = [i for i, e in enumerate(log) if e[:2] == ["stream_sync", stream] and i > downs[-1]]
        assert waits, f"nothing waits for {stream}"
        freed = [i for i, e in enumerate(log) if e[0] in ("host_free", "graph_destroy") and i > downs[-1]]
        assert not freed or waits[0] < freed[0]


def test_one_lane_remaindering_counts_its_own_coefficients(stub):
    few = [e[1] for e in run(stub, "few_small_beside_many_large")]
    assert sum("k_crt_digits" in k for k in few) == 1 and sum("k_crtm_digits" in k for k in few) == 1
    assert not any("k_crt_small" in k for k in few)
    many = [e[1] for e in run(stub, "many_small_beside_few_large")]
    assert sum("k_crt_small" in k for k in many) == 1 and sum("k_crtm_digits" in k for k in many) == 1
    assert not any("k_crt_digits" in k for k in many)


def test_pinned_blocks_kept_by_a_context_are_bounded(stub):
    """The output block a context keeps is at most 64 MiB; a call that needs more returns its own."""
    bound = 64 << 20
    calls = [[int(v) for v in e] for e in run(stub, "pinned_blocks_of_single_calls")]
    assert [c[0] > bound for c in calls] == [False, False, False, True, False]
    assert calls[1][0] > bound // 2
    for need, *held in calls:  # the block for the inputs, smaller here, and the one for the results
        assert max(held) <= bound
        assert need > bound or any(v >= need for v in held)


@pytest.mark.parametrize("scenario,first,second", [
    ("two_tails_class_first", "k_eval_elimILi8", "k_eval_elimILi32"),
    ("two_tails_general_first", "k_elim_general_all", "k_eval_elim"),
])
def test_first_tail_travels_beside_the_second(stub, scenario, first, second):
    log = run(stub, scenario)
    text = [" ".join(e) for e in log]
    launches = [i for i, e in enumerate(log) if e[0] == "graph_launch"]
    downs = [i for i, e in enumerate(log) if e[0] == "download"]
    assert len(launches) == 2
    capture = [i for i, e in enumerate(log) if e[0] == "capture"]
    assert any(first in t for t in text[capture[0]:launches[0]])
    assert not any(second in t for t in text[capture[0]:launches[0]])
    assert any(second in t for t in text[capture[1]:launches[1]])
    assert not any(first in t for t in text[capture[1]:launches[1]])
    early = [i for i in downs if i < launches[1]]
    assert early and len(early) < len(downs)
    side = {log[i][3] for i in early}
    assert len(side) == 1 and USER not in side
    # an event on the caller's stream lies between the tail and its download on the other stream
    assert any(log[i] == ["event_record", USER] for i in range(launches[0], early[0]))
    assert all(log[i][3] == USER for i in downs if i > launches[1])


@pytest.mark.parametrize("scenario", ["one_tail_of_one_class", "one_tail_of_a_submitted_run"])
def test_one_tail(stub, scenario):
    log = run(stub, scenario)
    assert sum(e[0] == "graph_launch" for e in log) == 1
    assert len({e[3] for e in log if e[0] == "download"}) == 1


def test_static_memory_loaded_with_a_context(stub):
    """The tables whose code objects snc_create loads, at 0.42 ms a megabyte: 388 MB, and resultants load no more."""
    created, used = map(int, run(stub, "static_memory")[0])
    assert created < 390e6
    assert used == created


if __name__ == "__main__":
    print("\n".join(globals()[sys.argv[2]](Host(sys.argv[1]))))
    sys.stdout.flush()
    os._exit(0)  # no device to tear down
