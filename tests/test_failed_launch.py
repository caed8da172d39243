"""Calls in which a launch or an event fails, on the host alone: the HIP runtime's entry points that the library calls are taken by a
small stand-in that notes which kernels are launched, runs none, and fails the calls it is told to.  In a process of its own."""
import ctypes as C
import os
import re
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

STAND_IN = r"""
#include <cstddef>
#include <cstdint>
#include <map>
#include <string>
struct D3 { uint32_t x, y, z; };
static std::map<const void *, std::string> names;
static std::string log_;
static int fail_launch, fail_create, fail_record, last, captured;  // fail_*: the n-th call from now on (0: none)
static bool hit(int &n) { return n > 0 && --n == 0; }
static D3 g, b; static size_t shm; static void *str;
extern "C" {
void **__hipRegisterFatBinary(const void *) { static void *h; return &h; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *f, char *, const char *n, unsigned, void *, void *, void *, void *, int *) { names[f] = n; }
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
int __hipPushCallConfiguration(D3 gg, D3 bb, size_t s, void *st) { g = gg, b = bb, shm = s, str = st; return 0; }
int __hipPopCallConfiguration(D3 *gg, D3 *bb, size_t *s, void **st) { *gg = g, *bb = b, *s = shm, *st = str; return 0; }
int hipLaunchKernel(const void *f, D3, D3, void **, size_t lds, void *) {
  if (hit(fail_launch)) return last = 2;
  log_ += names[f] + " lds=" + std::to_string(lds) + "\n";
  return 0;
}
int hipGetLastError() { int e = last; last = 0; return e; }
int hipEventCreate(void **e) { static char c; *e = &c; return hit(fail_create) ? 2 : 0; }
int hipEventDestroy(void *) { return 0; }
int hipEventRecord(void *, void *) { return hit(fail_record) ? 400 : 0; }
int hipEventSynchronize(void *) { return 0; }
int hipEventElapsedTime(float *t, void *, void *) { *t = 1.0f; return 0; }
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipGetSymbolAddress(void **p, const void *) { *p = (void *)0x1000; return 0; }
int hipStreamIsCapturing(void *, int *s) { *s = captured; return 0; }
void stand_in(int launch, int create, int record, int cap) { fail_launch = launch, fail_create = create, fail_record = record, captured = cap; }
const char *stand_in_log() { static std::string out; out = log_; log_.clear(); return out.c_str(); }
}
"""

# the same for launches alone, in front of the real runtime
ON_THE_GPU = r"""
#include <cstddef>
#include <cstdint>
struct D3 { uint32_t x, y, z; };
typedef int (*Launch)(const void *, D3, D3, void **, size_t, void *);
typedef int (*Last)();
static Launch real_launch;
static Last real_last;
static int fail_launch, last;
extern "C" {
void in_front(void *launch, void *last_error) { real_launch = (Launch)launch, real_last = (Last)last_error; }
void fail(int n) { fail_launch = n; }
int hipLaunchKernel(const void *f, D3 g, D3 b, void **a, size_t s, void *st) {
  if (fail_launch > 0 && --fail_launch == 0) return last = 2;
  return real_launch(f, g, b, a, s, st);
}
int hipGetLastError() { int e = last; last = 0; return e ? e : real_last(); }
}
"""


class Library:
    """The library on the stand-in: `call` returns its code and the kernels it launched."""

    def __init__(self, so):
        self.fake = C.CDLL(so, mode=C.RTLD_GLOBAL)
        self.fake.stand_in_log.restype = C.c_char_p
        from paper_2605_06113_amd import binding
        self.binding, self.lib = binding, binding.load()

    def context(self, cfg):
        hist = dict(hist=1 << 30, hist_sum=1 << 30, hist_n=100) if cfg.H > 0 and cfg.pred_mode == 2 else {}
        c = self.binding.make_config(cfg, workspace=1 << 20, workspace_bytes=1 << 40, **hist)
        self.ctx = C.c_void_p()
        assert self.lib.br_init(C.byref(c), None, C.byref(self.ctx)) == 0
        self.fake.stand_in_log()

    def call(self, name, *args, launch=0, create=0, record=0, capture=0):
        self.fake.stand_in(launch, create, record, capture)
        rc = getattr(self.lib, name)(self.ctx, *args)
        self.fake.stand_in(0, 0, 0, 0)
        self.log = self.fake.stand_in_log().decode()
        return rc, re.findall(r"br_k_[a-z_0-9]*[a-z]", self.log)

    def free(self):
        self.lib.br_free(self.ctx)

    def advance(self, steps, scores=False, **fail):
        out = self.binding.StepOut(best_g=1 << 30, best_i=1 << 30) if scores else self.binding.StepOut()
        return self.call("br_route_advance", None, C.byref(out), steps, **fail)


def lookahead():
    from paper_2605_06113_amd import workloads as wl
    return wl.config("c3", n_inst=4, max_wait=200, B=96, G=16, H=4)


def a_failed_round_is_resumed(lib):
    lib.context(lookahead())
    whole = (0, ["br_k_project_advance", "br_k_assign"])
    assert lib.advance(5) == whole
    assert lib.advance(5, launch=2) == (-3, ["br_k_project_advance"])
    assert lib.lib.br_last_hip_error(lib.ctx) == 2
    for other in (lambda: lib.advance(4), lambda: lib.advance(0), lambda: lib.call("br_route_step", None, None), lambda: lib.advance(5, capture=1),
                  lambda: lib.call("br_route_step_static", None, None), lambda: lib.call("br_advance_decode", 5)):
        assert other() == (-3, [])
    assert lib.advance(5, launch=1) == (-3, [])       # (fails again)
    assert lib.advance(5, scores=True) == (0, ["br_k_route_helped"])  # the round alone, whatever is asked of it
    assert lib.advance(5) == whole and lib.advance(3) == whole
    assert lib.advance(5, launch=1) == (-3, [])       # nothing was launched: nothing to resume
    assert lib.advance(2) == whole
    assert lib.advance(5, launch=2, capture=1) == (-3, ["br_k_project_advance"])  # a capture that failed has run nothing
    assert lib.advance(2) == whole


def a_failed_round_of_calls_that_only_project_is_run_again(lib):
    lib.context(lookahead())
    assert lib.call("br_route_step", None, None, launch=2) == (-3, ["br_k_project_rows"])
    assert lib.advance(5) == (0, ["br_k_project_advance", "br_k_assign"])


def events_are_there_before_the_first_launch(lib):
    lib.context(lookahead())
    assert lib.call("br_profile_enable", 1) == (0, [])
    for n in (1, 2, 5, 8):  # (pairs created one after the other)
        assert lib.advance(5, create=n) in ((-3, []), (0, ["br_k_project_advance", "br_k_assign"]))
    assert lib.call("br_profile_read", (C.c_double * 7)(), (C.c_int64 * 7)()) == (0, [])
    assert lib.advance(5, create=1) == (0, ["br_k_project_advance", "br_k_assign"])  # (those read are there again)


def a_failed_record_says_what_is_on_the_stream(lib):
    lib.context(lookahead())
    assert lib.call("br_profile_enable", 1) == (0, [])
    whole = (0, ["br_k_project_advance", "br_k_assign"])
    assert lib.advance(5, record=1) == (-3, []) and lib.advance(2) == whole                       # before the projection
    assert lib.advance(5, record=2) == (-3, ["br_k_project_advance"])                             # behind it
    assert lib.advance(2) == (-3, []) and lib.advance(5) == (0, ["br_k_assign"])
    assert lib.advance(5, record=3) == (-3, ["br_k_project_advance"])                             # before the round
    assert lib.advance(5) == (0, ["br_k_assign"])
    assert lib.advance(5, record=4) == (-3, whole[1]) and lib.advance(2) == whole                 # behind the round: it is on the stream


SCENARIOS = [a_failed_round_is_resumed, a_failed_round_of_calls_that_only_project_is_run_again, events_are_there_before_the_first_launch,
             a_failed_record_says_what_is_on_the_stream]


def a_resumed_round_is_that_of_a_call_that_did_not_fail(so):
    """On the GPU: a call whose round is not launched, then the same call again, against the oracle."""
    import numpy as np
    import torch
    torch.zeros(1, device="cuda:0")
    path = next(line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64" in line)
    real, front = C.CDLL(path), C.CDLL(so, mode=C.RTLD_GLOBAL)
    front.in_front(C.cast(real.hipLaunchKernel, C.c_void_p), C.cast(real.hipGetLastError, C.c_void_p))
    from oracle import br_oracle
    from paper_2605_06113_amd import binding, workloads as wl
    from tests.parity import compare_outputs, compare_state
    for H, mode, scores in ((4, 0, True), (8, 3, False)):
        cfg, init, arr = wl.random_case(77 + H, N=5, G=9, B=40, max_wait=300, H=H, fill=0.7, n_wait=120, pred_mode=mode, gate_pfin=0.3)
        arr.o[:, ::2] = 1 + arr.o[:, ::2] % 7
        oc, r = br_oracle.OracleCluster(cfg, init), binding.Router(cfg, init)
        nothing = wl.Arrivals(arr.count * 0, arr.s, arr.o, arr.id, arr.pred)
        for rnd in range(3):
            front.fail(2 if rnd == 1 else 0)
            if rnd == 1:
                with pytest.raises(binding.BrError):
                    r.route_step(nothing, matrix=False, scores=scores, advance=6)
                with pytest.raises(binding.BrError):
                    r.advance(6)
            ref, out = oc.route_step(arr), r.route_step(arr, matrix=False, scores=scores, advance=6)
            compare_outputs({k: v for k, v in ref.items() if k in out}, out, cfg, f"resumed H={H} r{rnd}")
            oc.advance(6)
            compare_state(oc, r.state(), cfg, f"resumed H={H} r{rnd}")
        assert int(np.sum(oc.n)) > 0
        r.close()


def build(at, source):
    (at / "hip.cpp").write_text(source)
    subprocess.check_call(["g++", "-shared", "-fPIC", "-O1", "-o", str(at / "hip.so"), str(at / "hip.cpp")])
    return str(at / "hip.so")


@pytest.fixture(scope="module")
def stand_in(tmp_path_factory):
    return build(tmp_path_factory.mktemp("hip"), STAND_IN)


def in_a_process(so, scenario, seconds):
    run = subprocess.run([sys.executable, os.path.abspath(__file__), so, scenario.__name__], cwd=ROOT, capture_output=True, text=True, timeout=seconds)
    assert run.returncode == 0, run.stderr[-2000:]


@pytest.mark.parametrize("scenario", SCENARIOS, ids=lambda f: f.__name__)
def test_failed_calls(stand_in, scenario):
    in_a_process(stand_in, scenario, 300)


@pytest.mark.gpu
def test_resumed_round_on_the_gpu(tmp_path):
    in_a_process(build(tmp_path, ON_THE_GPU), a_resumed_round_is_that_of_a_call_that_did_not_fail, 100)


if __name__ == "__main__":
    sys.path.insert(0, ROOT)
    run = next((f for f in SCENARIOS if f.__name__ == sys.argv[2]), None)
    if run:
        run(Library(sys.argv[1]))
    else:
        a_resumed_round_is_that_of_a_call_that_did_not_fail(sys.argv[1])
