"""BR-H calls with decode steps: which launch applies them (on the host, by the kernels launched on a stand-in for the runtime), and the
results on both sides of that rule against the oracle."""
import os
import re
import subprocess
import sys

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

from tests.test_failed_launch import STAND_IN, Library, build  # noqa: E402

# clusters, workers, slots, queue, horizon, gate, decode steps: by the waves that have routed the cluster
BY_THE_ROUND = [
    (3073, 8, 256, 64, 4, 0.0, 8), (3073, 5, 256, 300, 8, 0.0, 9), (4096, 40, 40, 40, 4, 0.0, 20), (3073, 13, 130, 60, 7, 0.0, 8),
    (4096, 4, 256, 40, 8, 0.3, 16), (3300, 9, 131, 260, 6, 0.3, 16), (3400, 16, 80, 128, 5, 0.3, 25),
]
# and one step outside the rule each: by the projection
BY_THE_PROJECTION = [
    (3072, 9, 256, 64, 4, 0.0, 8), (4097, 8, 256, 64, 4, 0.0, 8), (3073, 8, 256, 64, 4, 0.0, 7), (3073, 7, 256, 64, 4, 0.0, 8), (3073, 10, 256, 64, 3, 0.0, 8),
    (4096, 4, 256, 40, 8, 0.3, 15), (3073, 3, 256, 40, 8, 0.3, 16), (4096, 7, 256, 40, 8, 0.3, 16), (3100, 17, 80, 128, 6, 0.3, 25),
]

# both sides of the lines of the projection's pass, below and above 2048 clusters: in it or not, clusters, workers, slots, queue, horizon, mode of prediction, window
SIDES = [
    (True, 3, 5, 256, 200, 4, 0, 4), (False, 3, 5, 257, 200, 4, 0, 4), (True, 2050, 3, 256, 64, 4, 0, 4), (False, 2050, 3, 257, 64, 4, 0, 4),
    (True, 2, 6, 60, 512, 8, 0, 4), (False, 2, 6, 60, 513, 8, 0, 4), (True, 2050, 2, 20, 512, 3, 0, 4), (False, 2050, 2, 20, 513, 3, 0, 4),
    (True, 3, 7, 60, 200, 6, 0, 8), (False, 3, 7, 60, 200, 6, 0, 9), (True, 2050, 3, 30, 64, 4, 3, 8), (False, 2050, 3, 30, 64, 4, 3, 9),
    (True, 3, 6, 60, 200, 4, 1, 5), (False, 3, 6, 60, 200, 4, 2, 5), (True, 2050, 3, 30, 64, 8, 1, 6), (False, 2050, 3, 30, 64, 8, 2, 6),
]


def places(lib):
    from paper_2605_06113_amd import workloads as wl
    for where, cases in (("round", BY_THE_ROUND), ("projection", BY_THE_PROJECTION)):
        for N, G, B, Q, H, gate, steps in cases:
            lib.context(wl.RouteConfig(name="places", n_inst=N, G=G, B=B, max_wait=Q, H=H, gate_pfin=gate))
            for scores in (False, True):
                rc, _ = lib.advance(steps, scores=scores)
                got = " ".join(re.findall(r"br_k_[a-zA-Z0-9_]*?E(?=Ev)", lib.log))
                size = f"ILi{4 if Q <= 256 else 8}ELi{4 if H <= 4 else 8}E"
                if where == "round":
                    want = rf"br_k_project_rows\S* br_k_route_h{size}Lb1E"
                else:
                    want = rf"br_k_project_advance\S* br_k_(route_h{size}Lb0E|assign{size}Li0\S*)"
                assert rc == 0 and re.fullmatch(want, got), f"{where} {(N, G, B, Q, H, gate, steps)} scores={scores}: {got}"
            lib.free()


def sides(lib):
    from paper_2605_06113_amd import workloads as wl
    for ahead, N, G, B, Q, H, mode, R in SIDES:
        lib.context(wl.RouteConfig(name="sides", n_inst=N, G=G, B=B, max_wait=Q, H=H, pred_mode=mode, R_max=R))
        for scores in (False, True):
            rc, got = lib.advance(5, scores=scores)
            case = f"{(N, G, B, Q, H, mode, R)} scores={scores}: {got}"
            assert rc == 0 and ("br_k_project_advance" in got) == ahead and any(k.startswith("br_k_advance") for k in got) != ahead, case
            assert lib.advance(0, scores=scores)[1][0] == "br_k_project_rows", case
        lib.free()


def lds(lib):
    """A BR-0 round has no room for what the projection of a BR-H call leaves to it."""
    from paper_2605_06113_amd import workloads as wl
    for H, more in ((0, 0), (4, 192)):
        lib.context(wl.RouteConfig(name="lds", n_inst=4, G=8, B=20, max_wait=200, H=H))
        assert lib.call("br_route_step", None, None)[0] == 0
        assert int(re.search(r"br_k_assign\S* lds=(\d+)", lib.log).group(1)) == (4 * 64 + 4 * 64 + 64 + more) * 4
        lib.free()


@pytest.mark.parametrize("scenario", ["places", "sides", "lds"])
def test_launches(tmp_path, scenario):
    run = subprocess.run([sys.executable, os.path.abspath(__file__), build(tmp_path, STAND_IN), scenario], cwd=ROOT, capture_output=True, text=True, timeout=300)
    assert run.returncode == 0, run.stderr[-2000:]


@pytest.mark.gpu
@pytest.mark.parametrize("N,G,B,Q,H,gate,steps", BY_THE_ROUND)
def test_decode_steps_by_the_waves_of_the_round(N, G, B, Q, H, gate, steps):
    """Lists of every width, rows of whole 16-byte words and of five to seven floats, workers that lose nothing, something and everything, clusters
    without arrivals and without free slots."""
    from oracle import br_oracle
    from paper_2605_06113_amd import binding, workloads as wl
    from tests.parity import compare_outputs, compare_state
    cfg, init, arr = wl.random_case(1600 + N + B + H, N=N, G=G, B=B, max_wait=Q, H=H, fill=0.7, n_wait=Q // 3, gate_pfin=gate)
    rng = np.random.default_rng(B + H)
    arr.count[::7] = np.arange(len(arr.count[::7])) % 9
    arr.o[:, ::3] = 1 + arr.o[:, ::3] % (2 * steps)
    init.rem[:] = np.where((rng.random((N, G, 1)) < 0.4) & (init.rem > 0), init.rem + 3 * steps, init.rem)
    for i, g, n, rem in ((0, 0, 0, 0), (1, G - 1, B, 500), (2, 0, B, 1)):
        init.n[i, g] = n
        init.rem[i, g, :n], init.kv[i, g, :n] = rem, np.maximum(init.kv[i, g, :n], 1)
    print(f"[case] decode by the round N={N} G={G} B={B} Q={Q} H={H} gate={gate} steps={steps}", flush=True)
    oc, r = br_oracle.OracleCluster(cfg, init), binding.Router(cfg, init)
    for rnd in range(3):
        ref = oc.route_step(arr)
        out = r.route_step(arr, matrix=rnd == 1, scores=rnd < 2, advance=steps)
        compare_outputs({k: v for k, v in ref.items() if k in out}, out, cfg, f"decode by the round r{rnd}")
        oc.advance(steps)
        compare_state(oc, r.state(), cfg, f"decode by the round r{rnd}")
    r.close()


@pytest.mark.gpu
@pytest.mark.parametrize("gate,watermark", [(0.3, False), (0.0, True)])
@pytest.mark.parametrize("ahead,N,G,B,Q,H,mode,R", SIDES)
def test_both_sides_of_the_projections_pass(ahead, N, G, B, Q, H, mode, R, gate, watermark):
    """Windows of 4 to 9, with and without gate and token watermark, calls that ask for the reductions, for nothing and for the decisions, without
    arrivals; and where the decode steps ran."""
    from oracle import br_oracle
    from paper_2605_06113_amd import binding, workloads as wl
    from tests.parity import compare_outputs, compare_state
    steps = 6
    cfg, init, arr = wl.random_case(1700 + N + B + Q + R + mode, N=N, G=G, B=B, max_wait=Q, H=H, fill=0.7, n_wait=Q // 2, pred_mode=mode, gate_pfin=gate, R_max=R,
                                    token_watermark=int(B * 0.7 * 2048 * 1.05) if watermark else 0)
    arr.o[:, ::2] = 1 + arr.o[:, ::2] % (2 * steps)
    init.n[0, 0] = 0
    hist = np.sort(np.random.default_rng(N + B).integers(1, 60, 500)).astype(np.int32) if mode == 2 else None
    print(f"[case] sides N={N} G={G} B={B} Q={Q} H={H} mode={mode} R={R} gate={gate} watermark={cfg.token_watermark}", flush=True)
    oc, r = br_oracle.OracleCluster(cfg, init, hist=hist), binding.Router(cfg, init, hist=hist)
    r.profile(True)
    nothing = wl.Arrivals(arr.count * 0, arr.s, arr.o, arr.id, arr.pred)
    for rnd in range(4):
        a = nothing if rnd == 2 else arr
        ref = oc.route_step(a)
        if rnd == 1:
            r.route_advance_device(binding.DeviceArrivals(a, "cuda:0", r.Pq), {}, steps)
        else:
            out = r.route_step(a, matrix=False, scores=rnd == 0, advance=steps)
            compare_outputs({k: v for k, v in ref.items() if k in out}, out, cfg, f"sides r{rnd}")
        oc.advance(steps)
        compare_state(oc, r.state(), cfg, f"sides r{rnd}")
    ran = {k: n for k, (_, n) in r.profile_read().items()}
    assert ran["project"] == 4 and ran["assign"] == 4 and ran["advance"] == (0 if ahead else 4), ran
    r.close()


if __name__ == "__main__":
    {"places": places, "sides": sides, "lds": lds}[sys.argv[2]](Library(sys.argv[1]))
