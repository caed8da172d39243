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


def lds(lib):
    """A BR-0 round has no room for what the projection of a BR-H call leaves to it."""
    from paper_2605_06113_amd import workloads as wl
    for H, more in ((0, 0), (4, 192)):
        lib.context(wl.RouteConfig(name="lds", n_inst=4, G=8, B=20, max_wait=200, H=H))
        assert lib.call("br_route_step", None, None)[0] == 0
        assert int(re.search(r"br_k_assign\S* lds=(\d+)", lib.log).group(1)) == (4 * 64 + 4 * 64 + 64 + more) * 4
        lib.free()


@pytest.mark.parametrize("scenario", ["places", "lds"])
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
    for rnd in range(2):
        ref = oc.route_step(arr)
        out = r.route_step(arr, matrix=False, scores=rnd == 0, advance=steps)
        compare_outputs({k: v for k, v in ref.items() if k in out}, out, cfg, f"decode by the round r{rnd}")
        oc.advance(steps)
        compare_state(oc, r.state(), cfg, f"decode by the round r{rnd}")
    r.close()


if __name__ == "__main__":
    {"places": places, "lds": lds}[sys.argv[2]](Library(sys.argv[1]))
