"""The lifetime of the captured iterations of a solve's stages (csrc/stage_graphs.h, the code the
solves run): on the CPU with a simulated stream (tests/serve/stage_graphs.cpp), no graph goes before
its launches have run and a long schedule holds four at a time; on the GPU, a solve of many
stages replays to the bits of the eager one."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def sim(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("no host C++ compiler")
    exe = str(tmp_path_factory.mktemp("stages") / "stage_graphs")
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_1210_4931_amd", "csrc"),
                    os.path.join(ROOT, "tests", "serve", "stage_graphs.cpp"), "-o", exe], check=True)

    def run(stages):
        text = "%d\n" % len(stages) + "".join("%d %d\n" % s for s in stages)
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True, timeout=60)
        early, most, left, waited = map(int, out.stdout.split())
        return early, most, left, waited
    return run


# (launches, ticks until the next stage): a stream that keeps up, one that never runs by itself, one
# that falls behind, single stages
@pytest.mark.parametrize("stages,most", [([(5, 9)] * 300, 1), ([(7, 0)] * 300, 4), ([(10, 8)] * 300, 4), ([(3, 0)], 1),
                                         ([(100, 1), (1, 0), (1, 0)], 3)])
def test_graphs_outlive_their_launches_and_stay_few(sim, stages, most):
    early, got, left, waited = sim(stages)
    assert early == 0 and left == 0
    assert got == most and waited <= sum(s[0] for s in stages)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_many_stages_replay_to_the_eager_bits(dtype):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1210_4931_amd import mfwf
    from paper_1210_4931_amd import workloads as W
    nside, lmax, n = 16, 32, 2
    g = torch.Generator(device="cuda").manual_seed(2)
    d = torch.randn(n, 12 * nside * nside, generator=g, dtype=torch.float64, device="cuda")
    p = mfwf.Plan(nside, lmax, max_batch=n, dtype=dtype)
    p.set_covariances(W.cl_damped(lmax, 20.0), torch.rand(12 * nside * nside, generator=g, dtype=torch.float64, device="cuda") + 0.5)
    lam = [1.0 + 99.0 / (k + 1) for k in range(60)] + [1.0]
    its = [3 + k % 4 for k in range(61)]
    a, m, _ = p.solve(d, lam=lam, iters=its, use_graph=False)
    for n_check in (0, 7):  # stages that end in a check and stages that do not
        b, q, *_ = p.solve(d, lam=lam, iters=its, n_check=n_check)
        assert torch.equal(a, b) and torch.equal(m, q)
