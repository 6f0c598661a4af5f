"""Group-kernel contexts on streams of their own, at the same time: every run ends and gives the bits that it
gives alone, whatever part of the chip it gets. Enqueued by one thread (several runs per stream without waiting),
by a thread per context, as replays of a recorded graph beside eager runs of other contexts, and beside a kernel
without groups that holds some of the CUs for about two seconds."""
import threading

import numpy as np
import pytest

import instances

pytestmark = pytest.mark.gpu

T_F = 400


def _normal(n):
    u = np.triu(np.random.default_rng(n).normal(size=(n, n)), 1)
    return u + u.T


# few replicas on the whole chip, the large tile, real couplings, FP8 spins
KINDS = {
    "sk2000_r100": (lambda: instances.sk(2000, 91).J, "bf16", 100),
    "g2000_r1024": (lambda: instances.gnp(2000, 0.5, 92).J, "fp8j_bf16s", 1024),
    "normal1500_r40": (lambda: _normal(1500), "bf16", 40),
    "g1000_fp8s_r200": (lambda: instances.gnp(1000, 0.5, 93).J, "fp8j_fp8s", 200),
    "sk300_r64": (lambda: instances.sk(300, 94).J, "bf16", 64),
    "5sk1300_r1024": (lambda: 5.0 * instances.sk(1300, 95).J, "bf16", 1024),
}


@pytest.fixture(scope="module")
def env():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1806_08422_amd import nmfa

    solvers, want = {}, {}
    for name, (make, precision, R) in KINDS.items():
        s = nmfa.Solver(make(), None, precision=precision)
        solvers[name], want[name] = s, []
        for seed in (1, 2):
            s.anneal(R, T_F, seed)
            want[name].append((s.energies()[0], s.spins()))
    yield nmfa, torch, solvers, want
    for s in solvers.values():
        s.close()


def _same(s, want):
    assert np.array_equal(s.energies()[0], want[0]) and np.array_equal(s.spins(), want[1])


@pytest.mark.parametrize("names", [
    ("sk2000_r100", "normal1500_r40"), ("g2000_r1024", "sk300_r64", "sk2000_r100"), tuple(KINDS)])
def test_one_thread(env, names):
    nmfa, torch, solvers, want = env
    streams = [torch.cuda.Stream() for _ in names]
    for round_ in range(3):
        for seed in (2, 1):  # the second run waits for the first on its own stream only
            for name, st in zip(names, streams):
                solvers[name].anneal(KINDS[name][2], T_F, seed, st.cuda_stream)
        for name in names:
            _same(solvers[name], want[name][0])


def test_a_thread_each(env):
    nmfa, torch, solvers, want = env
    failures = []

    def work(name, stream):
        try:
            for k in range(6):
                solvers[name].anneal(KINDS[name][2], T_F, 1 + k % 2, stream.cuda_stream)
                _same(solvers[name], want[name][k % 2])
        except BaseException as e:  # reported by the main thread
            failures.append((name, repr(e)))

    threads = [threading.Thread(target=work, args=(name, torch.cuda.Stream())) for name in KINDS]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not failures


def test_replays_beside_eager_runs(env):
    nmfa, torch, solvers, want = env
    made = {}
    for name in ("sk2000_r100", "normal1500_r40", "g1000_fp8s_r200"):
        make, precision, R = KINDS[name]
        s = nmfa.Solver(make(), None, precision=precision)
        s.anneal(R, T_F, 1)  # allocates
        s.energies()
        g = torch.cuda.CUDAGraph()
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.graph(g, stream=side):
            s.anneal(R, T_F, 2, torch.cuda.current_stream().cuda_stream)
        made[name] = (s, g, torch.cuda.Stream())
    torch.cuda.synchronize()
    other = torch.cuda.Stream()
    for round_ in range(4):
        for s, g, st in made.values():
            with torch.cuda.stream(st):
                g.replay()
        solvers["sk2000_r100"].anneal(100, T_F, 1, other.cuda_stream)
        solvers["sk300_r64"].anneal(64, T_F, 2, other.cuda_stream)
        torch.cuda.synchronize()
        for name, (s, g, st) in made.items():
            _same(s, want[name][1])
        _same(solvers["sk2000_r100"], want["sk2000_r100"][0])
        _same(solvers["sk300_r64"], want["sk300_r64"][1])
    for s, g, st in made.values():
        del g
        s.close()


def test_beside_a_long_kernel(env):
    nmfa, torch, solvers, want = env
    st = [torch.cuda.Stream(), torch.cuda.Stream()]
    with nmfa.Solver(instances.sk(31, 98).J, None, precision="fp64") as long_run:
        long_run.anneal(1024, 1000, 1)
        per_iteration = long_run.last_timing()["anneal_ms"] / 1000
        t_f = int(2000 / per_iteration)
        long_run.anneal(1024, t_f, 1, st[0].cuda_stream)
        solvers["sk2000_r100"].anneal(100, T_F, 1, st[1].cuda_stream)
        _same(solvers["sk2000_r100"], want["sk2000_r100"][0])
        assert long_run.last_timing()["launches"] == 1
