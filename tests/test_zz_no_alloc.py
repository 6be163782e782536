"""sage_topm_static (the entry point that allocates nothing) against sage_topm, through the C ABI."""
import ctypes as C

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _scores(n, seed, torch):
    g = torch.Generator(device="cpu").manual_seed(seed)
    a = torch.rand(n, generator=g, dtype=torch.float32) * 2 - 1
    # heavy ties around the threshold, and both zeros
    a[::7] = 0.25
    a[3::1001] = -0.0
    a[5::1003] = 0.0
    return a.cuda()


def test_static_topm_matches_allocating_topm_on_two_calls_in_a_row():
    import torch

    from paper_2510_02470_amd import binding

    L = binding.lib()
    stream = C.c_void_p(torch.cuda.current_stream().cuda_stream)
    # the second call is smaller: what the first left in the shared work space must not leak into it
    for n, m, seed in ((1_000_003, 100_000, 1), (70_001, 3_333, 2), (2_049, 2_049, 3), (5, 1, 4)):
        a = _scores(n, seed, torch)
        want = torch.empty(m, dtype=torch.int64, device="cuda")
        got = torch.full((m,), -1, dtype=torch.int64, device="cuda")
        print("topm_static case", n, m, flush=True)
        assert L.sage_topm(C.c_void_p(a.data_ptr()), n, m, C.c_void_p(want.data_ptr()), stream) == 0
        assert L.sage_topm_static(C.c_void_p(a.data_ptr()), n, m, C.c_void_p(got.data_ptr()), stream) == 0
        torch.cuda.synchronize()
        assert torch.equal(got, want)
        # and against a plain sort of (score descending, index ascending)
        ah = a.cpu().numpy()
        order = np.lexsort((np.arange(n), -(ah + np.float32(0.0))))[:m]
        assert np.array_equal(np.sort(order), got.cpu().numpy())


def test_static_topm_rejects_what_it_cannot_hold():
    import torch

    from paper_2510_02470_amd import binding

    L = binding.lib()
    a = torch.zeros(16, dtype=torch.float32, device="cuda")
    out = torch.zeros(16, dtype=torch.int64, device="cuda")
    p, q = C.c_void_p(a.data_ptr()), C.c_void_p(out.data_ptr())
    # sizes are checked before any pointer is used
    assert L.sage_topm_static(p, binding.TOPM_STATIC_MAX_N + 1, 1, q, None) == binding.SAGE_ERR_CAPACITY
    assert L.sage_topm_static(p, 16, 17, q, None) == binding.SAGE_ERR_ARG
    assert L.sage_topm_static(None, 16, 1, q, None) == binding.SAGE_ERR_ARG
    assert L.sage_topm_static(p, 16, 0, None, None) == 0


def test_static_topm_leaves_its_work_space_clear():
    """Runs that take several launches clear their histograms behind them: calls and replays in any order, at the smallest such
    size, at both block lengths and at the most keys there may be, give what a sort gives."""
    import torch

    from paper_2510_02470_amd import binding

    def check(a, m, got):
        order = torch.sort(a + 0.0, descending=True, stable=True).indices[:m]
        assert torch.equal(torch.sort(order).values, got)

    a = _scores(300_001, 11, torch)
    out = torch.empty(20_000, dtype=torch.int64, device="cuda")
    binding.topm_static(a, 20_000, out)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        binding.topm_static(a, 20_000, out)
    for i, (n, m) in enumerate([(32_769, 1), (4_194_305, 70_000), (binding.TOPM_STATIC_MAX_N, 5), (1000, 10), (40_000, 40_000)]):
        a.copy_(_scores(300_001, 20 + i, torch))
        out.fill_(-1)
        graph.replay()
        check(a, 20_000, out)
        b = _scores(n, 30 + i, torch)
        check(b, m, binding.topm_static(b, m, torch.empty(m, dtype=torch.int64, device="cuda")))


def test_captured_static_topm_relies_on_no_other_run():
    """A run that was cut short leaves the histograms as they were, and a graph may be replayed after it: a captured run has its own
    clearing launch, whatever came before (five kernels; up to 32,768 scores one, which uses no work space)."""
    import torch

    from paper_2510_02470_amd import binding

    hip = C.CDLL(next(l.split()[-1] for l in open("/proc/self/maps") if "libamdhip64" in l))  # (the one that is in use)
    hip.hipGraphGetNodes.argtypes = [C.c_void_p, C.c_void_p, C.POINTER(C.c_size_t)]
    for n, kernels in ((300_001, 5), (32_768, 1)):
        a = _scores(n, n, torch)
        out = torch.empty(3000, dtype=torch.int64, device="cuda")
        want = binding.topm_static(a, 3000, out).clone()
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph(keep_graph=True)
        with torch.cuda.graph(graph):
            binding.topm_static(a, 3000, out)
        nodes = C.c_size_t()
        assert hip.hipGraphGetNodes(graph.raw_cuda_graph(), None, C.byref(nodes)) == 0
        assert nodes.value == kernels
        for _ in range(3):
            out.fill_(-1)
            graph.replay()
            assert torch.equal(out, want)
