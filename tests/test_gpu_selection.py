"""Selections at the edges of their variants: one work-group against several, slices of a work-group, class sizes around
the rank / radix boundary, ties at every threshold."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [1, 63, 1024, 1025, 2047, 2049, 4097, 8193, 16_385, 32_767, 32_768, 32_769, 36_865, 600_001])
@pytest.mark.parametrize("ties", [False, True])
def test_topm_at_the_edges_of_its_variants(N, ties):
    import torch

    from paper_2510_02470_amd.binding import topm, topm_static

    rng = np.random.default_rng(N)
    a = (rng.integers(-3, 4, size=N) / 4.0 if ties else np.tanh(0.1 + 0.3 * rng.standard_normal(N))).astype(np.float32)
    ad = torch.from_numpy(a).cuda()
    for m in sorted({1, (N + 2) // 3, N - 1, N} - {0}):
        want = oracle.topm_f32(a, m).tolist()
        assert topm(ad, m).cpu().tolist() == want
        assert topm_static(ad, m, torch.empty(m, dtype=torch.int64, device="cuda")).cpu().tolist() == want


# work-groups of the histograms: one a block, 64, a quarter of the blocks; blocks of 4096 keys, then of 16,384
@pytest.mark.parametrize("N", [65 * 4096, 257 * 4096 + 1, 4_194_304, 4_194_305, 5_000_003])
@pytest.mark.parametrize("ties", [False, True])
def test_topm_at_the_edges_of_its_blocks(N, ties):
    import torch

    from paper_2510_02470_amd.binding import topm, topm_static

    rng = np.random.default_rng(N)
    a = (rng.integers(-3, 4, size=N) / 4.0 if ties else np.tanh(0.1 + 0.3 * rng.standard_normal(N))).astype(np.float32)
    ad = torch.from_numpy(a).cuda()
    for m in (1, N // 100, N - 1):
        want = oracle.topm_f32(a, m)
        assert np.array_equal(topm(ad, m).cpu().numpy(), want)
        assert np.array_equal(topm_static(ad, m, torch.empty(m, dtype=torch.int64, device="cuda")).cpu().numpy(), want)


# class sizes: the rank select takes up to 256 rows; a mean above 256 rows takes the wider work-group; many classes leave
# no room for counters in LDS
@pytest.mark.parametrize("sizes", [(255, 256, 257, 0, 1, 30), (3000, 256, 257, 1025), (5000,), (2,) * 300 + (700,),
                                   (1,) * 4090 + (0,) * 10], ids=["small", "large", "single", "many", "no_lds"])
@pytest.mark.parametrize("distinct", [3, 100_000])
def test_class_selection_at_the_edges_of_its_variants(sizes, distinct):
    import torch

    from paper_2510_02470_amd.binding import Sage

    rng = np.random.default_rng(len(sizes))
    N, C = sum(sizes), len(sizes)
    labels = rng.permutation(np.repeat(np.arange(C), sizes)).astype(np.int32)
    G = rng.standard_normal((min(distinct, N), 40)).astype(np.float32)[rng.integers(0, min(distinct, N), size=N)]
    s = Sage(16, 40)
    s.set_basis(torch.from_numpy(rng.standard_normal((6, 40)).astype(np.float32)).cuda())
    s.score_labeled(torch.from_numpy(G).cuda(), torch.from_numpy(labels).cuda())
    for keep in (0.03, 0.4, 0.999):
        for rule in ("proportional", "equal"):
            idx = s.select_cb(keep, C, rule=rule).cpu().numpy()
            want = oracle.cb_select_from_alpha(s.scores().cpu().numpy(), labels, C, keep, rule)
            assert idx.tolist() == want.tolist()
    s.close()


# Rows of any width and start: whole windows only, a partial one, less than one; every basis width; a batch that starts in the
# middle of a line. The 3-part products are good to fp32, so the tolerance is fp32's.
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("D", [31, 33, 64, 65, 127, 1001, 4099])
@pytest.mark.parametrize("k", [3, 40, 100])
def test_projection_of_rows_of_any_alignment(dtype, D, k):
    import torch

    from paper_2510_02470_amd.binding import Sage

    rng = np.random.default_rng(D + k)
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    n = 700
    flat = torch.from_numpy(rng.standard_normal(n * D + 1).astype(np.float32)).to(td).cuda()
    G = flat[1:].view(n, D)  # not on a multiple of 16 bytes
    V = torch.from_numpy(rng.standard_normal((k, D)).astype(np.float32)).cuda()
    s = Sage(max(2 * k, 2), D, dtype=dtype, max_rows=2 * n)
    s.set_basis(V)
    s.score(G)
    s.score(G[:1].clone())
    got = s.zhat().cpu().double()
    Z = G.double().cpu() @ V.double().cpu().T
    norm = Z.norm(dim=1, keepdim=True)
    scale = G.double().cpu().norm(dim=1, keepdim=True) * V.double().cpu().norm(dim=1).max()
    assert ((got[:n] - Z / norm).abs() * norm / scale).max() <= 3e-7
    assert (got[n] - got[0]).abs().max() <= 1e-4  # (an aligned start may take the two-part basis)
    s.close()


# Rows on multiples of 8 columns, and of 4 (a basis in three parts): one window to some, partial ones, rows that start anywhere
# in a line, row counts that end inside a wave's rows and at each number of row loads, several row tiles, a batch over 4 GiB
# (lane offsets have 32 bits).
@pytest.mark.parametrize("n,D,k,dtype", [(n, D, k, t) for n in (1, 63, 700) for D in (64, 72, 1000) for k in (3, 40, 100)
                                         for t in ("f32", "bf16")]
                         + [(n, D, k, "f32") for n in (1, 63, 700) for D in (36, 68, 100, 1004) for k in (3, 40, 100)]
                         + [(n, D, k, t) for n in (64, 65, 128, 129, 256, 257) for D, k in ((1000, 40), (1001, 100))
                            for t in ("f32", "bf16")]
                         + [(1100, 1_048_576, 100, "f32"), (1100, 1_048_580, 100, "f32"), (1100, 2_049_000, 100, "bf16"),
                            (1100, 2_049_001, 100, "bf16")])
def test_projection_of_aligned_rows_at_the_edges_of_its_tiles(n, D, k, dtype):
    import torch

    from paper_2510_02470_amd.binding import Sage

    gen = torch.Generator(device="cuda").manual_seed(n + D + k)
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    off = 8 if D % 8 == 0 else 4 if D % 4 == 0 else 1
    flat = torch.empty(n * D + off, dtype=td, device="cuda")
    for i in range(0, n * D + off, 1 << 28):
        part = flat[i:i + (1 << 28)]
        part.copy_(torch.randn(part.numel(), generator=gen, device="cuda"))
    G = flat[off:].view(n, D)
    V = torch.randn(k, D, generator=gen, device="cuda")
    s = Sage(max(2 * k, 2), D, dtype=dtype, max_rows=n)
    s.set_basis(V)
    s.score(G)
    got = s.zhat().double()
    Vd = V.double().T.contiguous()
    Z = torch.cat([G[i:i + 32].double() @ Vd for i in range(0, n, 32)])
    norm = Z.norm(dim=1, keepdim=True)
    scale = torch.cat([G[i:i + 32].double().norm(dim=1, keepdim=True) for i in range(0, n, 32)]) * V.double().norm(dim=1).max()
    # Rows and basis in two bf16 parts: each good to 2^-17, and their low parts' product of 2^-18 is left out. Three parts are
    # good to fp32.
    tol = 2.0 ** -16 + 2.0 ** -18 if D % 8 == 0 else 3e-7
    assert float(((got - Z / norm).abs() * norm / scale).max()) <= tol
    s.close()


# the answer's signal: more callers than words, and the largest export that one work-group copies
def test_topm_from_many_threads():
    from concurrent.futures import ThreadPoolExecutor

    import torch

    from paper_2510_02470_amd.binding import topm

    def calls(i):
        with torch.cuda.stream(torch.cuda.Stream()):
            a = np.random.default_rng(i).standard_normal(500 + 37 * i).astype(np.float32)
            ad = torch.from_numpy(a).cuda()
            return all(topm(ad, m).cpu().tolist() == oracle.topm_f32(a, m).tolist() for m in (1, 7, 200, 499))

    with ThreadPoolExecutor(40) as pool:
        assert all(pool.map(calls, range(80)))


@pytest.mark.parametrize("N", [1, 1025, 32_768, 32_769])
def test_scores_export_at_the_edges_of_its_variants(N):
    import torch

    from paper_2510_02470_amd.binding import Sage

    rng = np.random.default_rng(N)
    V, G = rng.standard_normal((2, 8)).astype(np.float32), (0.3 + rng.standard_normal((N, 8))).astype(np.float32)
    s = Sage(4, 8)
    s.set_basis(torch.from_numpy(V).cuda())
    s.score(torch.from_numpy(G).cuda())
    idx = s.select(0.5).cpu().numpy()
    alpha = s.scores().cpu().numpy()
    z = G.astype(np.float64) @ V.T.astype(np.float64)
    z /= np.linalg.norm(z, axis=1, keepdims=True)
    u = z.sum(0)
    np.testing.assert_allclose(alpha, z @ (u / np.linalg.norm(u)), atol=2e-5)
    assert idx.tolist() == oracle.topm_f32(alpha, len(idx)).tolist()
    s.close()


def test_factored_and_unaligned_rows_in_turn():
    """A pass that takes factored rows (a basis of two parts) and row-major rows of an unaligned width (three parts) in turn:
    the images of the basis are made once each, and a new basis replaces both."""
    import torch

    from paper_2510_02470_amd.binding import Sage

    rng = np.random.default_rng(0)
    C, dh, n = 3, 128, 200
    D = C * (dh + 1)  # 387: rows start on no multiple of 16 bytes
    E, H, G = (torch.from_numpy(rng.standard_normal((n, w)).astype(np.float32)).cuda() for w in (C, dh, D))
    bases = [torch.from_numpy(rng.standard_normal((k, D)).astype(np.float32)).cuda() for k in (6, 6, 40)]

    def alone(V, outer):
        s = Sage(80, D)
        s.set_basis(V)
        s.score_outer(E, H) if outer else s.score(G)
        return s.zhat()

    s = Sage(80, D)
    for V in bases:
        want = torch.cat([alone(V, True), alone(V, False)] * 3)
        s.set_basis(V)
        s.score_outer(E, H)
        s.score(G)
        s.profile_enable(True)
        for _ in range(2):
            s.score_outer(E, H)
            s.score(G)
        assert s.profile_read()["rebuild"][1] == 0
        s.profile_enable(False)
        assert torch.equal(s.zhat(), want)
