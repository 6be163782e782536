"""The direct eigensolve (tridiagonal reduction, divide and conquer) at every padded size, on spectra that exercise its
branches: deflation of every kind, equal poles across a merge, ranks far below the size, scales far from one."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _matrices(n):
    rng = np.random.default_rng(n)
    Q, _ = np.linalg.qr(rng.standard_normal((n, n)))
    h = n // 8
    A = rng.standard_normal((n, 700)) * np.exp(rng.standard_normal((n, 1)))
    lap = np.diag(np.full(n, 2.0)) - np.diag(np.ones(n - 1), 1) - np.diag(np.ones(n - 1), -1)
    top = np.sort(rng.random(n // 2))[::-1]
    X = 0.1 * rng.standard_normal((n // 2, n))
    cross = np.zeros((n, n))
    cross[: n // 2, : n // 2] = np.diag(top)
    cross[n // 2:, n // 2:] = X @ X.T
    cross[n // 2:, : n // 2] = 0.1 * rng.standard_normal((n // 2, n // 2)) * np.sqrt(top)
    cross = np.tril(cross) + np.tril(cross, -1).T
    spec = {
        "clustered": np.concatenate([np.full(2 * h, 1.0), 1 + 1e-9 * np.arange(3 * h), np.linspace(0.5, 1e-8, n - 5 * h)]),
        "rank8": np.concatenate([np.linspace(3, 1, 8), np.zeros(n - 8)]),
        "graded": 10.0 ** (-np.arange(n) / 8.0),
        "signal_and_noise": np.concatenate([1.0 / np.arange(1, n // 4 + 1), 1e-4 * np.exp(rng.standard_normal(n - n // 4))]),
    }
    out = {k: (Q * v) @ Q.T for k, v in spec.items()}
    out.update(gram=A @ A.T, tiny=(A @ A.T) * 1e-60, huge=(A @ A.T) * 1e60, zero=np.zeros((n, n)), diagonal=np.diag(rng.random(n)),
               ones=np.ones((n, n)), laplace=lap, identity=np.eye(n), blocks=np.kron(np.eye(n // 32), A[:32] @ A[:32].T),
               after_a_shrink=cross)
    return out


@pytest.mark.parametrize("ell", [32, 64, 128, 256])
def test_eigensolve_at_every_padded_size(ell):
    import torch

    from paper_2510_02470_amd.binding import Sage

    s, n = Sage(ell, 64), 2 * ell
    for name, C in _matrices(n).items():
        C = (C + C.T) / 2
        Y, lam, _ = s.probe_eig_matrix(torch.from_numpy(C).cuda())
        Y, lam = Y.cpu().numpy(), lam.cpu().numpy()
        scale = max(np.abs(C).max(), 1e-300) * n
        assert np.abs(Y.T @ Y - np.eye(n)).max() <= 1e-13, name
        assert np.abs((Y * lam) @ Y.T - C).max() <= 1e-14 * scale, name
        assert np.abs(np.sort(lam) - np.linalg.eigvalsh(C)).max() <= 1e-14 * scale, name


@pytest.mark.parametrize("m", [4, 8, 16])
@pytest.mark.parametrize("ell", [32, 64, 256])
def test_small_merges_of_different_kinds_side_by_side(ell, m):
    """Merges of 4, 8 and 16 rows share a wave: those that rotate equal poles together (a segment with one value on its diagonal and one
    beside it: its halves have the same poles), those without survivors (nothing beside the diagonal) and ordinary ones, in every
    order. The reduction leaves a tridiagonal matrix one. Bars as above."""
    import torch

    from paper_2510_02470_amd.binding import Sage

    n = 2 * ell
    rng = np.random.default_rng(n + m)
    s = Sage(ell, 64)
    for joined in (False, True):
        d, e = 10.0 + rng.standard_normal(n), rng.standard_normal(n - 1)
        for j in range(n // m):
            kind, lo = rng.integers(3), j * m
            if kind < 2:
                d[lo:lo + m] = 10.0
                e[lo:lo + m - 1] = kind
            if not joined and lo:
                e[lo - 1] = 0.0
        C = np.diag(d) + np.diag(e, 1) + np.diag(e, -1)
        Y, lam, _ = s.probe_eig_matrix(torch.from_numpy(C).cuda())
        Y, lam = Y.cpu().numpy(), lam.cpu().numpy()
        scale = np.abs(C).max() * n
        assert np.abs(Y.T @ Y - np.eye(n)).max() <= 1e-13
        assert np.abs((Y * lam) @ Y.T - C).max() <= 1e-14 * scale
        assert np.abs(np.sort(lam) - np.linalg.eigvalsh(C)).max() <= 1e-14 * scale
    s.close()


def test_contexts_in_several_streams_share_the_gpu():
    """More contexts than XCDs, each on a stream of its own with work in flight at the same time: the reductions that keep
    work-groups of one XCD in step must not starve each other."""
    import torch

    from paper_2510_02470_amd.binding import Sage

    g = torch.Generator(device="cuda").manual_seed(3)
    G = torch.randn((256 * 5, 900), generator=g, device="cuda")
    ref = Sage(256, 900)
    ref.fd_update(G)
    want = ref.sketch()
    streams = [torch.cuda.Stream() for _ in range(18)]
    torch.cuda.synchronize()
    ctx = []
    for st in streams:
        with torch.cuda.stream(st):
            ctx.append(Sage(256, 900))
    for lo in range(0, G.shape[0], 256):
        for st, c in zip(streams, ctx):
            with torch.cuda.stream(st):
                c.fd_update(G[lo:lo + 256])
    for st, c in zip(streams, ctx):
        with torch.cuda.stream(st):
            got = c.sketch()
            st.synchronize()
        # one call or five: the same rows, the last bits of the Gram blocks may differ
        assert torch.allclose(got.T @ got, want.T @ want, rtol=0, atol=1e-5 * float((want.T @ want).abs().max()))
        assert c.stats().n_unconverged == 0    # (nobody had to wait for work-groups that could not run beside another's)
        c.close()


def test_a_context_joins_an_xcd_whose_reductions_are_in_flight():
    """Eight contexts, one an XCD, have many solves enqueued when eight more are created and start theirs: each of those
    comes after what is in flight on its XCD, and no solve is held up until it is given up."""
    import torch

    from paper_2510_02470_amd.binding import Sage

    g = torch.Generator(device="cuda").manual_seed(5)
    G = torch.randn((256 * 12, 600), generator=g, device="cuda")
    torch.cuda.synchronize()
    st = [torch.cuda.Stream() for _ in range(16)]
    ctx = []
    for i, t in enumerate(st):
        with torch.cuda.stream(t):
            ctx.append(Sage(256, 600))
            if i < 8:
                ctx[i].fd_update(G)
    for t, c in zip(st[8:], ctx[8:]):
        with torch.cuda.stream(t):
            c.fd_update(G)
    want = None
    for t, c in zip(st, ctx):
        with torch.cuda.stream(t):
            B = c.sketch()
            assert c.stats().n_unconverged == 0
            want = B if want is None else want
            assert torch.equal(B, want)
            c.close()


@pytest.mark.parametrize("ell,rows", [(ell, rows) for ell in (64, 128, 256) for rows in (1, 2, 5, 20, 60, 70, 131, 259)
                                      if rows < 2 * ell])
def test_basis_of_a_buffer_with_few_rows(ell, rows):
    """A basis taken early: the reduction runs on the rows in use, so most of its work-groups have no column or leave it
    before the end. Orthonormal to 1e-5, invariant under the rows' covariance and with all of its energy to 1e-6 (fp32 Gram)."""
    import torch

    from paper_2510_02470_amd.binding import Sage

    D = 700
    G = np.random.default_rng(rows).standard_normal((rows, D)).astype(np.float32) * np.exp(np.linspace(0, -3, rows))[:, None].astype(np.float32)
    s = Sage(ell, D)
    s.fd_update(torch.from_numpy(G).cuda())
    k = min(rows, ell - 1, 128)
    s.fd_basis(k)
    V = s.basis().cpu().numpy().astype(np.float64)
    A = G.astype(np.float64)
    fro, sig2 = (A ** 2).sum(), np.linalg.svd(A, compute_uv=False)[:k] ** 2
    AV = A @ V.T
    H = AV.T @ AV
    assert np.abs(V @ V.T - np.eye(k)).max() <= 1e-5
    assert np.abs(np.diag(H) - sig2).max() <= 1e-6 * fro
    assert np.linalg.norm(A.T @ AV - V.T @ H, 2) <= 1e-6 * fro
    assert abs(s.stats().frob2 - fro) <= 1e-6 * fro


@pytest.mark.parametrize("ell", [64, 128, 256])
def test_solves_beside_other_work_on_the_gpu(ell):
    """A stream of copies and one of matrix products keep CUs of every XCD busy while a context works: same bits as alone."""
    import torch

    from paper_2510_02470_amd.binding import Sage

    g = torch.Generator(device="cuda").manual_seed(ell)
    G = torch.randn((ell * 7 + 3, 1500), generator=g, device="cuda")

    def stream_of_rows(s):
        s.fd_update(G[:20])
        s.fd_basis(4)                      # an early basis: few rows
        for lo in range(20, G.shape[0], 3 * ell):
            s.fd_update(G[lo:lo + 3 * ell])
        s.fd_basis(ell // 2)

    alone = Sage(ell, 1500)
    stream_of_rows(alone)
    want, basis = alone.sketch(), alone.basis()
    src, dst = (torch.ones(1 << 26, device="cuda") for _ in range(2))
    a = torch.randn((2048, 2048), generator=g, device="cuda")
    torch.cuda.synchronize()
    st = [torch.cuda.Stream() for _ in range(2)]
    busy = Sage(ell, 1500)
    for _ in range(40):
        with torch.cuda.stream(st[0]):
            dst.copy_(src)
        with torch.cuda.stream(st[1]):
            a @ a
    stream_of_rows(busy)
    assert torch.equal(busy.sketch(), want) and torch.equal(busy.basis(), basis)
    torch.cuda.synchronize()
    assert busy.stats().n_unconverged == 0


@pytest.mark.parametrize("how", [1, 2, 3])
@pytest.mark.parametrize("ell", [64, 128, 256])
def test_solves_that_their_work_groups_cannot_do_together(ell, how):
    """1: the work-groups of the reduction give each other up after one look, as they do after a long wait where other work keeps
    them from running together, and one repeats the solve. 2: one does it from the start (at ell = 64 a kernel of its own), as
    where they cannot be placed on one XCD. 3: none is on the XCD it is expected on. Every solve succeeds, to the bars of the usual way."""
    import torch

    from paper_2510_02470_amd.binding import Sage

    s, n = Sage(ell, 64), 2 * ell
    s.debug_impatient_solves(how)
    solves = 0
    for name, C in _matrices(n).items():
        C = (C + C.T) / 2
        Y, lam, _ = s.probe_eig_matrix(torch.from_numpy(C).cuda())
        Y, lam = Y.cpu().numpy(), lam.cpu().numpy()
        solves += 1
        scale = max(np.abs(C).max(), 1e-300) * n
        assert np.abs(Y.T @ Y - np.eye(n)).max() <= 1e-13, name
        assert np.abs((Y * lam) @ Y.T - C).max() <= 1e-14 * scale, name
        assert np.abs(np.sort(lam) - np.linalg.eigvalsh(C)).max() <= 1e-14 * scale, name
    counted = 0 if (ell, how) == (64, 2) else solves
    assert s.stats().n_unconverged == counted
    s.debug_impatient_solves(0)
    s.probe_eig_matrix(torch.eye(n, dtype=torch.float64, device="cuda"))
    assert s.stats().n_unconverged == counted

    # a whole round, with few rows first; the usual way for comparison
    g = torch.Generator(device="cuda").manual_seed(ell)
    G = torch.randn((ell * 4 + 3, 900), generator=g, device="cuda") * torch.linspace(1, 0.1, 900, device="cuda")
    out = []
    for impatient in (0, how):
        c = Sage(ell, 900)
        c.debug_impatient_solves(impatient)
        for rows in (1, 2, 5, 19, ell):
            c.fd_update(G[:rows])
            c.fd_basis(1)
        c.fd_update(G)
        c.fd_basis(8)
        c.score(G)
        idx = c.select(0.1)
        assert (c.stats().n_unconverged > 0) == (impatient > 0 and counted > 0)
        B = c.sketch().double()
        out.append((B.T @ B, c.scores(), idx, c.stats().sum_delta))
    top = float(out[0][0].abs().max())
    assert float((out[0][0] - out[1][0]).abs().max()) <= 1e-6 * top
    assert abs(out[0][3] - out[1][3]) <= 1e-9 * out[0][3]
    assert float((out[0][1] - out[1][1]).abs().max()) <= 1e-4


@pytest.mark.parametrize("ell,dtype", [(32, "f32"), (64, "f32"), (128, "bf16"), (256, "bf16")])
def test_captured_update_replays(ell, dtype):
    """Two cycles of a stream captured in a graph and replayed with new rows, other work of the program between the
    replays: the sketch of the same calls made one by one. (Not bit for bit: a replay forms the Gram block of its first rows
    itself, in other partial sums than the eager call that had it formed ahead. Ten cycles with up to 8 roundings of 2^-24 each
    in a sum stay below 1e-5 of the largest entry.)"""
    import torch

    from paper_2510_02470_amd.binding import Sage

    D, td = 1200, torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator(device="cuda").manual_seed(ell)
    G = [torch.randn((n * ell, D), generator=g, device="cuda").to(td) for n in (2, 1, 2, 2, 2, 2, 2)]
    st = torch.cuda.Stream()
    st.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(st):
        eager, s = Sage(ell, D, dtype=dtype), Sage(ell, D, dtype=dtype)
        for c in (eager, s):
            c.fd_update(G[0])
            c.fd_update(G[1])          # ends on a full buffer, nothing stored ahead: where the captured call begins and ends
        rows = G[2].clone()
        st.synchronize()
        graph = torch.cuda.CUDAGraph()
        graph.capture_begin(capture_error_mode="thread_local")
        s.fd_update(rows)
        graph.capture_end()
        for B in G[2:]:
            rows.copy_(B)
            graph.replay()
            eager.fd_update(B)
            a = torch.randn((512, 512), device="cuda")
            (a @ a).sum().item()
        st.synchronize()
        want, got = eager.sketch().double(), s.sketch().double()
        want, got = want.T @ want, got.T @ got
        assert float((got - want).abs().max()) <= 1e-5 * float(want.abs().max())
        assert eager.stats().n_unconverged == 0 and s.stats().n_unconverged == 0


@pytest.mark.parametrize("ell,rows", [(64, 64), (64, 65), (64, 66), (64, 127), (128, 64), (128, 65), (128, 129), (128, 194),
                                      (256, 65), (256, 128), (256, 321), (256, 449), (256, 450), (256, 511)])
def test_basis_where_the_reduction_ends_near_a_multiple_of_64_rows(ell, rows):
    """The reduction's loop is written out per 64 steps: it ends just before, at and just after such a boundary."""
    test_basis_of_a_buffer_with_few_rows(ell, rows)


@pytest.mark.parametrize("rows", [1, 2, 3, 15, 16, 17, 18, 31, 32, 33, 34, 47, 48, 49, 63])
def test_basis_where_one_work_group_reduces(rows):
    """64 rows: the loop is written out per 16 steps."""
    test_basis_of_a_buffer_with_few_rows(32, rows)
