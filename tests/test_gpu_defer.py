"""Shrinks whose rows are written later (csrc/fd_defer.hip) against Frequent Directions in 64 bits, for streams cut into calls in the
ways that take different paths through it."""
import pytest

pytestmark = pytest.mark.gpu

# Of |A|_F^2, for the covariance after some nine cycles, whose Gram entries are fp32 sums over slabs and whose rows are rounded to fp32 once
# for every rebuild. Such streams leave 1.2e-7 to 2.3e-7 (18 sizes, four cuts, three seeds each). With the third bf16 part of the
# coefficients or of the rows left out of the rebuild it would be 9e-7 to 2.6e-6 (a model in 64 bits, six sizes).
BAR = 4e-7


def _shrink(A, ell):
    import torch

    lam, Y = torch.linalg.eigh((A @ A.T).cpu())
    lam, Y = lam.flip(0)[:ell].to(A.device), Y.flip(1)[:, :ell].to(A.device)
    keep = (lam - lam[ell - 1]).clamp(min=0)
    w = torch.where(keep > 0, (keep / lam.clamp(min=1e-300)).sqrt(), torch.zeros_like(keep))
    return (w[:, None] * Y.T) @ A, float(lam[ell - 1])


def _sketch64(G, ell):
    """What is in the buffer after all rows: at least ell - 1 rows of a sketch and those that came after its last shrink."""
    import torch

    B, delta = G[:ell].double(), 0.0
    for lo in range(ell, len(G), ell):
        B = torch.cat([B, G[lo:lo + ell].double()])
        if len(B) == 2 * ell:
            B, d = _shrink(B, ell)
            delta += d
    return B, delta


def _cov_diff(A, B):
    """|A^T A - B^T B|_F without forming either: by the Gram matrix of all rows with signs."""
    import torch

    P = torch.cat([A, B])
    K = P @ P.T
    K[:, len(A):] *= -1.0
    return float((K @ K).trace().clamp(min=0).sqrt())


# 128, 256 and 512 buffer rows with and without padding, row types, widths that are a multiple of nothing; then both sides of the widths
# where a plan ends: one beside each eigensolve, or two at a time (bf16 at 512 buffer rows), or all at once
@pytest.mark.parametrize("ell,dtype,D", [(33, "f32", 701), (64, "f32", 5130), (64, "bf16", 2113), (65, "f32", 1300), (100, "bf16", 25447),
                                         (128, "f32", 3001), (129, "bf16", 1999), (200, "f32", 2050), (256, "bf16", 4097),
                                         (129, "bf16", 589_825), (129, "f32", 131_071), (200, "bf16", 262_145),
                                         (129, "f32", 98_304), (129, "f32", 98_305), (136, "bf16", 180_224), (136, "bf16", 180_225),
                                         (40, "f32", 196_608), (40, "f32", 196_609)])
def test_streams_in_calls_of_many_few_and_part_cycles(ell, dtype, D):
    """Against |A|_F^2, ||A||_F^2 itself and the covariance to BAR and the sum of the deltas to 5e-9, of which 1.3e-9 is the most (fp32 sums
    over D of squares of one sign are off by up to 2e-7, the deltas' errors are of either sign)."""
    import torch

    from paper_2510_02470_amd.binding import Sage

    g = torch.Generator(device="cuda").manual_seed(ell + D)
    N = 9 * ell + ell // 3
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    k = ell // 2
    signal = torch.randn((N, k), generator=g, device="cuda") * torch.arange(1, k + 1, device="cuda") ** -0.5
    G = (signal @ torch.randn((k, D), generator=g, device="cuda") + 0.1 * torch.randn((N, D), generator=g, device="cuda")).to(td)
    want, delta = _sketch64(G, ell)
    fro = float((G.double() ** 2).sum())
    cuts = {"one call": [N], "whole cycles": [ell] * 9 + [ell // 3], "calls of several": [4 * ell, 3 * ell, 2 * ell, ell // 3],
            "part cycles": [2 * ell + ell // 2, 3 * ell + 1, ell - 1, 2 * ell, N - 8 * ell - ell // 2]}
    for name, sizes in cuts.items():
        assert sum(sizes) == N
        s, lo = Sage(ell, D, dtype=dtype), 0
        for n in sizes:
            s.fd_update(G[lo:lo + n].contiguous())
            lo += n
        st = s.stats()
        assert st.rows_seen == N and st.n_unconverged == 0, name
        assert abs(st.frob2 - fro) <= BAR * fro and abs(st.sum_delta - delta) <= 5e-9 * fro, name
        assert _cov_diff(s.sketch().double(), want) <= BAR * fro, name
        s.close()


@pytest.mark.parametrize("ell,dtype,D,ring", [(20, "f32", 3001, 2), (64, "f32", 5130, 4), (256, "bf16", 270_000, 3)])
def test_contexts_where_memory_is_short(ell, dtype, D, ring):
    """Where the halves for rows ahead and deferred shrinks do not fit, a context does with those it needs and shrinks at once: the
    same covariance up to what rounding leaves (as above)."""
    import torch

    from paper_2510_02470_amd import binding

    L, lp = binding.lib(), max(32, 1 << (ell - 1).bit_length())
    half = (D + 15) // 16 * 16 * lp * 4
    held, refused = {}, []

    def take(size, stream, user):
        if size == ring * half:
            refused.append(size)
            return None
        t = torch.empty(size + 256, dtype=torch.uint8, device="cuda")
        p = (t.data_ptr() + 255) // 256 * 256
        held[p] = t
        return p

    def give(p, user):
        torch.cuda.synchronize()
        held.pop(p, None)

    fns = binding._ALLOC_FN(take), binding._FREE_FN(give)
    G = torch.randn((7 * ell + 3, D), device="cuda", generator=torch.Generator(device="cuda").manual_seed(D))
    G = G.to(torch.bfloat16 if dtype == "bf16" else torch.float32)
    out = []
    for short in (False, True):
        if short:
            L.sage_set_allocator(fns[0], fns[1], None)
        try:
            s = binding.Sage(ell, D, dtype=dtype)
            s.fd_update(G)
            s.fd_update(G[:2 * ell])
            out.append((s.sketch(), s.stats()))
            s.close()
        finally:
            if short:
                binding._torch_memory(L)
    assert refused and not held
    fro = out[0][1].frob2
    assert abs(out[1][1].frob2 - fro) <= BAR * fro and abs(out[1][1].sum_delta - out[0][1].sum_delta) <= BAR * fro
    assert _cov_diff(out[0][0].double(), out[1][0].double()) <= BAR * fro


@pytest.mark.parametrize("ell,dtype,D", [(64, "f32", 5130), (100, "bf16", 2113), (256, "bf16", 4097)])
def test_probe_of_a_matrix_leaves_a_pending_shrink_alone(ell, dtype, D):
    """A call of several cycles that ends on a full buffer has the Gram matrix of the pending shrink already; the eigensolve of another
    matrix (sage_probe_eig_matrix: "the sketch is not modified") must not take its place. The sketches differ by the Gram matrix formed
    anew, in other partial sums: bar as above."""
    import torch

    from paper_2510_02470_amd.binding import Sage

    g = torch.Generator(device="cuda").manual_seed(D)
    G = torch.randn((6 * ell, D), generator=g, device="cuda").to(torch.bfloat16 if dtype == "bf16" else torch.float32)
    n = 2 * max(32, 1 << (ell - 1).bit_length())
    X = torch.randn((n, n), generator=g, device="cuda", dtype=torch.float64)
    out = []
    for probe in (False, True):
        s = Sage(ell, D, dtype=dtype)
        s.fd_update(G)
        if probe:
            s.probe_eig_matrix(X @ X.T)
        out.append((s.sketch().double(), s.stats()))
        s.close()
    fro = out[0][1].frob2
    assert abs(out[1][1].frob2 - fro) <= BAR * fro and abs(out[1][1].sum_delta - out[0][1].sum_delta) <= BAR * fro
    assert _cov_diff(out[0][0], out[1][0]) <= BAR * fro


@pytest.mark.parametrize("ell,dtype,D", [(64, "f32", 1200), (128, "bf16", 1200), (256, "bf16", 1200), (256, "f32", 1200), (130, "bf16", 300_000)])
def test_eager_calls_between_replays_of_a_captured_one(ell, dtype, D):
    """A graph holds the halves that were in use when it was captured: eager calls of an even number of cycles leave the rows in them, as
    the captured call does. Against all calls made one by one, bar as above."""
    import torch

    from paper_2510_02470_amd.binding import Sage

    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator(device="cuda").manual_seed(ell)
    G = [torch.randn((n * ell, D), generator=g, device="cuda").to(td) for n in (2, 1, 2, 4, 2, 2, 2, 6, 2)]
    st = torch.cuda.Stream()
    st.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(st):
        eager, s = Sage(ell, D, dtype=dtype), Sage(ell, D, dtype=dtype)
        for c in (eager, s):
            c.fd_update(G[0])
            c.fd_update(G[1])          # ends on a full buffer, nothing stored ahead
        rows = G[2].clone()
        st.synchronize()
        graph = torch.cuda.CUDAGraph()
        graph.capture_begin(capture_error_mode="thread_local")
        s.fd_update(rows)
        graph.capture_end()
        for i, B in enumerate(G[2:]):
            if i % 2 == 0:
                rows.copy_(B)
                graph.replay()
            else:
                s.fd_update(B)
            eager.fd_update(B)
        st.synchronize()
        want, got = eager.sketch().double(), s.sketch().double()
        fro = eager.stats().frob2
        assert _cov_diff(want, got) <= BAR * fro


@pytest.mark.parametrize("ell,dtype,D,keep,halves,rest", [(20, "f32", 30_001, 1, 2, 3), (64, "f32", 51_300, 2, 4, 64), (64, "f32", 51_300, 2, 4, 0),
                                                          (100, "bf16", 20_003, 2, 4, 33), (256, "bf16", 400_000, 2, 3, 100)])
def test_contexts_where_memory_gets_short_later(ell, dtype, D, keep, halves, rest):
    """A context that was created with the halves for rows ahead and deferred shrinks gives them back when something else it needs does not
    fit, so that the job goes through in the memory it took without them: the same scores, and the same covariance after further rows (bar
    as above). rest = 0: against a basis of the caller's, with a shrink pending whose Gram matrix is there."""
    import torch

    from paper_2510_02470_amd import binding

    L, lp = binding.lib(), max(32, 1 << (ell - 1).bit_length())
    extra = (halves - keep) * ((D + 15) // 16 * 16 * lp * 4)
    held, limit, refused, peak = {}, [None], [], [0]

    def take(size, stream, user):
        used = sum(t.numel() for t in held.values())
        if limit[0] is not None and used + size > limit[0]:
            refused.append(size)
            return None
        peak[0] = max(peak[0], used + size)
        t = torch.empty(size + 256, dtype=torch.uint8, device="cuda")
        p = (t.data_ptr() + 255) // 256 * 256
        held[p] = t[:size]
        return p

    def give(p, user):
        torch.cuda.synchronize()
        held.pop(p, None)

    fns = binding._ALLOC_FN(take), binding._FREE_FN(give)
    N, k = 7 * ell + rest, ell // 2
    g = torch.Generator(device="cuda").manual_seed(D)
    G = (torch.randn((N, k), generator=g, device="cuda") @ torch.randn((k, D), generator=g, device="cuda")
         + 0.1 * torch.randn((N, D), generator=g, device="cuda")).to(torch.bfloat16 if dtype == "bf16" else torch.float32)
    out = []
    L.sage_set_allocator(fns[0], fns[1], None)
    try:
        for short in (False, True):
            s = binding.Sage(ell, D, dtype=dtype, max_rows=N)
            s.fd_update(G)
            if short:
                limit[0] = peak[0] - extra
            if rest:
                s.fd_basis(min(k, 128))
            else:
                s.set_basis(G[:k].float())
            s.score(G)
            s.select(0.1)
            alpha = s.scores()
            s.fd_update(G[:3 * ell])
            out.append((s.sketch().double(), s.stats(), alpha))
            s.close()
    finally:
        binding._torch_memory(L)
    assert refused and not held
    fro = out[0][1].frob2
    assert torch.equal(out[0][2], out[1][2])
    assert abs(out[1][1].frob2 - fro) <= BAR * fro and abs(out[1][1].sum_delta - out[0][1].sum_delta) <= BAR * fro
    assert _cov_diff(out[0][0], out[1][0]) <= BAR * fro


@pytest.mark.parametrize("refused,later,store,want", [((5,), 0, 0, [3]), ((5, 3), 0, 0, [2]), ((), 2, 2.5, [5, 3]), ((), 3, 2.5, [5, 3, 2]),
                                                      ((), 3, 0, [5, 2])])
def test_four_blocks_together_are_given_up_for_two_first(refused, later, store, want):
    """A wide bf16 context has a ring of five halves. Where those do not fit at its creation (refused), or something that a later call needs
    does not fit beside them (later: so many halves too few, and a score store of that many), it takes three and shrinks in pairs, and two
    only if three do not fit either. Against the usual context: the same covariance (bar as above), and other bits in the sketch than
    with any other plan."""
    import torch

    from paper_2510_02470_amd import binding

    ell, D = 129, 524_289
    L, half = binding.lib(), (D + 15) // 16 * 16 * 256 * 4
    held, limit, rings, peak, refuse = {}, [None], [], [0], [()]

    def take(size, stream, user):
        used = sum(t.numel() for t in held.values())
        if limit[0] is not None and used + size > limit[0] or size in [r * half for r in refuse[0]]:
            return None
        peak[0] = max(peak[0], used + size)
        t = torch.empty(size + 256, dtype=torch.uint8, device="cuda")
        p = (t.data_ptr() + 255) // 256 * 256
        held[p] = t[:size]
        if size in (2 * half, 3 * half, 4 * half, 5 * half):
            rings.append(size // half)
        return p

    def give(p, user):
        torch.cuda.synchronize()
        held.pop(p, None)

    fns = binding._ALLOC_FN(take), binding._FREE_FN(give)
    N = 6 * ell + 50
    G = torch.randn((N, D), device="cuda", generator=torch.Generator(device="cuda").manual_seed(1)).to(torch.bfloat16)
    out = []
    L.sage_set_allocator(fns[0], fns[1], None)
    try:
        for plan, short in (((), 0), (refused, later), ((5, 3), 0)):
            refuse[0], limit[0] = plan, None
            del rings[:]
            s = binding.Sage(ell, D, dtype="bf16", max_rows=max(N, int(store * half / 512)))
            s.fd_update(G[:3])
            if short:
                limit[0] = peak[0] - short * half
            s.fd_basis(64)
            s.score(G[:300])
            s.select(0.1)
            s.fd_update(G[3:])
            out.append((s.sketch().double(), s.stats(), list(rings)))
            s.close()
    finally:
        binding._torch_memory(L)
    assert not held
    (a, sa, ra), (b, sb, rb), (c, _, rc) = out
    assert ra == [5] and rb == want and rc == [2]
    assert abs(sb.frob2 - sa.frob2) <= BAR * sa.frob2 and abs(sb.sum_delta - sa.sum_delta) <= BAR * sa.frob2
    assert _cov_diff(a, b) <= BAR * sa.frob2
    assert not torch.equal(a, b) and torch.equal(b, c) == (want[-1] == 2)
