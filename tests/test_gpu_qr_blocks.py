"""The QR from fp64 Gram matrices (small rotations in one workgroup, larger ones by blocks of 256 columns) at the edges of its
tiles and blocks, against 64 bits."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2511_04063_amd import binding as B  # noqa: E402


def _latent(n, kind):
    g = torch.Generator(device="cuda")
    g.manual_seed(31 * n + len(kind))
    Z = torch.randn(n, n, generator=g, device="cuda", dtype=torch.float64)
    if kind == "rotation":       # a rotation as the start, moved by the steps since
        Z = torch.linalg.qr(Z)[0] + 0.3 / np.sqrt(n) * torch.randn(n, n, generator=g, device="cuda", dtype=torch.float64)
    elif kind == "lengths":      # columns of all lengths, 2^-40 to 2^40 among them
        Z *= torch.exp2(torch.linspace(-40, 40, n, device="cuda", dtype=torch.float64)[torch.randperm(n, generator=g, device="cuda")])
    elif kind == "parallel":     # columns of one block parallel to 1e-5: solved by substitution
        Z[:, n // 2 + 3] = Z[:, n // 2] + 1e-5 * torch.randn(n, generator=g, device="cuda", dtype=torch.float64)
    elif kind == "spanned":      # the last column nearly spanned by the first ones: the second pass has most of it to take off
        Z[:, n - 1] = Z[:, :40] @ torch.randn(40, generator=g, device="cuda", dtype=torch.float64) / 6.0 + 1e-5 * Z[:, n - 1]
    elif kind == "triangle":     # condition number 2^n and more, though no column cancels against another
        Z = torch.triu(Z)
        Z.diagonal().abs_().add_(0.5)
    elif kind == "decaying":     # condition number 1e7: blocks that the second pass finds ill-conditioned
        Q = torch.linalg.qr(Z)[0]
        Z = (Q * torch.logspace(0, -7, n, device="cuda", dtype=torch.float64)) @ torch.linalg.qr(Z.T.contiguous())[0]
    # what is singular, exactly or in fp32
    elif kind == "zero column":
        Z[:, n // 2 + 1] = 0.0
    elif kind == "every other zero":
        Z[:, ::2] = 0.0
    elif kind == "right half zero":
        Z[:, n // 2:] = 0.0
    elif kind == "all zero":
        Z.zero_()
    elif kind == "equal columns":
        Z[:, [n // 3, n - 2, n - 1]] = Z[:, [1]]
    elif kind == "all equal":
        Z.fill_(1.0)
    elif kind == "rank one":
        Z = Z[:, :1] @ Z[:1, :]
    elif kind == "half rank":
        Z = Z[:, :n // 2] @ Z[n // 2:, :][: n // 2]
    elif kind == "half the rows":      # the right half is spanned by the left one, and what rounding leaves of it is as well
        Z[n // 2:, :] = 0.0
    elif kind == "beyond":             # condition number 1e12
        Z = (torch.linalg.qr(Z)[0] * torch.logspace(0, -12, n, device="cuda", dtype=torch.float64)) @ torch.linalg.qr(Z.T.contiguous())[0]
    elif kind == "turned triangle":
        Z = torch.linalg.qr(Z.T.contiguous())[0] @ torch.triu(Z).contiguous()
    ld = -(-n // 4) * 4
    out = torch.full((n, ld), float("nan"), device="cuda")
    out[:, :n] = Z
    return out[:, :n]


def _padded(n):
    buf = torch.full((n, -(-n // 4) * 4 + 4), 7.0, device="cuda")
    return buf, buf[:, :n]


SINGULAR = ["zero column", "every other zero", "right half zero", "all zero", "equal columns", "all equal", "rank one", "half rank",
            "half the rows", "beyond", "turned triangle"]
KINDS = ["gauss", "rotation", "lengths", "parallel", "spanned", "triangle", "decaying"]


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("n", [129, 144, 191, 255, 256, 257, 272, 511, 513, 770])
def test_blocks_of_256_columns(n, kind):
    """Last blocks of 1 to 256 columns, full and cut 16- and 64-column tiles.  R^T R - I, R U - Z column by column and the form of
    U; the same bits whichever way the streams wait for each other, on one stream, call after call and without U; nothing
    written beside R and U.  Bars: an fp32 factor can be orthogonal and reproduce Z to some 2^-24 (measured up to 2.6e-7 and
    7e-7 over all kinds, LAPACK's fp32 QR 8e-7 and 1.2e-6)."""
    Z = _latent(n, kind)
    # what cancels strongly inside a block is reported
    inside = (kind == "parallel" and n // 2 // 256 == (n // 2 + 3) // 256) or (kind == "spanned" and n <= 256)
    first = None
    for device_sync, single in ((1, 0), (1, 0), (0, 0), (0, 1)):
        c = B.Context()
        try:
            c.ensure_workspace(1, n, 1, B.DQ_F32)
            c.dq_set_option(B.DQ_OPT_DEVICE_SYNC, device_sync)
            c.dq_set_option(B.DQ_OPT_SINGLE_STREAM, single)
            (Rb, R), (Ub, U) = _padded(n), _padded(n)
            c.dq_qr_orth(Z, R, U)
            R2 = torch.empty_like(Rb)[:, :n]
            c.dq_qr_orth(Z, R2, None)
            flags = c.dq_device_flags()
            if kind not in ("triangle", "decaying"):
                assert flags == (B.DQ_FLAG_ILLCOND_PANEL if inside else 0)
            assert flags & ~B.DQ_FLAG_ILLCOND_PANEL == 0
            assert torch.equal(R, R2) and torch.all(Rb[:, n:] == 7.0) and torch.all(Ub[:, n:] == 7.0)
            if first is None:
                first = (R.clone(), U.clone())
            assert torch.equal(R, first[0]) and torch.equal(U, first[1])
        finally:
            torch.cuda.synchronize()
            c.close()
    _check(Z, *first)


@pytest.mark.parametrize("kind", SINGULAR)
@pytest.mark.parametrize("n", [129, 200, 256, 257, 300, 513, 770])
def test_blocks_singular(n, kind):
    """R is a rotation and reproduces Z whatever Z's rank: columns that are zero, exactly or but for rounding in the span of others,
    in the same lot of 16, the same block and other ones, in the last, cut lot, all of them.  The same bits with one stream, call after
    call and without U; a column that is zero from the start raises DQ_FLAG_SINGULAR."""
    _singular(n, kind)


@pytest.mark.parametrize("n,kind", [(1536, "decaying"), (1536, "all equal"), (2064, "half the rows"), (2064, "rank one"), (4112, "zero column"),
                                    (4112, "parallel"), (4112, "beyond")])
def test_large_singular(n, kind):
    """The same where a workgroup of the finish has more than one strip of 16 rows, and of the solve two."""
    _singular(n, kind)


@pytest.mark.parametrize("n", [100, 129, 300, 770])
def test_lengths_at_the_ends_of_the_range(n):
    """Columns of all lengths from 2^-101 to 2^118 give R and U as ordinary ones do, without a flag; shorter ones count as zeros and longer
    ones are reported, alone and among others (n > 128; smaller rotations take any whose U is finite).  What the products on split
    operands lose of an entry, 2^-134, is some 2^-30 of such a column: no more than the bars of ordinary ones."""
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    base = torch.linalg.qr(torch.randn(n, n, generator=g, device="cuda", dtype=torch.float64))[0]
    base = base + 0.3 / np.sqrt(n) * torch.randn(n, n, generator=g, device="cuda", dtype=torch.float64)
    base = base / base.norm(dim=0)
    spread = torch.exp2(torch.linspace(-101, 118, n, device="cuda", dtype=torch.float64)[torch.randperm(n, generator=g, device="cuda")])
    one = torch.ones(n, device="cuda", dtype=torch.float64)
    short, long = one.clone(), one.clone()
    short[n // 3], long[n // 3] = 2.0 ** -104, 2.0 ** 121
    big = n > 128
    c = B.Context()
    try:
        c.ensure_workspace(1, n, 1, B.DQ_F32)
        for lengths, flags in ((spread, 0), (one * 2.0 ** -101, 0), (one * 2.0 ** 118, 0), (short, B.DQ_FLAG_SINGULAR if big else 0),
                               (one * 2.0 ** -104, B.DQ_FLAG_SINGULAR if big else 0), (long, B.DQ_FLAG_NONFINITE if big else 0)):
            _, Z = _padded(n)
            Z.copy_(base * lengths)
            R, U = (_padded(n)[1] for _ in range(2))
            c.dq_qr_orth(Z, R, U)
            assert c.dq_device_flags() & ~B.DQ_FLAG_ILLCOND_PANEL == flags
            if flags == B.DQ_FLAG_NONFINITE:
                continue
            kept = torch.where(lengths >= 2.0 ** -102, lengths, 0.0) if big else lengths
            scale = torch.where(kept > 0, 1.0 / lengths, 1.0)      # columns at unit length
            _check((base * kept).float().double() * scale, R, U.double() * scale, singular=True)
    finally:
        torch.cuda.synchronize()
        c.close()


def _singular(n, kind):
    Z = _latent(n, kind)
    first = None
    for single in (0, 0, 1):
        c = B.Context()
        try:
            c.ensure_workspace(1, n, 1, B.DQ_F32)
            c.dq_set_option(B.DQ_OPT_SINGLE_STREAM, single)
            (Rb, R), (Ub, U) = _padded(n), _padded(n)
            R2 = torch.empty_like(Rb)[:, :n]
            c.dq_qr_orth(Z, R, U)
            c.dq_qr_orth(Z, R2, None)
            flags = c.dq_device_flags()
            assert flags & ~(B.DQ_FLAG_ILLCOND_PANEL | B.DQ_FLAG_SINGULAR) == 0
            assert flags & B.DQ_FLAG_SINGULAR or "zero" not in kind
            assert torch.equal(R, R2) and torch.all(Rb[:, n:] == 7.0) and torch.all(Ub[:, n:] == 7.0)
            if first is None:
                first = (R.clone(), U.clone())
            assert torch.equal(R, first[0]) and torch.equal(U, first[1])
        finally:
            torch.cuda.synchronize()
            c.close()
    _check(Z, *first, singular=True)


def _check(Z, R, U, singular=False):
    n = Z.shape[0]
    R, U, Z = R.double(), U.double(), Z.double()
    assert float((R.T.contiguous() @ R - torch.eye(n, device="cuda", dtype=torch.float64)).abs().max()) < 1e-6
    length = Z.norm(dim=0)
    res = (R @ U - Z).norm(dim=0) / torch.where(length > 0, length, 1.0)
    assert float(res.max()) < 2e-6
    assert int(torch.count_nonzero(torch.tril(U, -1))) == 0
    assert bool((U.diagonal() >= 0).all()) if singular else bool((U.diagonal() > 0).all())


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("n", [2, 16, 33, 64, 65, 80, 95, 100, 113, 128])
def test_small_rotations(n, kind):
    """One workgroup a latent: tiles cut short, 64 x 64 blocks of 1 to 64 columns, a second pass that is not needed, is by a few terms, by
    another factorisation, and column by column; several latents in one launch, one alone, without U."""
    if (n < 41 and kind == "spanned") or (n < 6 and kind == "parallel"):
        pytest.skip("fewer columns than the kind speaks of")
    c = B.Context()
    try:
        c.ensure_workspace(4, n, 1, B.DQ_F32)
        ld = -(-n // 4) * 4 + 4
        Z, R, U, R1 = (torch.full((4, n, ld), 7.0, device="cuda") for _ in range(4))
        for i, k in enumerate((kind, "gauss", "rotation", kind)):
            Z[i, :, :n] = _latent(n, k)
        c.dq_qr_orth(Z[..., :n], R[..., :n], U[..., :n])
        c.dq_qr_orth(Z[3:, :, :n], R1[3:, :, :n], None)
        assert torch.equal(R[0], R[3]) and torch.equal(U[0], U[3]) and torch.equal(R1[3], R[3])
        assert torch.all(R[..., n:] == 7.0) and torch.all(U[..., n:] == 7.0)
        for i in range(3):
            _check(Z[i, :, :n], R[i, :, :n], U[i, :, :n])
        assert c.dq_device_flags() == 0
    finally:
        torch.cuda.synchronize()
        c.close()


@pytest.mark.parametrize("kind", SINGULAR)
@pytest.mark.parametrize("n", [3, 17, 64, 70, 96, 101, 128])
def test_small_singular(n, kind):
    """R is a rotation and reproduces Z whatever Z's rank, the neighbours in the launch as well; a column that is zero from the
    start raises DQ_FLAG_SINGULAR, and nothing else is ever raised.  Also scaled far down and up."""
    c = B.Context()
    try:
        c.ensure_workspace(3, n, 1, B.DQ_F32)
        ld = -(-n // 4) * 4
        for scale in (1.0, 2.0 ** -90, 2.0 ** 110):
            Z, R, U = (torch.full((3, n, ld), 7.0, device="cuda") for _ in range(3))
            for i, k in enumerate(("gauss", kind, "rotation")):
                Z[i, :, :n] = _latent(n, k) * scale
            c.dq_qr_orth(Z[..., :n], R[..., :n], U[..., :n])
            flags = c.dq_device_flags()
            for i in range(3):
                _check(Z[i, :, :n] / scale, R[i, :, :n], U[i, :, :n] / scale, singular=i == 1)
            assert flags & ~B.DQ_FLAG_SINGULAR == 0
            if "zero" in kind:
                assert flags == B.DQ_FLAG_SINGULAR
    finally:
        torch.cuda.synchronize()
        c.close()


@pytest.mark.parametrize("n", [64, 80, 96, 112, 128])
def test_small_rotated_triangles(n):
    """Triangles times a rotation, diagonals from 0.4 to 1.4: R of the first factor is off by anything from rounding to all of it, so
    that some latents lie on either side of each line between finished, corrected, factored again and taken column by column."""
    b = 64
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    Z = torch.triu(torch.randn(b, n, n, generator=g, device="cuda", dtype=torch.float64))
    Z.diagonal(dim1=1, dim2=2).abs_().add_(torch.linspace(0.4, 1.4, b, device="cuda", dtype=torch.float64)[:, None])
    Z = (torch.linalg.qr(torch.randn(b, n, n, generator=g, device="cuda", dtype=torch.float64))[0].contiguous() @ Z.contiguous()).float()
    c = B.Context()
    try:
        c.ensure_workspace(b, n, 1, B.DQ_F32)
        R, U = torch.empty_like(Z), torch.empty_like(Z)
        c.dq_qr_orth(Z, R, U)
        for i in range(b):
            _check(Z[i], R[i], U[i])
        assert c.dq_device_flags() == 0
    finally:
        torch.cuda.synchronize()
        c.close()


@pytest.mark.parametrize("kinds", [("gauss", "rotation", "lengths", "gauss"),
                                   ("gauss", "zero column", "turned triangle", "rotation", "half the rows", "turned triangle")],
                         ids=["ordinary", "singular"])
@pytest.mark.parametrize("n", [300, 770])
def test_blocks_under_capture(n, kinds):
    """The same launches recorded into a graph, in a context that has met its stream before and in one that has not: every replay, on
    other latents and with eager calls in between, gives the eager call's bits.  Also where what is done differs from replay to replay: by
    blocks, 16 columns at a time, with a finish."""
    latents = [_latent(n, k) for k in kinds]
    for met in (True, False):
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            c, e = B.Context(s), B.Context(s)
            Z, R, U, Re, Ue = (_padded(n)[1] for _ in range(5))
            Z.copy_(latents[0])
            try:
                for x in (c, e):
                    x.ensure_workspace(1, n, 1, B.DQ_F32)
                if met:
                    c.dq_qr_orth(Z, R, U)
                s.synchronize()
                graph = torch.cuda.CUDAGraph()
                with torch.cuda.graph(graph, stream=s):
                    c.dq_qr_orth(Z, R, U)
                for Zi in latents:
                    Z.copy_(Zi)
                    graph.replay()
                    e.dq_qr_orth(Zi, Re, Ue)
                    s.synchronize()
                    assert torch.equal(R, Re) and torch.equal(U, Ue)
                flags = c.dq_device_flags()
                assert flags == (B.DQ_FLAG_SINGULAR | B.DQ_FLAG_ILLCOND_PANEL if "zero column" in kinds else 0)
            finally:
                s.synchronize()
                c.close()
                e.close()


@pytest.mark.parametrize("n", [300, 1100])
def test_singular_latents_on_several_streams(n):
    """Four contexts on streams of their own factor latents whose workgroups wait for each other, all at the same time: the bits that
    each gives alone, and no wait that ran into its limit."""
    kinds = ("turned triangle", "zero column", "half rank", "beyond")
    latents = [_latent(n, k) for k in kinds]
    streams = [torch.cuda.Stream() for _ in kinds]
    contexts, want, got = [], [], []
    try:
        for Z, s in zip(latents, streams):
            with torch.cuda.stream(s):
                c = B.Context(s)
                c.ensure_workspace(1, n, 1, B.DQ_F32)
                contexts.append(c)
                R, U = _padded(n)[1], _padded(n)[1]
                c.dq_qr_orth(Z, R, U)
                got.append((_padded(n)[1], _padded(n)[1]))
            torch.cuda.synchronize()
            want.append((R, U))
        for _ in range(3):
            for Z, s, c, (R, U) in zip(latents, streams, contexts, got):
                with torch.cuda.stream(s):
                    c.dq_qr_orth(Z, R, U)
        torch.cuda.synchronize()
        for c, (R, U), (Rw, Uw) in zip(contexts, got, want):
            assert c.dq_device_flags() & B.DQ_FLAG_SYNC_TIMEOUT == 0
            assert torch.equal(R, Rw) and torch.equal(U, Uw)
    finally:
        torch.cuda.synchronize()
        for c in contexts:
            c.close()


@pytest.mark.parametrize("value", [float("nan"), float("inf")])
@pytest.mark.parametrize("n", [100, 300, 1100])
def test_latents_that_are_not_finite(n, value):
    """One such entry is reported and nothing else is, wherever it lies, also where columns are zero or parallel and workgroups wait for
    each other; the context's next latent is factored as ever."""
    c = B.Context()
    try:
        c.ensure_workspace(1, n, 1, B.DQ_F32)
        good = _latent(n, "gauss")
        for kind in ("gauss", "parallel", "zero column"):
            for row, col in ((0, 0), (n // 2, n // 2), (n - 1, n - 1)):
                Z = _latent(n, kind)
                Z[row, col] = value
                R, U = (_padded(n)[1] for _ in range(2))
                c.dq_qr_orth(Z, R, U)
                flags = c.dq_device_flags()
                assert flags & B.DQ_FLAG_NONFINITE
                assert flags & ~(B.DQ_FLAG_NONFINITE | B.DQ_FLAG_SINGULAR | B.DQ_FLAG_ILLCOND_PANEL) == 0
        c.dq_qr_orth(good, R, U)
        assert c.dq_device_flags() == 0
        _check(good, R, U)
    finally:
        torch.cuda.synchronize()
        c.close()
