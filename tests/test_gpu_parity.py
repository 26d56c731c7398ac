"""GPU parity: the HIP path (through the C ABI) against the CPU FP64 oracle.

Every block of L and of the selected inverse must match the oracle within
1e-10 relative Frobenius error; strict upper triangles of the diagonal
factor blocks must be exact zeros; symmetric outputs exactly symmetric.
"""
import ctypes

import numpy as np
import pytest

import oracle
from paper_2503_17528_amd import synth
from tests.gpu_util import TOL, errs, say, to_dev, to_np

pytestmark = pytest.mark.gpu

# (n, b, a): ragged tiles, a = 0, n = 1, a wider than one tile, several tiles
SHAPES = [
    (1, 3, 0), (1, 64, 4), (2, 5, 1), (3, 64, 0), (4, 100, 3), (2, 130, 70),
    (16, 64, 4), (5, 192, 6), (3, 257, 2), (6, 128, 0), (2, 64, 64), (1, 200, 17),
    # arrow tip wider than the diagonal blocks (the paper's b = 1024, a = 256 ratio and beyond)
    (4, 128, 256), (3, 96, 257),
]


@pytest.fixture(scope="module")
def torch_cuda():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2503_17528_amd import bta

    bta.lib()  # raises if the library is missing: never a silent fallback
    return torch


def _run(torch, Q, inplace=False):
    from paper_2503_17528_amd import bta

    D, B, R, T = to_dev(Q)
    if inplace:
        L = bta.factor(D, B, R, T, out=(D, B, R, T))
        X = bta.selinv(*L[:4], out=L[:4])
    else:
        L = bta.factor(D, B, R, T)
        X = bta.selinv(*L[:4])
    torch.cuda.synchronize()
    return to_np(L[:4]), int(L[4].item()), to_np(X)


def _check(Lg, Xg, F, Xo, n, b, a):
    eL = errs(dict(zip("DBRT", Lg)), {"D": F["LD"], "B": F["LB"], "R": F["LR"], "T": F["LT"]})
    eX = errs(dict(zip("DBRT", Xg)), {"D": Xo["XD"], "B": Xo["XB"], "R": Xo["XR"], "T": Xo["XT"]}, lower=())
    say(f"   L err {eL}\n   X err {eX}")
    assert max(eL.values()) < TOL, eL
    assert max(eX.values()) < TOL, eX
    for i in range(n):
        assert np.all(np.triu(Lg[0][i], 1) == 0.0)
        assert np.array_equal(Xg[0][i], Xg[0][i].T)
    if a:
        assert np.all(np.triu(Lg[3], 1) == 0.0)
        assert np.array_equal(Xg[3], Xg[3].T)


@pytest.mark.parametrize("n,b,a", SHAPES)
def test_factor_selinv_parity(torch_cuda, n, b, a):
    say(f"case factor+selinv n={n} b={b} a={a}")
    wl = synth.workload(n, b, a)
    Q = synth.make_np(wl, 3)
    F = oracle.pobtaf(Q["D"], Q["B"], Q["R"], Q["T"])
    Xo = oracle.pobtasi(F["LD"], F["LB"], F["LR"], F["LT"])
    Lg, info, Xg = _run(torch_cuda, Q)
    assert info == 0
    _check(Lg, Xg, F, Xo, n, b, a)


@pytest.mark.parametrize("n,b,a", [(1, 1, 1), (2, 63, 1), (2, 65, 3), (2, 127, 65), (3, 129, 0), (2, 191, 129), (2, 128, 129),
                                   (3, 320, 1)])
def test_odd_extents(torch_cuda, n, b, a):
    """Odd b or a: the 4-byte operand loads (and, for an even b with an odd tip
    of one tile, the 16-byte ones), at the edges of the 64-tiles."""
    test_factor_selinv_parity(torch_cuda, n, b, a)


@pytest.mark.parametrize("n,b,a", [(2, 31, 33), (5, 32, 2), (4, 96, 32), (3, 766, 4), (3, 768, 2), (3, 769, 65), (2, 1088, 130),
                                   (2, 1087, 3)])
def test_sweep_tiles(torch_cuda, n, b, a):
    """The persistent backward sweep at the edges of its 32- and 64-tiles, with
    16- and 4-byte operand loads, out of place and in place."""
    test_factor_selinv_parity(torch_cuda, n, b, a)
    from paper_2503_17528_amd import bta

    Q = synth.make_np(synth.workload(n, b, a), 3)
    L = bta.factor(*to_dev(Q))[:4]
    X = bta.selinv(*L)
    Y = bta.selinv(*L, out=L)  # in place
    for x, y in zip(X, Y):
        assert torch_cuda.equal(x, y)


# blocks that the persistent sweep takes (ragged, odd, split-k, wide tips), the first sizes it does not, one block
@pytest.mark.parametrize("n,b,a", [(7, 33, 2), (7, 130, 70), (8, 520, 4), (6, 641, 3), (6, 768, 130), (6, 1024, 0), (6, 1087, 2),
                                   (3, 1089, 3), (3, 1282, 4), (1, 1500, 4), (1, 512, 700)])
def test_selinv_product_by_product(torch_cuda, n, b, a):
    """The selected inversion with the least workspace (the sweep product by
    product on several streams), out of place, twice, and in place: against the
    oracle, and the same bits each time."""
    from paper_2503_17528_amd import bta

    say(f"case selinv least workspace n={n} b={b} a={a}")
    wl = synth.workload(n, b, a, "literal" if b <= 512 else "scaled")
    Q = synth.make_np(wl, 6)
    F = oracle.pobtaf(Q["D"], Q["B"], Q["R"], Q["T"])
    Xo = oracle.pobtasi(F["LD"], F["LB"], F["LR"], F["LT"])
    L = to_dev({k: F["L" + k] for k in "DBRT"})
    work = torch_cuda.empty(bta.bta_workspace_min_bytes(bta.BTA_OP_SELINV, n, b, a), dtype=torch_cuda.uint8, device="cuda")
    X = bta.selinv(*L, work=work)
    Y = bta.selinv(*L, work=work)
    Z = bta.selinv(*L, out=L, work=work)
    for x, y, z in zip(X, Y, Z):
        assert torch_cuda.equal(x, y) and torch_cuda.equal(x, z)
    e = errs(dict(zip("DBRT", to_np(X))), {"D": Xo["XD"], "B": Xo["XB"], "R": Xo["XR"], "T": Xo["XT"]}, lower=())
    say(f"   X err {e}")
    assert max(e.values()) < TOL


@pytest.mark.parametrize("mode", [1, 3, 4, 5, 6, 7])
@pytest.mark.parametrize("n,b,a", [(7, 384, 6), (6, 193, 130)])
def test_selinv_product_by_product_kernels(torch_cuda, n, b, a, mode):
    """The same path with every product kernel."""
    from paper_2503_17528_amd import bta

    prev = bta.gemm_mode(mode)
    try:
        test_selinv_product_by_product(torch_cuda, n, b, a)
    finally:
        bta.gemm_mode(prev)


def test_workspace_falls_back_to_the_least(torch_cuda, monkeypatch):
    """No room for the workspace that the selected inversion asks for: the binding
    takes the least one, and the result is the product-by-product one; a call with
    nothing smaller to fall back to raises."""
    from paper_2503_17528_amd import bta

    torch, n, b, a = torch_cuda, 20, 256, 4
    say(f"case workspace fallback n={n} b={b} a={a}")
    L = bta.factor(*to_dev(synth.make_np(synth.workload(n, b, a), 2)))[:4]
    full, least = (f(bta.BTA_OP_SELINV, n, b, a) for f in (bta.bta_workspace_bytes, bta.bta_workspace_min_bytes))
    out = [torch.empty_like(t) for t in L]
    want = bta.selinv(*L, work=torch.empty(least, dtype=torch.uint8, device="cuda"))
    real = torch.empty

    def no_room(*size, **kw):
        if kw.get("dtype") == torch.uint8 and size[0] > least:
            raise torch.OutOfMemoryError("no room")
        return real(*size, **kw)

    monkeypatch.setattr(torch, "empty", no_room)
    work, nbytes = bta.workspace(bta.BTA_OP_SELINV, n, b, a, "cuda")
    assert nbytes == work.numel() == least < full
    bta.selinv(*L, out=out)
    with pytest.raises(torch.OutOfMemoryError):
        bta.workspace(bta.BTA_OP_SOLVE, 400, b, a, "cuda", 64)
    monkeypatch.undo()
    for x, y in zip(out, want):
        assert torch.equal(x, y)


@pytest.mark.parametrize("mode", [1, 2])
@pytest.mark.parametrize("n,b,a", [(3, 384, 6), (2, 520, 8), (4, 136, 2), (2, 64, 130), (5, 192, 0)])
def test_selinv_gemm_kernels(torch_cuda, n, b, a, mode):
    """Both GEMM kernel families of the selected inversion (register-staged,
    direct-to-LDS with 128 and 64 tiles) against the oracle."""
    from paper_2503_17528_amd import bta

    say(f"case selinv gemm mode={mode} n={n} b={b} a={a}")
    wl = synth.workload(n, b, a)
    Q = synth.make_np(wl, 4)
    F = oracle.pobtaf(Q["D"], Q["B"], Q["R"], Q["T"])
    Xo = oracle.pobtasi(F["LD"], F["LB"], F["LR"], F["LT"])
    prev = bta.gemm_mode(mode)
    try:
        Lg, info, Xg = _run(torch_cuda, Q)
    finally:
        bta.gemm_mode(prev)
    assert info == 0
    _check(Lg, Xg, F, Xo, n, b, a)


@pytest.mark.parametrize("n,b,a", [(4, 100, 3), (3, 64, 0), (2, 130, 70), (3, 128, 256)])
def test_inplace_matches(torch_cuda, n, b, a):
    say(f"case in-place n={n} b={b} a={a}")
    Q = synth.make_np(synth.workload(n, b, a), 8)
    F = oracle.pobtaf(Q["D"], Q["B"], Q["R"], Q["T"])
    Xo = oracle.pobtasi(F["LD"], F["LB"], F["LR"], F["LT"])
    Lg, info, Xg = _run(torch_cuda, Q, inplace=True)
    assert info == 0
    # in place: the L outputs were overwritten by X; check X only
    eX = errs(dict(zip("DBRT", Xg)), {"D": Xo["XD"], "B": Xo["XB"], "R": Xo["XR"], "T": Xo["XT"]}, lower=())
    say(f"   X err {eX}")
    assert max(eX.values()) < TOL


def test_garbage_upper_triangle_is_ignored(torch_cuda):
    n, b, a = 3, 96, 5
    say(f"case garbage-upper n={n} b={b} a={a}")
    Q = synth.make_np(synth.workload(n, b, a), 4)
    F = oracle.pobtaf(Q["D"], Q["B"], Q["R"], Q["T"])
    Xo = oracle.pobtasi(F["LD"], F["LB"], F["LR"], F["LT"])
    G = {k: v.copy() for k, v in Q.items()}
    for i in range(n):
        G["D"][i] += np.triu(np.full((b, b), np.nan), 1)
    G["T"] += np.triu(np.full((a, a), 1e300), 1)
    Lg, info, Xg = _run(torch_cuda, G)
    assert info == 0
    _check(Lg, Xg, F, Xo, n, b, a)


@pytest.mark.parametrize("where", ["first", "middle", "tip", "nan"])
def test_not_positive_definite_reports_row(torch_cuda, where):
    from paper_2503_17528_amd import bta

    n, b, a = 4, 80, 3
    say(f"case not-PD {where}")
    Q = synth.make_np(synth.workload(n, b, a), 6)
    if where == "first":
        Q["D"][0][5, 5] = -1.0
    elif where == "middle":
        Q["D"][2][70, 70] = -1e6
    elif where == "tip":
        Q["T"][1, 1] = -1e6
    else:
        Q["D"][1][10, 10] = np.nan
    F = oracle.pobtaf(Q["D"], Q["B"], Q["R"], Q["T"])
    assert F["info"] > 0
    D, B, R, T = to_dev(Q)
    L = bta.factor(D, B, R, T, check=False)
    torch_cuda.cuda.synchronize()
    assert int(L[4].item()) == F["info"]
    with pytest.raises(bta.NotPositiveDefinite) as ei:
        bta.factor(D, B, R, T)
    assert ei.value.row == F["info"]


@pytest.mark.parametrize("n,b,a,nrhs", [(1, 3, 0, 1), (4, 100, 3, 1), (3, 64, 0, 2), (2, 130, 70, 3), (16, 64, 4, 1),
                                            (4, 128, 256, 2)])
def test_solve_and_logdet(torch_cuda, n, b, a, nrhs):
    from paper_2503_17528_amd import bta

    say(f"case solve/logdet n={n} b={b} a={a} nrhs={nrhs}")
    wl = synth.workload(n, b, a)
    Q = synth.make_np(wl, 9)
    y = synth.rhs_np(wl, 9, nrhs)
    F = oracle.pobtaf(Q["D"], Q["B"], Q["R"], Q["T"])
    xo = oracle.pobtas(F["LD"], F["LB"], F["LR"], F["LT"], y)
    ldo = oracle.logdet(F["LD"], F["LT"])
    D, B, R, T = to_dev(Q)
    L = bta.factor(D, B, R, T)
    yd = torch_cuda.from_numpy(y).to("cuda")
    x = bta.solve(*L[:4], yd)
    ld = bta.logdet(L[0], L[3])
    torch_cuda.cuda.synchronize()
    xg = x.cpu().numpy()
    e = np.linalg.norm(xg - xo) / np.linalg.norm(xo)
    say(f"   solve rel err {e:.3e}  logdet {float(ld.item())} vs {ldo}")
    assert e < TOL
    assert abs(float(ld.item()) - ldo) <= TOL * abs(ldo)


# edges of a task's 16 rows, of a wave's and a chunk's k range (512, 1024), one and
# several groups of right-hand sides (up to 4 singly, then 16 at a time), wide tips
@pytest.mark.parametrize("n,b,a,nrhs", [(1, 1, 0, 5), (3, 15, 1, 4), (4, 16, 0, 16), (3, 17, 3, 17), (3, 513, 2, 5),
                                        (3, 530, 70, 33), (3, 1025, 2, 1), (2, 1040, 130, 4), (5, 128, 40, 64)])
def test_solve_groups(torch_cuda, n, b, a, nrhs):
    test_solve_and_logdet(torch_cuda, n, b, a, nrhs)


# the same with more right-hand sides: singly up to 192 tasks of 16 rows a phase, else 16 wide
@pytest.mark.parametrize("n,b,a,nrhs", [(2, 16, 3, 192), (2, 16, 3, 193), (3, 17, 0, 97), (3, 1, 1, 200), (2, 512, 5, 6),
                                        (2, 511, 129, 7), (4, 256, 2, 12)])
def test_solve_group_edges(torch_cuda, n, b, a, nrhs):
    test_solve_and_logdet(torch_cuda, n, b, a, nrhs)


@pytest.mark.parametrize("nrhs", [1, 6])
def test_solve_chunks(torch_cuda, nrhs):
    """More blocks than inverses fit in the workspace at once (14 of 4096: two
    chunks, the first formed again for the backward sweep): x from y = L L^T x."""
    from paper_2503_17528_amd import bta

    torch, n, b, a = torch_cuda, 14, 4096, 3
    say(f"case solve in chunks n={n} b={b} a={a} nrhs={nrhs}")
    wl = synth.workload(n, b, a, "scaled")
    L = [torch.zeros(z, dtype=torch.float64, device="cuda") for z in ((n, b, b), (n - 1, b, b), (n, a, b), (a, a))]
    for i in range(n):
        L[0][i] = synth.factor_block_torch(wl, 2, synth.KIND_DIAG, i, "cuda")
        L[2][i] = synth.factor_block_torch(wl, 2, synth.KIND_ARROW, i, "cuda")
        if i < n - 1:
            L[1][i] = synth.factor_block_torch(wl, 2, synth.KIND_SUB, i, "cuda")
    L[3].copy_(synth.factor_block_torch(wl, 2, synth.KIND_TIP, 0, "cuda"))
    x = torch.randn(n * b + a, nrhs, dtype=torch.float64, device="cuda", generator=torch.Generator("cuda").manual_seed(4))
    xb, xt = x[:n * b].view(n, b, nrhs), x[n * b:]
    u = torch.zeros_like(xb)  # L^T x, then L u
    for i in range(n):
        u[i] = L[0][i].T @ xb[i] + L[2][i].T @ xt + (L[1][i].T @ xb[i + 1] if i < n - 1 else 0.0)
    ut = L[3].T @ xt
    y = torch.zeros_like(x)
    for i in range(n):
        y[i * b:(i + 1) * b] = L[0][i] @ u[i] + (L[1][i - 1] @ u[i - 1] if i else 0.0)
    y[n * b:] = L[3] @ ut + sum(L[2][i] @ u[i] for i in range(n))
    got = bta.solve(*L, y)
    e = float((got - x).norm() / x.norm())
    say(f"   solve rel err {e:.3e}")
    assert e < TOL


# bit patterns: the NaN that marks a vector element as not yet written, that NaN negated, NaN, infinities
@pytest.mark.parametrize("bits", [0x7FF8B17AB17AB17A, 0xFFF8B17AB17AB17A, 0x7FF8000000000000, 0x7FF0000000000000,
                                  0xFFF0000000000000], ids=hex)
@pytest.mark.parametrize("nrhs", [3, 20])
@pytest.mark.parametrize("a", [0, 5])
def test_solve_right_hand_side_not_finite(torch_cuda, a, nrhs, bits):
    """Right-hand sides with NaNs and infinities, among them the value by which
    single vectors mark elements that are pending: the call ends, every x of such a
    right-hand side is not finite, and the other ones keep their bits."""
    from paper_2503_17528_amd import bta

    torch, n, b = torch_cuda, 4, 256
    say(f"case solve not finite a={a} nrhs={nrhs} {bits:#x}")
    L = bta.factor(*to_dev(synth.make_np(synth.workload(n, b, a), 3)))[:4]
    N = n * b + a
    y = torch.randn(N, nrhs, dtype=torch.float64, device="cuda", generator=torch.Generator("cuda").manual_seed(1))
    want = bta.solve(*L, y)
    bad = y.clone()
    w = bad.view(torch.int64)
    v = bits - (1 << 64) if bits >> 63 else bits
    w[0, 0] = w[b + 17, 0] = w[2 * b:2 * b + 40, 0] = w[N - 1, 0] = v  # first, inner, a run, last
    w[N - 1, 2] = v
    x = bta.solve(*L, bad)
    torch.cuda.synchronize()
    for j in range(nrhs):
        if j in (0, 2):
            assert not bool(x[:, j].isfinite().any()), j
        else:
            assert torch.equal(x[:, j], want[:, j]), j


@pytest.mark.parametrize("n,b,a", [(6, 256, 4), (5, 193, 0), (4, 800, 70)])
def test_wait_that_gives_up_leaves_nan(torch_cuda, n, b, a):
    """Waits of the persistent sweeps that give up (in the solve the first to find
    its data pending, in the selected inversion all): everything that depends on them
    is NaN, all of x included, the call ends, and the next one is as good as any."""
    from paper_2503_17528_amd import bta

    torch = torch_cuda
    say(f"case waits give up n={n} b={b} a={a}")
    lib = bta.lib()
    lib.bta_internal_wait_limit.argtypes = [ctypes.c_longlong]
    lib.bta_internal_wait_limit.restype = ctypes.c_longlong
    L = bta.factor(*to_dev(synth.make_np(synth.workload(n, b, a, "scaled"), 2)))[:4]
    y = [torch.randn(n * b + a, k, dtype=torch.float64, device="cuda") for k in (1, 64)]
    want = list(bta.selinv(*L)) + [bta.solve(*L, v) for v in y]
    torch.cuda.synchronize()
    prev = lib.bta_internal_wait_limit(0)
    try:
        void = list(bta.selinv(*L)) + [bta.solve(*L, v) for v in y]
        torch.cuda.synchronize()
    finally:
        lib.bta_internal_wait_limit(prev)
    assert all(bool(t.isnan().all()) for t in void[:3] + void[4:])
    assert torch.equal(void[3], want[3])  # X_nn does not depend on the sweep
    again = list(bta.selinv(*L)) + [bta.solve(*L, v) for v in y]
    assert all(torch.equal(p, q) for p, q in zip(want, again))


def test_abi_rejects_bad_workspace_on_device(torch_cuda):
    from paper_2503_17528_amd import bta

    n, b, a = 2, 64, 4
    Q = synth.make_np(synth.workload(n, b, a), 1)
    D, B, R, T = to_dev(Q)
    work = torch_cuda.empty(16, dtype=torch_cuda.uint8, device="cuda")
    with pytest.raises(bta.BTAError) as ei:
        bta.factor(D, B, R, T, work=work)
    assert ei.value.status == bta.BTA_EINVAL


@pytest.mark.parametrize("delay", [0, 1, 3, 10])
def test_factor_sub_delays(torch_cuda, delay):
    """Every SUB dispatch delay gives the oracle's factor (the delay only
    reorders the tickets of the coupling block's tiles): a 10 x 10 tile band
    with ragged tiles and a two-tile tip, the delay set through the tuning
    table (10 = every SUB task after its step's last column)."""
    from paper_2503_17528_amd import autotune, bta

    n, b, a = 4, 610, 70
    say(f"case sub_delay={delay} n={n} b={b} a={a}")
    k = autotune.key("factor", b, a, "sub_delay")
    autotune.set_entry(k, delay)
    try:
        wl = synth.workload(n, b, a)
        Q = synth.make_np(wl, 12)
        F = oracle.pobtaf(Q["D"], Q["B"], Q["R"], Q["T"])
        D, B, R, T = to_dev(Q)
        L = bta.factor(D, B, R, T)
        torch_cuda.cuda.synchronize()
        e = errs(dict(zip("DBRT", to_np(L[:4]))), {"D": F["LD"], "B": F["LB"], "R": F["LR"], "T": F["LT"]})
        say(f"   L err {e}")
        assert max(e.values()) < TOL, e
    finally:
        autotune.clear()
