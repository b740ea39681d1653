"""GPU parity: the HIP path (through the C ABI) against the CPU oracle on the same seeded inputs.
`assert_close` bounds the error of every element (one unit in the last place of the storage type plus the
accumulated arithmetic error, scaled by the row), of every row and of the whole block."""
import hashlib

import numpy as np
import pytest
import torch

import paper_2601_07396_amd as pkg
from oracle import ref_fit_basis, ref_full_step, ref_forecast
from synth import WORKLOADS, FeatureStream, is_full_step, torch_dtype
from util import TOL, TWO_LAUNCHES, to_np, rel_err, assert_close, principal_sines

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _rand_problem(B, N, D, k, dtype, seed, ldf=None):
    g = torch.Generator().manual_seed(seed)
    ldf = D if ldf is None else ldf
    buf = torch.zeros(B, N, ldf, dtype=dtype)
    buf[:, :, :D] = torch.randn(B, N, D, generator=g).to(dtype)
    V = torch.linalg.qr(torch.randn(B, D, k, generator=g, dtype=torch.float64))[0].float().contiguous()
    S = torch.randn(B, N, k, generator=g)
    return buf, V, S


def _run_full(Fbuf, D, V, S, alpha, init, want_C=True, inplace=False, packed="auto"):
    F = Fbuf.to(DEV)
    Fv = F[:, :, :D]
    shape = pkg.make_shape(Fv, V.shape[2])
    Vd, Sd = V.to(DEV), S.clone().to(DEV)
    pk = pkg.pack_basis(shape, Vd) if packed == "auto" else None
    R = F if inplace else torch.full_like(F, 7.0)
    Cd = torch.empty_like(Sd) if want_C else None
    pkg.svdcache_full_step(shape, Fv, Vd, pk, R[:, :, :D], Sd, Cd, alpha, init)
    torch.cuda.synchronize()
    return R, Sd, Cd, shape, pk


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16], ids=["f32", "bf16"])
@pytest.mark.parametrize("B,N,D,k", [(2, 256, 64, 8), (1, 37, 72, 5), (3, 130, 200, 17), (1, 1, 8, 1),
                                     (1, 20, 16, 16), (2, 67, 264, 40)])
def test_full_step_and_forecast_general_shapes(dtype, B, N, D, k):
    store = "f32" if dtype == torch.float32 else "bf16"
    Fbuf, V, S0 = _rand_problem(B, N, D, k, dtype, seed=B * 1000 + N)
    for init in (True, False):
        R, S, Cc, shape, pk = _run_full(Fbuf, D, V, S0, 0.3, init)
        Fh = torch.empty_like(R)
        pkg.svdcache_forecast(shape, S, V.to(DEV), pk, R, Fh)
        torch.cuda.synchronize()
        for b in range(B):
            Rr, Sr, Cr = ref_full_step(to_np(Fbuf[b]), to_np(V[b]), to_np(S0[b]), 0.3, init, store)
            assert_close(to_np(R[b]), Rr, store, f"R[{b}]", floor_of=to_np(Fbuf[b]))
            assert_close(to_np(S[b]), Sr, "f32", f"S[{b}]")
            assert_close(to_np(Cc[b]), Cr, "f32", f"C[{b}]")
            # the oracle forecasts from its OWN state: nothing computed on the GPU is fed to it
            Fr = ref_forecast(Sr, to_np(V[b]), Rr, store)
            assert_close(to_np(Fh[b]), Fr, store, f"Fhat[{b}]", scale_of=to_np(Fbuf[b]), ulp_of=Rr)


@pytest.mark.parametrize("B,N,D,k", [(1, 17, 24, 15), (2, 16, 40, 16), (1, 33, 1304, 33), (1, 70, 296, 65), (2, 131, 392, 129),
                                     (1, 1030, 1040, 1024)])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16], ids=["f32", "bf16"])
def test_general_kernels_at_the_edges_of_their_tiles(dtype, B, N, D, k):
    """Ragged 16-row tiles, 32-channel chunks and 16-, 32- and 64-coefficient groups, the largest rank; a row that holds
    an infinity or a NaN stays the only one affected."""
    store = "f32" if dtype == torch.float32 else "bf16"
    if dtype == torch.float32:
        D += 4                          # a chunk whose last piece of eight channels is half outside
    Fbuf, V, S0 = _rand_problem(B, N, D, k, dtype, seed=N + k)
    R, S, Cc, shape, pk = _run_full(Fbuf, D, V, S0, 0.3, False)
    assert pk is None
    Fh = torch.empty_like(R)
    pkg.svdcache_forecast(shape, S, V.to(DEV), None, R, Fh)
    torch.cuda.synchronize()
    for b in range(B):
        Rr, Sr, Cr = ref_full_step(to_np(Fbuf[b]), to_np(V[b]), to_np(S0[b]), 0.3, False, store)
        assert_close(to_np(R[b]), Rr, store, f"R[{b}]", floor_of=to_np(Fbuf[b]))
        assert_close(to_np(S[b]), Sr, "f32", f"S[{b}]")
        assert_close(to_np(Cc[b]), Cr, "f32", f"C[{b}]")
        Fr = ref_forecast(Sr, to_np(V[b]), Rr, store)
        assert_close(to_np(Fh[b]), Fr, store, f"Fhat[{b}]", scale_of=to_np(Fbuf[b]), ulp_of=Rr)
    bad = Fbuf.clone()
    bad[0, 3, 1], bad[0, 5, D - 1] = float("inf"), float("nan")
    R2, S2, C2, _, _ = _run_full(bad, D, V, S0, 0.3, False)
    Fh2 = torch.empty_like(R)
    pkg.svdcache_forecast(shape, S2, V.to(DEV), None, R2, Fh2)
    torch.cuda.synchronize()
    keep = torch.ones(N, dtype=torch.bool)
    keep[[3, 5]] = False
    for got, want in ((R2, R), (S2, S), (C2, Cc), (Fh2, Fh)):
        assert torch.equal(got[0][keep], want[0][keep]) and not torch.isfinite(got[0][[3, 5]].float()).all(dim=1).any()


@pytest.mark.parametrize("dtype,N,D,k", [(torch.bfloat16, 601, 2008, 64), (torch.bfloat16, 8101, 520, 50), (torch.bfloat16, 8701, 520, 50),
                                         (torch.bfloat16, 5003, 520, 127), (torch.float32, 8701, 796, 50), (torch.float32, 5003, 796, 100),
                                         (torch.bfloat16, 8101, 1288, 50), (torch.float32, 6001, 1032, 117)])
def test_general_kernels_in_bf16_parts(dtype, N, D, k):
    """Tiles of 16, 32 and 48 rows, ragged rows, channels (an odd number of chunks, a chunk that is partly outside) and coefficients."""
    test_general_kernels_at_the_edges_of_their_tiles(dtype, 1, N, D, k)


# (float32 rows of 8101 x 3304 at rank 33 stay on the float32 instructions, whose chains the test above is about)
@pytest.mark.parametrize("dtype,N,D,k", [(torch.bfloat16, 8701, 1408, 50), (torch.float32, 8701, 1408, 50), (torch.bfloat16, 8101, 3304, 33)])
def test_general_projection_in_parts_is_as_good_as_float32(dtype, N, D, k):
    """C from bf16 parts: the leading products of a chunk of 32 channels are one matrix instruction, whose 32 products and sum
    are rounded a few times (at most like a chain over them, 0.41 u sqrt(32 / 2) of the chunk's share of C, u = 2^-24), the
    chunks are added in float64, the other products are 2^-8 of that, and the result is rounded once: 0.41 u sqrt(17)."""
    g = torch.Generator().manual_seed(D + k)
    F = torch.randn(1, N, D, generator=g).to(dtype)
    V = torch.randn(1, D, k, generator=g) / D ** 0.5
    _, _, Cc, _, pk = _run_full(F, D, V, torch.zeros(1, N, k), 0.3, True)
    assert pk is None
    assert rel_err(to_np(Cc[0]), to_np(F[0]) @ to_np(V[0])) <= 0.41 * 2.0 ** -24 * 17 ** 0.5


@pytest.mark.parametrize("N,D,k,cached", [(6001, 1036, 117, True), (8701, 1408, 50, False)])
def test_general_reconstruction_in_parts_is_as_good_as_float32(N, D, k, cached):
    """R and Fhat of float32 rows that lie mostly in the span of the basis.  P = C V^T from bf16 parts: the leading products of 32
    coefficients are one matrix instruction (0.41 u sqrt(32 / 2) of P at most, as for C), up to four of them and the other products
    are added to it, and R or Fhat is rounded once more: 0.41 u sqrt(20) of P, 1.1e-7; the float32 instructions stay within that too."""
    g = torch.Generator().manual_seed(D + k)
    V = torch.linalg.qr(torch.randn(1, D, k, generator=g, dtype=torch.float64))[0].float().contiguous()
    A = torch.randn(1, N, k, generator=g)
    F = ((A.double() @ V.double().transpose(1, 2)) + 0.05 * torch.randn(1, N, D, generator=g) * (k / D) ** 0.5).float()
    R, S, Cc, shape, pk = _run_full(F, D, V, torch.zeros(1, N, k), 0.3, True)
    assert pk is None
    P = to_np(Cc[0]) @ to_np(V[0]).T
    bound = 0.41 * 2.0 ** -24 * 20 ** 0.5 * np.linalg.norm(P)
    assert np.linalg.norm(to_np(R[0]) - (to_np(F[0]) - P)) <= bound
    if cached:
        Fh = torch.empty_like(R)
        pkg.svdcache_forecast(shape, S, V.to(DEV), None, R, Fh)
        torch.cuda.synchronize()
        assert np.linalg.norm(to_np(Fh[0]) - (to_np(S[0]) @ to_np(V[0]).T + to_np(R[0]))) <= bound


@pytest.mark.parametrize("dtype,N,D,k", [(torch.bfloat16, 601, 2008, 64), (torch.bfloat16, 8101, 520, 50), (torch.bfloat16, 8701, 520, 50),
                                         (torch.bfloat16, 8101, 1288, 50), (torch.float32, 8701, 796, 50), (torch.float32, 6001, 1036, 117)])
def test_general_kernels_in_parts_keep_the_range_of_float32(dtype, N, D, k):
    """Infinities, a NaN, values next to the largest float32, and rows and basis columns down to the smallest normal ones: what
    float64 says is infinite, NaN or finite is so in the results, and finite results are within 16 u (u = 2^-24) of the norm of
    their row and, for a basis column of its own scale, of that column (the sums of a product are off by 0.41 u sqrt(17) or less)."""
    store = "f32" if dtype == torch.float32 else "bf16"
    tol, inf, nan, big = 16 * 2.0 ** -24, float("inf"), float("nan"), 3.395e38 if store == "f32" else 3.38e38
    Fbuf, V, S0 = _rand_problem(1, N, D, k, dtype, seed=N + k)
    F, S0 = Fbuf.clone(), S0 * 1e-3
    odd = {3: "inf", 17: "-inf and inf", 40: "big", 100: "tiny", 130: "nan", N - 1: "big and last"}
    F[0, 3, 1], F[0, 17, 2], F[0, 17, D - 1], F[0, 40, 7], F[0, 130, 0], F[0, N - 1, D - 2] = inf, -inf, inf, big, nan, -big
    F[0, 100] *= 2.0 ** -112
    S0[0, list(odd)] = 0.0                                # S is 0.25 C there
    cols = {5: 2.0 ** -112, 9: 2.0 ** 100}
    Vs = V.clone()
    for j, scale in cols.items():
        Vs[0, :, j] *= scale

    def check(got, want, what, along=1):
        got = to_np(got)
        assert np.array_equal(np.isnan(got), np.isnan(want)), f"{what}: NaN"
        assert np.array_equal(np.isposinf(got), np.isposinf(want)) and np.array_equal(np.isneginf(got), np.isneginf(want)), f"{what}: inf"
        fin = np.isfinite(want).all(axis=along)
        got, want = (got[fin], want[fin]) if along == 1 else (got[:, fin].T, want[:, fin].T)
        err, ref = np.linalg.norm(got - want, axis=1), np.linalg.norm(want, axis=1)
        assert (err <= (2.0 ** -8 if what in ("R", "Fhat") and store == "bf16" else tol) * ref).all(), f"{what}: {(err / ref).max():.2e}"

    with np.errstate(all="ignore"):
        R, S, Cc, _, pk = _run_full(F, D, V, S0, 0.25, False)
        assert pk is None
        C64 = to_np(F[0]) @ to_np(V[0])
        check(Cc[0], C64, "C")
        check(S[0][list(odd)], 0.25 * C64[list(odd)], "S")
        Cg = to_np(Cc[0])
        R64 = to_np(F[0]) - Cg @ to_np(V[0]).T
        check(R[0], R64, "R")
        assert not np.isfinite(R64[[3, 17, 130]]).any() and np.isfinite(np.delete(R64, [3, 17, 130], axis=0)).all()
        # columns of very different scales: each to its own norm; then the rows of a state, with a residual of its scale
        _, _, Cs, _, _ = _run_full(Fbuf, D, Vs, S0, 0.25, True)
        check(Cs[0], to_np(Fbuf[0]) @ to_np(Vs[0]), "C", along=0)
        Sx = Cc.clone()                                   # with the infinities and the NaN of the features' rows
        Rx = Fbuf.to(DEV) * 0.5
        Rx[0, 100] *= 2.0 ** -112
        Fh = torch.empty_like(Rx)
        shape = pkg.make_shape(Rx, k)
        pkg.svdcache_forecast(shape, Sx, V.to(DEV), None, Rx, Fh)
        torch.cuda.synchronize()
        Fh64 = to_np(Sx[0]) @ to_np(V[0]).T + to_np(Rx[0])
        check(Fh[0], Fh64, "Fhat")
        pkg.svdcache_forecast_combine(shape, [Sx, S], [1.5, -0.5], V.to(DEV), None, Rx, Rx, Fh)
        torch.cuda.synchronize()
        Fh64 = (1.5 * to_np(Sx[0]) - 0.5 * to_np(S[0])) @ to_np(V[0]).T + 2 * to_np(Rx[0])
        check(Fh[0][:100], Fh64[:100], "Fhat")
        # the same with the results in place of the residual
        want = Fh.clone() * 0
        pkg.svdcache_forecast(shape, Sx, V.to(DEV), None, Rx, want)
        pkg.svdcache_forecast(shape, Sx, V.to(DEV), None, Rx, Rx)
        torch.cuda.synchronize()
        assert torch.equal(torch.nan_to_num(want.float()), torch.nan_to_num(Rx.float()))


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16], ids=["f32", "bf16"])
def test_general_projection_sums_in_short_chains(dtype):
    """C of many channels: float32 chains of at most 16 products, their sums in a chain of one link per 512 channels.  A chain
    of n terms of random sign is off by 0.41 u sqrt(n / 2) of its result (0.41 u: root mean square of the rounding of one
    addition, u = 2^-24), so 16 links and D / 512 links with the two additions between them and the final rounding give
    0.41 u sqrt(8 + D / 1024 + 3), 1.35e-7 at 20000 channels; one chain per accumulator would be at 4.4e-7."""
    N, D, k = 256, 20000, 21
    g = torch.Generator().manual_seed(D + k)
    F = torch.randn(1, N, D, generator=g).to(dtype)
    V = torch.randn(1, D, k, generator=g) / D ** 0.5
    R, S, Cc, _, pk = _run_full(F, D, V, torch.zeros(1, N, k), 0.3, True)
    assert pk is None
    bound = 1.5 * 0.41 * 2.0 ** -24 * (8 + D / 1024 + 3) ** 0.5
    assert rel_err(to_np(Cc[0]), to_np(F[0]) @ to_np(V[0])) <= bound


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16], ids=["f32", "bf16"])
def test_strided_rows_inplace_and_null_C(dtype):
    store = "f32" if dtype == torch.float32 else "bf16"
    B, N, D, k, ldf = 2, 50, 64, 8, 96
    Fbuf, V, S0 = _rand_problem(B, N, D, k, dtype, seed=5, ldf=ldf)
    R, S, Cc, shape, pk = _run_full(Fbuf, D, V, S0, 0.5, False, want_C=False, inplace=True)
    assert Cc is None and shape.ldf == ldf
    state = []
    for b in range(B):
        Rr, Sr, _ = ref_full_step(to_np(Fbuf[b, :, :D]), to_np(V[b]), to_np(S0[b]), 0.5, False, store)
        assert_close(to_np(R[b, :, :D]), Rr, store, "R in place")
        assert_close(to_np(S[b]), Sr, "f32", "S")
        state.append((Rr, Sr))
    # the padding columns beyond D are not touched
    assert torch.equal(R[:, :, D:].cpu(), Fbuf[:, :, D:])
    # forecast in place (Fhat aliases R); the oracle continues from its own state
    pkg.svdcache_forecast(shape, S, V.to(DEV), pk, R[:, :, :D], R[:, :, :D])
    torch.cuda.synchronize()
    for b in range(B):
        Fr = ref_forecast(state[b][1], to_np(V[b]), state[b][0], store)
        assert_close(to_np(R[b, :, :D]), Fr, store, "Fhat in place", scale_of=to_np(Fbuf[b, :, :D]), ulp_of=state[b][0])


def test_forecast_after_init_reproduces_F_exactly_in_fp32_tolerance():
    B, N, D, k = 1, 64, 128, 16
    Fbuf, V, S0 = _rand_problem(B, N, D, k, torch.float32, seed=9)
    R, S, Cc, shape, pk = _run_full(Fbuf, D, V, S0, 0.5, True)
    assert torch.equal(S, Cc)
    Fh = torch.empty_like(R)
    pkg.svdcache_forecast(shape, S, V.to(DEV), pk, R, Fh)
    torch.cuda.synchronize()
    assert rel_err(to_np(Fh), to_np(Fbuf)) <= 1e-6


def _fit_checks(F_cpu, V, sigma, fro2, k, store, lead=None):
    """Compare a fitted basis with the exact truncated SVD.  Several bases are correct (signs,
    rotations inside clusters of close singular values), so compare what is unique: singular values,
    captured energy, orthonormality, and the leading subspace scaled by its spectral gap."""
    tol = TOL[store]
    Fd = to_np(F_cpu)
    n_all = min(Fd.shape)
    _, s_all, _ = ref_fit_basis(Fd, n_all) if n_all <= 512 else (None, None, None)
    Vr, sr, fr = ref_fit_basis(Fd, k)
    Vg = to_np(V)
    assert np.abs(Vg.T @ Vg - np.eye(k)).max() <= 1e-5
    sg = to_np(sigma)
    assert np.all(np.diff(sg) <= 1e-6 * sg[0])
    assert np.abs(sg / sr - 1).max() <= tol, f"sigma rel err {np.abs(sg / sr - 1).max():.2e}"
    assert abs(float(fro2) / fr - 1) <= 1e-5
    captured = np.sum((Fd @ Vg) ** 2)
    assert 1 - captured / np.sum(sr ** 2) <= tol
    # sigma reported must be the norms of F v_j
    assert np.abs(np.linalg.norm(Fd @ Vg, axis=0) / sg - 1).max() <= max(tol, 1e-4)
    if s_all is not None:
        lead = lead or max(1, k // 2)
        gap = s_all[lead - 1] / (s_all[lead - 1] - s_all[lead])
        sines = principal_sines(Vg[:, :lead], Vr[:, :lead])
        assert sines.max() <= tol * gap + 2e-4 * gap, f"leading subspace off: {sines.max():.2e} (gap factor {gap:.1f})"


def test_fit_basis_tiny_config():
    wl = WORKLOADS["tiny"]
    F = torch.stack([FeatureStream(wl, b).at(0) for b in range(wl.B)])
    V, sigma, fro2 = pkg.fit_basis(F.to(DEV), wl.k)
    torch.cuda.synchronize()
    for b in range(wl.B):
        _fit_checks(F[b], V[b], sigma[b], fro2[b], wl.k, "f32")


@pytest.mark.parametrize("dtype,N,D,k", [(torch.float32, 300, 96, 12), (torch.bfloat16, 500, 160, 16),
                                          (torch.float32, 40, 64, 40), (torch.bfloat16, 129, 72, 3)])
def test_fit_basis_power_law_inputs(dtype, N, D, k):
    store = "f32" if dtype == torch.float32 else "bf16"
    wl = WORKLOADS["flux1"].with_(N=N, D=D, k=k, dtype=store, signal_rank=min(48, D, N), rho=0.05)
    F = FeatureStream(wl, 0).at(0).unsqueeze(0)
    V, sigma, fro2 = pkg.fit_basis(F.to(DEV), k, q=6 if store == "f32" else 0)
    torch.cuda.synchronize()
    _fit_checks(F[0], V[0], sigma[0], fro2[0], k, store)


@pytest.mark.parametrize("alpha,interval", [(None, None), (0.3, 5), (0.7, 8), (0.1, 3), (1.0, 2)],
                         ids=["config", "a0.3-N5", "a0.7-N8", "a0.1-N3", "reuse-N2"])
def test_tiny_trajectory_matches_oracle_step_by_step(alpha, interval):
    """Config 1: 2 blocks, 256 x 64, k = 8, fp32, 10 steps, every 3rd a full step, alpha = 0.5; then the EMA
    weights and caching intervals of the sweep configuration (alpha = 0.1 is the paper's beta = 0.9, alpha = 1
    plain reuse).  Both sides use the same basis: the generator's leading directions."""
    wl = WORKLOADS["tiny"]
    if alpha is not None:
        wl = wl.with_(alpha=alpha, interval=interval, T=17)
    streams = [FeatureStream(wl, b) for b in range(wl.B)]
    feats = [torch.stack([s.at(t) for s in streams]) for t in range(wl.T)]
    F0 = feats[0].to(DEV)
    shape = pkg.make_shape(F0, wl.k)
    # the basis both sides use is the generator's own set of leading directions (nothing fitted on the GPU is
    # handed to the oracle; the fit has its own tests)
    V = torch.stack([s.V[:, :wl.k].float() for s in streams]).contiguous().to(DEV)
    pk = pkg.pack_basis(shape, V)
    R = torch.empty_like(F0)
    S = torch.empty(wl.B, wl.N, wl.k, device=DEV)
    Fh = torch.empty_like(F0)
    Vn = [to_np(V[b]) for b in range(wl.B)]
    Rr = [None] * wl.B
    Sr = [None] * wl.B
    first = True
    for t in range(wl.T):
        if is_full_step(t, wl.interval):
            pkg.svdcache_full_step(shape, feats[t].to(DEV), V, pk, R, S, None, wl.alpha, first)
            torch.cuda.synchronize()
            for b in range(wl.B):
                Rr[b], Sr[b], _ = ref_full_step(to_np(feats[t][b]), Vn[b], Sr[b], wl.alpha, first, "f32")
                assert_close(to_np(R[b]), Rr[b], "f32", f"t={t} R[{b}]")
                assert_close(to_np(S[b]), Sr[b], "f32", f"t={t} S[{b}]")
            first = False
        else:
            pkg.svdcache_forecast(shape, S, V, pk, R, Fh)
            torch.cuda.synchronize()
            for b in range(wl.B):
                assert_close(to_np(Fh[b]), ref_forecast(Sr[b], Vn[b], Rr[b], "f32"), "f32", f"t={t} Fhat[{b}]")


def test_checkpoint_split_is_bit_identical():
    """The state is (V, S, R) in caller-owned tensors: 10 steps in one go equal 5 + restore + 5."""
    wl = WORKLOADS["tiny"]
    feats = [torch.stack([FeatureStream(wl, b).at(t) for b in range(wl.B)]).to(DEV) for t in range(wl.T)]
    shape = pkg.make_shape(feats[0], wl.k)
    V, _, _ = pkg.fit_basis(feats[0], wl.k)

    def run(t0, t1, R, S, outs):
        for t in range(t0, t1):
            if is_full_step(t, wl.interval):
                pkg.svdcache_full_step(shape, feats[t], V, None, R, S, None, wl.alpha, t == 0)
                outs.append(R.clone())
            else:
                Fh = torch.empty_like(R)
                pkg.svdcache_forecast(shape, S, V, None, R, Fh)
                outs.append(Fh)
        torch.cuda.synchronize()

    R1, S1, o1 = torch.zeros_like(feats[0]), torch.zeros(wl.B, wl.N, wl.k, device=DEV), []
    run(0, wl.T, R1, S1, o1)
    R2, S2, o2 = torch.zeros_like(feats[0]), torch.zeros(wl.B, wl.N, wl.k, device=DEV), []
    run(0, 5, R2, S2, o2)
    saved = (R2.cpu(), S2.cpu())
    R3, S3 = saved[0].to(DEV), saved[1].to(DEV)
    run(5, wl.T, R3, S3, o2)
    assert all(torch.equal(a, b) for a, b in zip(o1, o2))


def test_errors_reported_through_the_binding():
    F = torch.zeros(1, 16, 16, device=DEV)
    shape = pkg.make_shape(F, 4)
    V = torch.zeros(1, 16, 4, device=DEV)
    S = torch.zeros(1, 16, 4, device=DEV)
    with pytest.raises(pkg.SvdcError) as e:
        pkg.svdcache_full_step(shape, F, V, None, F, S, None, 0.0, True)
    assert e.value.code == -5
    with pytest.raises(pkg.SvdcError) as e:
        pkg.svdcache_fit_basis(shape, F, V, torch.zeros(1, 4, device=DEV), None,
                               torch.zeros(16, device=DEV, dtype=torch.uint8))
    assert e.value.code == -6


# ---------------------------------------------------------------------------------------------
# matrix-core (MFMA) path for bf16 features
# ---------------------------------------------------------------------------------------------

def _lowrank_problem(B, N, D, k, seed, rho=0.05):
    """bf16 features with most energy in span(V) (like the real workload) plus a 5 % residual,
    so that R is a small difference of large terms."""
    g = torch.Generator().manual_seed(seed)
    V = torch.linalg.qr(torch.randn(B, D, k, generator=g, dtype=torch.float64))[0]
    Cc = torch.randn(B, N, k, generator=g, dtype=torch.float64) * (torch.arange(1, k + 1) ** -0.6)
    sig = Cc @ V.transpose(1, 2)
    noise = torch.randn(B, N, D, generator=g, dtype=torch.float64)
    noise *= (rho / (1 - rho)) ** 0.5 * sig.norm() / noise.norm()
    F = (sig + noise) * (D ** 0.5 / (sig.norm() / (B * N) ** 0.5))
    S = Cc.float() * float(F.abs().mean() / sig.abs().mean())
    return F.to(torch.bfloat16), V.float().contiguous(), S.contiguous()


@pytest.mark.parametrize("B,N,D,k", [(2, 200, 256, 32), (1, 77, 512, 8), (3, 64, 256, 64), (1, 131, 512, 128),
                                     (2, 49, 256, 20), (1, 150, 3072, 32), (2, 70, 3072, 64), (1, 140, 3072, 128),
                                     (1, 33, 3072, 16), (1, 80, 1024, 32), (1, 70, 1536, 64), (1, 50, 2048, 16),
                                     (1, 130, 2048, 128), (1, 45, 4096, 32), (1, 66, 4096, 64),
                                     (1, 70, 1152, 32), (2, 70, 1152, 64), (1, 90, 1920, 16), (1, 140, 1920, 128),
                                     (1, 75, 2560, 32), (1, 80, 2560, 64), (1, 60, 5120, 32), (1, 130, 5120, 128)])
def test_mfma_full_step_and_forecast(B, N, D, k):
    F, V, S0 = _lowrank_problem(B, N, D, k, seed=N * 7 + k)
    shape = pkg.make_shape(F, k)
    assert pkg.svdcache_has_mfma_path(shape)
    for init in (True, False):
        R, S, Cc, shape, pk = _run_full(F, D, V, S0, 0.5, init)
        assert pk is not None
        Fh = torch.empty_like(R)
        pkg.svdcache_forecast(shape, S, V.to(DEV), pk, R, Fh)
        torch.cuda.synchronize()
        for b in range(B):
            Rr, Sr, Cr = ref_full_step(to_np(F[b]), to_np(V[b]), to_np(S0[b]), 0.5, init, "bf16")
            assert_close(to_np(R[b]), Rr, "bf16", f"R[{b}]", floor_of=to_np(F[b]))
            assert_close(to_np(S[b]), Sr, "f32", f"S[{b}]")
            assert_close(to_np(Cc[b]), Cr, "f32", f"C[{b}]")
            Fr = ref_forecast(Sr, to_np(V[b]), Rr, "bf16")      # the oracle's own state
            assert_close(to_np(Fh[b]), Fr, "bf16", f"Fhat[{b}]", scale_of=to_np(F[b]), ulp_of=Rr)
            # the split-operand arithmetic is far inside the bf16 budget: the error is the output rounding
            assert rel_err(to_np(R[b]), Rr) <= 3e-3 and rel_err(to_np(Fh[b]), Fr) <= 3e-3


def test_mfma_and_general_paths_agree():
    """Same inputs through the packed (MFMA) and the unpacked (general) kernels."""
    B, N, D, k = 2, 100, 512, 32
    F, V, S0 = _lowrank_problem(B, N, D, k, seed=3)
    Ra, Sa, Ca, shape, pk = _run_full(F, D, V, S0, 0.3, False)
    Rb, Sb, Cb, _, none = _run_full(F, D, V, S0, 0.3, False, packed=None)
    assert pk is not None and none is None
    assert rel_err(to_np(Sa), to_np(Sb)) <= 1e-5 and rel_err(to_np(Ca), to_np(Cb)) <= 1e-5
    assert rel_err(to_np(Ra), to_np(Rb)) <= 3e-3
    Fa, Fb = torch.empty_like(Ra), torch.empty_like(Ra)
    pkg.svdcache_forecast(shape, Sa, V.to(DEV), pk, Ra, Fa)
    pkg.svdcache_forecast(shape, Sa, V.to(DEV), None, Ra, Fb)
    torch.cuda.synchronize()
    assert rel_err(to_np(Fa), to_np(Fb)) <= 3e-3


@pytest.mark.parametrize("dtype,B,N,D,k,pad", [(torch.bfloat16, 1, 33, 3072, 32, 0), (torch.bfloat16, 2, 1001, 3072, 64, 64),
                                               (torch.bfloat16, 1, 2290, 4096, 32, 0), (torch.float32, 1, 403, 1536, 24, 32),
                                               (torch.bfloat16, 1, 4097, 3072, 32, 8)])
def test_small_calls_take_narrow_slabs_and_short_tiles(dtype, B, N, D, k, pad):
    """Calls that do not fill the machine: cached steps over narrow channel slabs with few row tiles per workgroup (packed
    and plain state, two forecaster states), full steps over 16-row tiles, ragged last tiles, padded rows."""
    from oracle import ref_forecast_combine
    store = "f32" if dtype == torch.float32 else "bf16"
    g = torch.Generator().manual_seed(N + k)
    wide = torch.randn(B, N, D + pad, generator=g).to(dtype)
    V = torch.linalg.qr(torch.randn(B, D, k, generator=g, dtype=torch.float64))[0].float().contiguous()
    S0 = torch.randn(B, N, k, generator=g)
    buf = wide.to(DEV)
    F = buf[:, :, :D]
    R, Fh, Fp, Fc = (torch.zeros_like(buf)[:, :, :D] for _ in range(4))
    S = S0.to(DEV)
    C = torch.empty_like(S)
    shape = pkg.make_shape(F, k)
    Vd = V.to(DEV)
    packed = pkg.pack_basis(shape, Vd)
    Sp = pkg.alloc_packed_state(shape, DEV)
    pkg.svdcache_full_step(shape, F, Vd, packed, R, S, C, 0.3, False)
    pkg.svdcache_pack_state(shape, S, Sp)
    pkg.svdcache_forecast(shape, S, Vd, packed, R, Fh)
    pkg.svdcache_forecast_packed(shape, Sp, packed, R, Fp)
    pkg.svdcache_forecast_combine(shape, [S, C], [1.5, -0.5], Vd, packed, R, F, Fc)
    torch.cuda.synchronize()
    assert torch.equal(Fh, Fp)
    rows = slice(0, N) if N < 500 else torch.tensor([0, 1, 15, 16, 17, N // 2, N - 17, N - 2, N - 1])
    for b in range(B):
        Fb, Vb = to_np(wide[b, rows, :D]), to_np(V[b])
        Rr, Sr, Cr = ref_full_step(Fb, Vb, to_np(S0[b, rows]), 0.3, False, store)
        assert_close(to_np(R[b].cpu()[rows]), Rr, store, f"R[{b}]", floor_of=Fb)
        assert_close(to_np(S[b].cpu()[rows]), Sr, "f32", f"S[{b}]")
        assert_close(to_np(Fh[b].cpu()[rows]), ref_forecast(Sr, Vb, Rr, store), store, f"Fhat[{b}]", scale_of=Fb, ulp_of=Rr)
        want = ref_forecast_combine([Sr, Cr], [1.5, -0.5], Vb, Rr, Fb, store)
        assert_close(to_np(Fc[b].cpu()[rows]), want, store, f"combine[{b}]", scale_of=Fb, ulp_of=Rr)
    if pad:
        assert float(torch.as_strided(Fh, (B, N, pad), Fh.stride(), D).abs().max()) == 0.0


@pytest.mark.parametrize("dtype,B,N,D,k,pad", [(torch.float32, 1, 12311, 3072, 64, 0), (torch.float32, 2, 5003, 3072, 128, 4),
                                               (torch.float32, 1, 1001, 2304, 100, 0), (torch.bfloat16, 28, 1009, 1152, 32, 0),
                                               (torch.bfloat16, 3, 5407, 1152, 24, 8)])
def test_wide_float32_slabs_and_full_height_smoothing_tiles(dtype, B, N, D, k, pad):
    """Large calls: float32 cached steps over six- and four-chunk slabs, float32 full steps with the deeper operand ring,
    smoothed residuals over full-height row tiles; ragged last tiles, padded rows."""
    from oracle import ref_full_step_residual_ema
    store = "f32" if dtype == torch.float32 else "bf16"
    g = torch.Generator().manual_seed(N + k)
    wide = torch.randn(B, N, D + pad, generator=g).to(dtype)
    prev = torch.randn(N, D + pad, generator=g).to(dtype)
    V = torch.linalg.qr(torch.randn(B, D, k, generator=g, dtype=torch.float64))[0].float().contiguous()
    S0 = torch.randn(B, N, k, generator=g)
    buf = wide.to(DEV)
    F = buf[:, :, :D]
    R, Fh = (torch.zeros_like(buf)[:, :, :D] for _ in range(2))
    Rs = prev.to(DEV).expand(B, -1, -1).contiguous()[:, :, :D]
    S, Ss = S0.to(DEV), S0.to(DEV)
    C = torch.empty_like(S)
    shape = pkg.make_shape(F, k)
    Vd = V.to(DEV)
    packed = pkg.pack_basis(shape, Vd)
    pkg.svdcache_full_step(shape, F, Vd, packed, R, S, C, 0.3, False)
    pkg.svdcache_forecast(shape, S, Vd, packed, R, Fh)
    pkg.svdcache_full_step_residual_ema(shape, F, Vd, packed, Rs, Rs, Ss, None, 0.3, 0.25, False)
    torch.cuda.synchronize()
    rows = torch.tensor([0, 1, 15, 16, 47, 48, 63, 64, N // 2, N - 64, N - 49, N - 17, N - 16, N - 2, N - 1])
    for b in {0, B // 2, B - 1}:
        Fb, Vb, Sb = to_np(wide[b, rows, :D]), to_np(V[b]), to_np(S0[b, rows])
        Rr, Sr, Cr = ref_full_step(Fb, Vb, Sb, 0.3, False, store)
        assert_close(to_np(R[b].cpu()[rows]), Rr, store, f"R[{b}]", floor_of=Fb)
        assert_close(to_np(S[b].cpu()[rows]), Sr, "f32", f"S[{b}]")
        assert_close(to_np(C[b].cpu()[rows]), Cr, "f32", f"C[{b}]")
        assert_close(to_np(Fh[b].cpu()[rows]), ref_forecast(Sr, Vb, Rr, store), store, f"Fhat[{b}]", scale_of=Fb, ulp_of=Rr)
        Re, Se, _ = ref_full_step_residual_ema(Fb, Vb, Sb, to_np(prev[rows, :D]), 0.3, 0.25, False, store)
        assert_close(to_np(Rs[b].cpu()[rows]), Re, store, f"smoothed R[{b}]", floor_of=Fb)
        assert_close(to_np(Ss[b].cpu()[rows]), Se, "f32", f"smoothed S[{b}]")
    if pad:
        assert float(torch.as_strided(Fh, (B, N, pad), Fh.stride(), D).abs().max()) == 0.0


@pytest.mark.parametrize("dtype,B,N,D,k,pad", [(torch.float32, 1, 16391, 1536, 100, 0), (torch.float32, 3, 4099, 2048, 128, 4)])
def test_wide_float32_slabs_below_3072_channels(dtype, B, N, D, k, pad):
    """The four-chunk slabs at rank 65..128 for widths that have a packed basis and are not the largest."""
    assert pkg.svdcache_has_mfma_path(pkg.make_shape(torch.empty(1, 1024, D, dtype=dtype, device="meta"), k))
    test_wide_float32_slabs_and_full_height_smoothing_tiles(dtype, B, N, D, k, pad)


@pytest.mark.parametrize("B,N,D,k,pad", [(28, 1009, 1152, 32, 0), (19, 751, 1024, 128, 8), (28, 1009, 256, 64, 0)])
def test_full_height_smoothing_tiles_with_single_operands(B, N, D, k, pad):
    """SVDC_FAST smoothing full steps of the sizes that take the tallest tile; ragged last tiles, padded rows, in place."""
    from oracle import ref_full_step_residual_ema
    g = torch.Generator().manual_seed(N + k)
    wide, prev = (torch.randn(N, D + pad, generator=g).to(torch.bfloat16) for _ in range(2))
    V = torch.linalg.qr(torch.randn(D, k, generator=g, dtype=torch.float64))[0].float().contiguous()
    S0 = torch.randn(N, k, generator=g)
    F, R = (t.to(DEV).expand(B, -1, -1).contiguous()[:, :, :D] for t in (wide, prev))
    Vd, S = (t.to(DEV).expand(B, -1, -1).contiguous() for t in (V, S0))
    C = torch.empty_like(S)
    shape = pkg.make_shape(F, k, pkg.SVDC_FAST)
    pkg.svdcache_full_step_residual_ema(shape, F, Vd, pkg.pack_basis(shape, Vd), R, R, S, C, 0.3, 0.25, False)
    torch.cuda.synchronize()
    assert all(torch.equal(t[b], t[0]) for t in (R, S, C) for b in range(1, B))     # the blocks are copies of one
    Rr, Sr, Cr = ref_full_step_residual_ema(to_np(wide[:, :D]), to_np(V), to_np(S0), to_np(prev[:, :D]), 0.3, 0.25, False, "bf16")
    assert_close(to_np(R[0]), Rr, "bf16", "smoothed R", floor_of=to_np(wide[:, :D]), fast=True)
    assert_close(to_np(S[0]), Sr, "bf16", "S", fast=True)
    assert_close(to_np(C[0]), Cr, "bf16", "C", fast=True)


@pytest.mark.parametrize("dtype,B,N,D,k,m", [(torch.bfloat16, 28, 435, 1024, 48, 2), (torch.bfloat16, 4, 1368, 5120, 64, 4),
                                             (torch.bfloat16, 2, 6753, 1920, 128, 3), (torch.float32, 28, 1548, 1920, 96, 2)])
def test_several_states_in_calls_that_fill_the_machine(dtype, B, N, D, k, m):
    """Slabs of one to three chunks are the widest for several states above rank 32: six to sixteen row tiles per workgroup,
    ragged last tiles and groups, with the added tensor and in its place."""
    from oracle import ref_forecast_combine
    store = "f32" if dtype == torch.float32 else "bf16"
    g = torch.Generator().manual_seed(N + k)
    R, X = (torch.randn(N, D, generator=g).to(dtype) for _ in range(2))
    V = torch.linalg.qr(torch.randn(D, k, generator=g, dtype=torch.float64))[0].float().contiguous()
    states = [torch.randn(N, k, generator=g) for _ in range(m)]
    w = [1.5, -0.75, 0.5, -0.25][:m]
    Rd, Xd, Vd, *Sd = (t.to(DEV).expand(B, -1, -1).contiguous() for t in (R, X, V, *states))
    shape = pkg.make_shape(Rd, k)
    packed = pkg.pack_basis(shape, Vd)
    Out = torch.empty_like(Rd)
    pkg.svdcache_forecast_combine(shape, Sd, w, Vd, packed, Rd, None, Out)
    pkg.svdcache_forecast_combine(shape, Sd, w, Vd, packed, Rd, Xd, Xd)
    torch.cuda.synchronize()
    assert all(torch.equal(t[b], t[0]) for t in (Out, Xd) for b in range(1, B))     # the blocks are copies of one
    rows = torch.tensor([0, 1, 15, 16, 95, 96, N // 2, N - 97, N - 17, N - 2, N - 1])
    Rn, Vn, Xn = to_np(R[rows]), to_np(V), to_np(X[rows])
    Sn = [to_np(t[rows]) for t in states]
    for got, added, what in ((Out, None, "without"), (Xd, Xn, "with the added tensor")):
        want = ref_forecast_combine(Sn, w, Vn, Rn, added, store)
        assert_close(to_np(got[0].cpu()[rows]), want, store, what, scale_of=Rn, ulp_of=Rn)


@pytest.mark.parametrize("k", [32, 64, 128])
def test_mfma_inplace_and_strided(k):
    """In-place residual (R aliases F), padded row stride, no coefficient output."""
    B, N, D, ldf = 2, 150, 256, 384
    F, V, S0 = _lowrank_problem(B, N, D, k, seed=11)
    buf = torch.zeros(B, N, ldf, dtype=torch.bfloat16)
    buf[:, :, :D] = F
    for init in (True, False):
        R, S, _, shape, pk = _run_full(buf, D, V, S0, 0.5, init, want_C=False, inplace=True)
        assert pk is not None and shape.ldf == ldf
        state = []
        for b in range(B):
            Rr, Sr, _ = ref_full_step(to_np(F[b]), to_np(V[b]), to_np(S0[b]), 0.5, init, "bf16")
            assert_close(to_np(R[b, :, :D]), Rr, "bf16", "R in place", floor_of=to_np(F[b]))
            assert_close(to_np(S[b]), Sr, "f32", "S")
            state.append((Rr, Sr))
        assert torch.equal(R[:, :, D:].cpu(), buf[:, :, D:])
    pkg.svdcache_forecast(shape, S, V.to(DEV), pk, R[:, :, :D], R[:, :, :D])
    torch.cuda.synchronize()
    for b in range(B):
        assert_close(to_np(R[b, :, :D]), ref_forecast(state[b][1], to_np(V[b]), state[b][0], "bf16"),
                     "bf16", "Fhat in place", scale_of=to_np(F[b]), ulp_of=state[b][0])


@pytest.mark.parametrize("dtype,B,N,D,k,mode", [
    (torch.bfloat16, 2, 200, 256, 32, 0), (torch.bfloat16, 1, 77, 512, 8, 0), (torch.bfloat16, 3, 130, 3072, 64, 0),
    (torch.bfloat16, 1, 145, 3072, 128, 0), (torch.bfloat16, 2, 333, 3072, 20, 1), (torch.bfloat16, 1, 90, 1024, 64, 1),
    (torch.float32, 1, 131, 512, 32, 0), (torch.float32, 1, 70, 3072, 64, 0)])
def test_packed_state_full_step_and_cached_step(dtype, B, N, D, k, mode):
    """The state handed over in the cached step's operand format: svdcache_full_step_packed writes it next to the
    float32 state, svdcache_pack_state makes it from a float32 state, svdcache_forecast_packed reads it.  Against the
    oracle at the usual bars, and bit for bit against the float32-state calls (same arithmetic, fewer conversions)."""
    store = "f32" if dtype == torch.float32 else "bf16"
    Fb, V, S0 = _lowrank_problem(B, N, D, k, seed=N + 3 * k)
    F = Fb.to(dtype)
    Fd, Vd = F.to(DEV), V.to(DEV)
    shape = pkg.make_shape(Fd, k, precision=mode)
    pk = pkg.pack_basis(shape, Vd)
    fast = mode == pkg.SVDC_FAST
    coef = "bf16" if fast else "f32"
    for init in (True, False):
        Sa, Sb = S0.clone().to(DEV), S0.clone().to(DEV)
        Ra, Rb = torch.empty_like(Fd), torch.empty_like(Fd)
        Ca, Cb = torch.empty_like(Sa), torch.empty_like(Sa)
        Sp = pkg.alloc_packed_state(shape, DEV)
        Sp.fill_(0xAB)
        pkg.svdcache_full_step(shape, Fd, Vd, pk, Ra, Sa, Ca, 0.4, init)
        pkg.svdcache_full_step_packed(shape, Fd, Vd, pk, Rb, Sb, Cb, Sp, 0.4, init)
        Fa, Fb2, Fc = torch.empty_like(Fd), torch.empty_like(Fd), torch.empty_like(Fd)
        pkg.svdcache_forecast(shape, Sa, Vd, pk, Ra, Fa)
        pkg.svdcache_forecast_packed(shape, Sp, pk, Rb, Fb2)
        Sp2 = torch.empty_like(Sp)
        pkg.svdcache_pack_state(shape, Sa, Sp2)
        pkg.svdcache_forecast_packed(shape, Sp2, pk, Ra, Fc)
        torch.cuda.synchronize()
        assert torch.equal(Ra, Rb) and torch.equal(Sa, Sb) and torch.equal(Ca, Cb)
        assert torch.equal(Sp, Sp2), "the full step's packed state differs from the packed float32 state"
        assert torch.equal(Fa, Fb2) and torch.equal(Fa, Fc)
        for b in range(B):
            Rr, Sr, _ = ref_full_step(to_np(F[b]), to_np(V[b]), to_np(S0[b]), 0.4, init, store)
            assert_close(to_np(Sb[b]), Sr, coef, f"S[{b}]", fast=fast)
            assert_close(to_np(Fb2[b]), ref_forecast(Sr, to_np(V[b]), Rr, store), store, f"Fhat[{b}] from packed state",
                         fast=fast, scale_of=to_np(F[b]), ulp_of=Rr)
    # a shape without a matrix-core path has no packed state
    odd = pkg.make_shape(torch.zeros(1, 16, 72, device=DEV), 4)
    assert pkg.svdcache_packed_state_bytes(odd) == 0


# ---------------------------------------------------------------------------------------------
# basis fit with the products on the matrix cores (bf16 features, D % 128 == 0, k + p <= 128)
# ---------------------------------------------------------------------------------------------

@pytest.mark.parametrize("N,D,k", [(300, 256, 16), (1000, 512, 32), (600, 3072, 32), (333, 384, 8), (700, 768, 64),
                                   (200, 128, 4), (20, 128, 4), (33, 128, 8), (65, 256, 40), (97, 128, 64)])
def test_fit_basis_mfma_path(N, D, k):
    wl = WORKLOADS["flux1"].with_(N=N, D=D, k=k, signal_rank=min(96, D, N))
    F = torch.stack([FeatureStream(wl, b).at(0) for b in range(2)])
    # at these small sizes the trailing singular values sit in the noise bulk (sigma_{l+1} / sigma_k close
    # to 1), where subspace iteration converges slowly: use more power iterations than the default
    V, sigma, fro2 = pkg.fit_basis(F.to(DEV), k, q=10)
    torch.cuda.synchronize()
    for b in range(2):
        _fit_checks(F[b], V[b], sigma[b], fro2[b], k, "bf16")


@pytest.mark.parametrize("dtype,k,p,rank", [(torch.float32, 50, 50, 55), (torch.float32, 60, 64, 124),
                                             (torch.bfloat16, 56, 56, 60)], ids=["f32-l100", "f32-l124", "bf16-l112"])
def test_fit_basis_wide_sketch_low_rank_features(dtype, k, p, rank):
    """Sketch widths 98..128: the small SVD keeps only one l x l matrix on chip and recovers the right vectors
    from the Cholesky factor at the end.  Features of exact rank < l (float32) make that factor as ill conditioned
    as the diagonal shift allows; the leading k directions must still come out orthonormal and exact."""
    store = "f32" if dtype == torch.float32 else "bf16"
    g = torch.Generator().manual_seed(k * 100 + rank)
    N, D = 400, 256
    left = torch.linalg.qr(torch.randn(N, rank, generator=g, dtype=torch.float64))[0]
    right = torch.linalg.qr(torch.randn(D, rank, generator=g, dtype=torch.float64))[0]
    spec = 10.0 * torch.arange(1, rank + 1, dtype=torch.float64) ** -0.8
    F = ((left * spec) @ right.T).to(dtype).unsqueeze(0).contiguous()
    V, sigma, fro2 = pkg.fit_basis(F.to(DEV), k, p=p, q=4)
    torch.cuda.synchronize()
    _fit_checks(F[0], V[0], sigma[0], fro2[0], k, store)


@pytest.mark.parametrize("dtype,N,D,k,p", [(torch.bfloat16, 600, 512, 96, 0), (torch.float32, 600, 512, 96, 0),
                                            (torch.bfloat16, 700, 384, 128, 0), (torch.float32, 520, 256, 128, 0),
                                            (torch.bfloat16, 450, 640, 100, 29), (torch.float32, 300, 320, 65, 64),
                                            (torch.bfloat16, 300, 256, 50, 50), (torch.float32, 300, 200, 40, 37),
                                            (torch.float32, 260, 384, 65, 65), (torch.bfloat16, 420, 256, 75, 75),
                                            (torch.bfloat16, 139, 256, 70, 70), (torch.float32, 400, 512, 100, 100),
                                            (torch.bfloat16, 500, 384, 110, 113)],
                         ids=["bf16-l192", "f32-l192", "bf16-l256", "f32-l256", "bf16-l129", "f32-l129",
                              "bf16-l100", "f32-l77-general", "f32-l130", "bf16-l150", "bf16-l139", "f32-l200",
                              "bf16-l223"])
def test_fit_basis_sketch_widths_65_to_256(dtype, N, D, k, p):
    """Sketch widths 65..256 (the default oversampling p = k puts every rank 33..128 there, config 5's k = 128
    at l = 256): singular values, captured energy, orthonormality and the leading subspace against the exact
    truncated SVD, for both storage types.  The widths are chosen to hit every branch of the l x l chain: a ragged
    last column block of the Cholesky factorisation and of its application (100 = 64 + 36, 130 = 2 x 64 + 2,
    200 = 3 x 64 + 8), the widest matrix that the single-workgroup Jacobi takes (129..138), and, for the Jacobi by
    column blocks, an odd number of blocks (139 and 150: five, 200 and 223: seven -- one block sits out per step)
    as well as an even one (192: six, 256: eight)."""
    store = "f32" if dtype == torch.float32 else "bf16"
    # full power-law spectrum sigma_i = 10 / i over all min(N, D) directions: no flat noise bulk at rank k, so a
    # few power iterations converge (sigma_{l+1} / sigma_k is about k / l)
    g = torch.Generator().manual_seed(N + D + k)
    r = min(N, D)
    spec = 10.0 / torch.arange(1, r + 1, dtype=torch.float64)
    blocks = []
    for _ in range(2):
        left = torch.linalg.qr(torch.randn(N, r, generator=g, dtype=torch.float64))[0]
        right = torch.linalg.qr(torch.randn(D, r, generator=g, dtype=torch.float64))[0]
        blocks.append(((left * spec) @ right.T).to(dtype))
    F = torch.stack(blocks).contiguous()
    V, sigma, fro2 = pkg.fit_basis(F.to(DEV), k, p=p, q=8)
    torch.cuda.synchronize()
    for b in range(2):
        _fit_checks(F[b], V[b], sigma[b], fro2[b], k, store)


@pytest.mark.parametrize("dtype,B,D,l,more", [
    (torch.float32, 2, 256, 1, 150), (torch.bfloat16, 1, 256, 16, 150), (torch.float32, 1, 200, 17, 150),
    (torch.float32, 1, 384, 63, 150), (torch.bfloat16, 2, 384, 64, 150), (torch.float32, 1, 328, 65, 150),
    (torch.float32, 2, 384, 127, 150), (torch.bfloat16, 1, 384, 129, 150), (torch.float32, 1, 384, 144, 150),
    (torch.float32, 1, 384, 193, 150), (torch.float32, 1, 640, 256, 150),
    # float32 features whose sketch between the two products has its two-part packed form, runs on into the areas behind
    # it (ragged rows), or is too large for them and stays float32 rows (66 columns padded to 128)
    (torch.float32, 1, 256, 128, 2880), (torch.float32, 2, 256, 64, 1937), (torch.float32, 1, 256, 66, 4001)])
def test_fit_basis_at_the_block_edges_of_the_small_matrices(dtype, B, D, l, more):
    """Sketch widths around the 16- and 64-column blocks of the Gram matrix, the factor, its inverse and their application,
    on features whose rank is the sketch width: every direction is found.  float32 values are accurate to the bf16
    high + low split, bf16 ones to the rounding of the features (compared with the exact values of the rounded F)."""
    g = torch.Generator().manual_seed(l)
    N = l + more
    U = torch.linalg.qr(torch.randn(B, N, l, generator=g, dtype=torch.float64))[0]
    W = torch.linalg.qr(torch.randn(B, D, l, generator=g, dtype=torch.float64))[0]
    s = torch.linspace(1.0, 0.3, l, dtype=torch.float64) * 30.0
    F = ((U * s) @ W.transpose(1, 2)).to(dtype)
    V, sigma, fro2, status = pkg.fit_basis(F.to(DEV), l, p=-1, q=2, return_status=True)
    torch.cuda.synchronize()
    assert status.tolist() == [0] * B
    for b in range(B):
        Fb, Vb = to_np(F[b]), to_np(V[b])
        exact = np.linalg.svd(Fb, compute_uv=False)[:l]
        assert np.abs(Vb.T @ Vb - np.eye(l)).max() <= 1e-5
        # bf16: the directions below the rounding noise of F (2^-9 of its entries) are not the sketch's to find
        tol = 1e-4 if dtype == torch.float32 else 2e-2
        assert np.abs(to_np(sigma[b]) / exact - 1).max() <= tol
        assert 1.0 - np.sum((Fb @ Vb) ** 2) / np.sum(exact ** 2) <= tol
        assert abs(float(fro2[b]) / np.sum(Fb * Fb) - 1) <= 1e-5


@pytest.mark.parametrize("l", [2, 3, 4, 5, 8, 9, 12, 15, 24, 25, 32, 33, 41, 49])
@pytest.mark.parametrize("D", [104, 256])       # the general products, and the matrix-core ones (the sketch goes on as operand words)
def test_fit_basis_at_the_widths_of_narrow_sketches(l, D):
    """Panels of 16 columns of the factor and its inverse, whole or padded, 8-column blocks of the Jacobi that are empty or partly
    filled."""
    test_fit_basis_at_the_block_edges_of_the_small_matrices(torch.float32, 2, D, l, 150)


@pytest.mark.parametrize("dtype,B,D,l,N", [
    (torch.float32, 1, 76, 5, 66001), (torch.bfloat16, 1, 136, 40, 65999), (torch.float32, 1, 72, 17, 16401),
    (torch.bfloat16, 2, 200, 33, 9001), (torch.float32, 1, 1028, 16, 33), (torch.float32, 3, 132, 32, 1000),
    (torch.bfloat16, 40, 264, 12, 131), (torch.float32, 1, 264, 136, 4099)])
def test_fit_basis_general_products(dtype, B, D, l, N):
    """The products with F for hidden sizes that are not multiples of 128: workgroups of 128, 32 and 16 rows, one or several
    shares of the tokens, ragged rows, channels (of F and of the 32- and 128-channel pieces) and columns."""
    test_fit_basis_at_the_block_edges_of_the_small_matrices(dtype, B, D, l, N - l)


@pytest.mark.parametrize("dtype,B,D,l,N", [
    (torch.bfloat16, 1, 128, 128, 300), (torch.bfloat16, 2, 384, 100, 1001), (torch.float32, 1, 128, 65, 16385),
    (torch.float32, 1, 640, 128, 515), (torch.bfloat16, 2, 128, 70, 16401)])
def test_fit_basis_products_in_shares_of_the_channels(dtype, B, D, l, N):
    """Sketches of 65 to 128 columns: slabs of 2 and 4 chunks in two shares, the second one with as many, one less or none;
    ragged rows, 16 and 32 per wave, and more of them than the two shares take."""
    test_fit_basis_at_the_block_edges_of_the_small_matrices(dtype, B, D, l, N - l)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16], ids=["f32", "bf16"])
@pytest.mark.parametrize("B,D,l,N", [
    (1, 128, 8, 15), (3, 128, 100, 209),                       # 1 tile per workgroup, waves without channels; an odd number of tiles
    (1, 384, 30, 4801), (2, 256, 64, 4505),                    # 2 and 3 tiles
    (7, 384, 16, 4081), (7, 128, 64, 4081),                    # 4
    (4, 640, 60, 4577), (1, 256, 128, 18417), (1, 384, 9, 18417),    # 5, the last workgroup with fewer
    (1, 128, 33, 22001), (6, 256, 70, 4001),                   # 6
    (20, 128, 12, 3333), (20, 256, 40, 3299), (20, 384, 128, 3333)])  # more tiles than 16 per compute unit
def test_fit_basis_streamed_projections(dtype, B, D, l, N):
    """Every number of row tiles that a workgroup of the streamed projection takes, with ragged rows, an odd last tile (half of the
    last operand word of Y is zero) and fewer chunks of channels than waves; large bf16 calls, which have other kernels."""
    test_fit_basis_at_the_block_edges_of_the_small_matrices(dtype, B, D, min(l, D), N - min(l, D))


@pytest.mark.parametrize("B,N,D,V_digest,sigma_digest", [(130, 512, 1024, "69908a374b01abf9", "62f922c358e915a4"),
                                                         (57, 1200, 3072, "027d9eb40febfd10", "42968fb35e9a79b2")])
def test_large_fits_of_width_64_keep_their_bits(B, N, D, V_digest, sigma_digest):
    """Calls that add nothing with atomics give the same bits every run, and those of bf16 features and width 64 the bits they gave when slabs of
    Q were held in registers (the digests are from that library): the streamed projection adds their channels up in that order."""
    h = torch.arange(B * N * D, device=DEV) * 6364136223846793005 + 1442695040888963407
    h = (h ^ (h >> 29)) * -4658895280553007687
    F = ((h >> 40) & 0xffff).float() / 65536 - 0.5
    F = (F.view(B, N, D) / (1 + torch.arange(D, device=DEV) / 8)).to(torch.bfloat16)
    V, sigma, _ = pkg.fit_basis(F, 32)
    digests = [hashlib.sha256(t.cpu().numpy().tobytes()).hexdigest()[:16] for t in (V, sigma)]
    assert digests == [V_digest, sigma_digest]


@pytest.mark.parametrize("dtype,B,D,l,N", [
    (torch.bfloat16, 1, 128, 12, 513), (torch.bfloat16, 2, 640, 30, 1300), (torch.bfloat16, 5, 1152, 64, 512),
    (torch.bfloat16, 1, 384, 128, 700), (torch.bfloat16, 1, 640, 200, 1029), (torch.float32, 1, 128, 20, 545),
    (torch.float32, 5, 1152, 40, 600), (torch.float32, 1, 384, 100, 1029), (torch.float32, 1, 640, 136, 2017),
    (torch.float32, 22, 768, 80, 514)])
def test_fit_basis_products_in_shares_of_the_rows(dtype, B, D, l, N):
    """Back-projections of small batches: the waves of a workgroup take every fourth step of 32 rows, some of them none; one and
    several groups of rows, one and two column ranges, more slabs than compute units."""
    test_fit_basis_at_the_block_edges_of_the_small_matrices(dtype, B, D, l, N - l)


@pytest.mark.parametrize("B,l", [(2, 48), (1, 80), (2, 81), (1, 96), (2, 112), (1, 113), (3, 128), (1, 208), (1, 209)])
def test_fit_basis_at_the_tile_edges_of_the_factor(B, l):
    """Panels of 16 columns: sketches of 65 to 128 columns are factored as a whole, wider ones by blocks of 64."""
    test_fit_basis_at_the_block_edges_of_the_small_matrices(torch.float32, B, 256, l, 150)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16], ids=["f32", "bf16"])
@pytest.mark.parametrize("N,D,k,rank", [(64, 264, 12, 10), (64, 264, 16, 10), (64, 256, 32, 10), (130, 264, 50, 10), (130, 256, 64, 3),
                                        (150, 264, 69, 10), (210, 256, 100, 10)])
def test_fit_of_many_rank_deficient_blocks(N, D, k, rank, dtype):
    """Features of a rank far below the sketch width: the Gram matrix has `rank` pivots of its own scale and, from somewhere inside
    a panel of the factor on, only those that its shift of 1e-14 leaves, which float64 resolves with a few digits.  A factor
    that loses those (products with an explicit inverse across such a panel) meets a negative pivot in one block of a hundred to a
    thousand and fills it with NaN; here every one of 400 blocks has to come out."""
    B = 400
    g = torch.Generator().manual_seed(N + k)
    left, right = torch.randn(B, N, rank, generator=g), torch.randn(B, rank, D, generator=g)
    F = (left @ right).to(dtype)
    V, sigma, fro2, status = pkg.fit_basis(F.to(DEV), k, return_status=True)
    torch.cuda.synchronize()
    assert torch.isfinite(sigma).all() and torch.isfinite(V).all()
    exact = torch.linalg.svdvals(torch.linalg.qr(left.double())[1] @ torch.linalg.qr(right.double().mT)[1].mT)
    tol = 1e-5 if dtype == torch.float32 else 2e-2
    assert ((sigma[:, :rank].double().cpu() - exact).abs() <= tol * exact[:, :1]).all()
    lead = V[:, :, :rank].double().cpu()
    assert (lead.mT @ lead - torch.eye(rank)).abs().max() <= 1e-5
    if dtype == torch.float32:
        assert (status & pkg.SVDC_FIT_RANK_DEFICIENT).all()


@pytest.mark.parametrize("k,p", [(4, -1), (24, 0), (96, -1), (120, 16),      # the wave Jacobi by width, the one of 129..138 columns,
                                 (96, 64), (128, 72)])                        # and the one by column blocks
@pytest.mark.parametrize("value", [float("nan"), float("-inf")], ids=["nan", "inf"])
def test_fit_writes_every_rank_of_a_block_that_is_not_finite(k, p, value):
    """Norms that compare with nothing still have one rank each: no output of such a block is left unwritten, and the other
    block's fit is not affected."""
    g = torch.Generator().manual_seed(k)
    F = ((torch.randn(2, 200, k, generator=g) * torch.logspace(0, -1, k)) @ torch.randn(2, k, 256, generator=g)).contiguous()
    F[0, 17, 33] = value
    shape = pkg.make_shape(F, k)
    V, sigma = torch.full((2, 256, k), -7.0, device=DEV), torch.full((2, k), -7.0, device=DEV)
    fro2 = torch.empty(2, device=DEV)
    ws = torch.empty(pkg.svdcache_workspace_bytes(shape, p), device=DEV, dtype=torch.uint8)
    pkg.svdcache_fit_basis(shape, F.to(DEV), V, sigma, fro2, ws, p)
    torch.cuda.synchronize()
    assert not (sigma == -7.0).any() and not (V == -7.0).any()
    # (the last pivot of the factor is clamped from below, which replaces a NaN: its value is a zero, ranked last)
    assert not torch.isfinite(sigma[0, 0]) and not torch.isfinite(V[0]).any() and not torch.isfinite(fro2[0])
    _fit_checks(F[1], V[1], sigma[1], fro2[1], k, "f32")


@pytest.mark.parametrize("dtype,N,D,k,p", [(torch.float32, 300, 128, 12, 20), (torch.bfloat16, 400, 256, 24, 40),
                                            (torch.bfloat16, 500, 256, 70, 90)], ids=["f32", "bf16-mfma", "bf16-l160"])
def test_fit_basis_without_power_iterations(dtype, N, D, k, p):
    """q = -1: the orthonormalised Gaussian test matrix goes straight into the Rayleigh-Ritz step.  On features of
    exact rank <= l the sketch then already spans the whole row space, so the result must be the exact decomposition
    (a plain randomized range finder is exact for rank-deficient inputs)."""
    store = "f32" if dtype == torch.float32 else "bf16"
    rank = k + p // 2
    g = torch.Generator().manual_seed(N + k)
    left = torch.linalg.qr(torch.randn(N, rank, generator=g, dtype=torch.float64))[0]
    right = torch.linalg.qr(torch.randn(D, rank, generator=g, dtype=torch.float64))[0]
    spec = 10.0 * torch.arange(1, rank + 1, dtype=torch.float64) ** -0.7
    Fx = (left * spec) @ right.T
    if store == "bf16":
        # bf16 rounding adds a full-rank perturbation of relative size 2^-9: its effect on the leading k values and
        # on the energy they capture is far inside the bf16 bar
        Fx = Fx.to(torch.bfloat16)
    F = Fx.to(dtype).unsqueeze(0).contiguous()
    V, sigma, fro2 = pkg.fit_basis(F.to(DEV), k, p=p, q=-1)
    torch.cuda.synchronize()
    _fit_checks(F[0], V[0], sigma[0], fro2[0], k, store, lead=max(1, k // 4))


def test_fit_status_words():
    """Per-block status of the fit, read from the workspace: 0 for well-conditioned features; the rank-deficiency
    flag for features of exact rank < l (the fitted basis still passes every check); the sweep-cap flag when the
    host allows the small SVD a single sweep (every kernel still runs to its normal end)."""
    g = torch.Generator().manual_seed(77)
    N, D, k = 400, 256, 24
    r_all = min(N, D)                                           # full power-law spectrum: well conditioned
    good = (torch.linalg.qr(torch.randn(N, r_all, generator=g, dtype=torch.float64))[0]
            * (10.0 / torch.arange(1, r_all + 1, dtype=torch.float64))) \
        @ torch.linalg.qr(torch.randn(D, r_all, generator=g, dtype=torch.float64))[0].T
    rank = 30                                                   # < l = 48
    left = torch.linalg.qr(torch.randn(N, rank, generator=g, dtype=torch.float64))[0]
    right = torch.linalg.qr(torch.randn(D, rank, generator=g, dtype=torch.float64))[0]
    low = ((left * (10.0 * torch.arange(1, rank + 1, dtype=torch.float64) ** -0.8)) @ right.T)
    for dtype, store in ((torch.bfloat16, "bf16"), (torch.float32, "f32")):
        # bf16 rounding would make the low-rank block full rank at the 2^-9 level: keep it exactly low rank by
        # building it from bf16-representable factors only in the float32 case
        F = torch.stack([good.to(dtype), low.to(dtype)]).contiguous()
        V, sigma, fro2, status = pkg.fit_basis(F.to(DEV), k, q=6, return_status=True)
        torch.cuda.synchronize()
        status = status.cpu().tolist()
        assert status[0] == 0, f"{store}: well-conditioned block reports {status[0]}"
        _fit_checks(F[0], V[0], sigma[0], fro2[0], k, store)
        if store == "f32":
            assert status[1] == pkg.SVDC_FIT_RANK_DEFICIENT, f"rank-deficient block reports {status[1]}"
            _fit_checks(F[1], V[1], sigma[1], fro2[1], k, store)
        # one sweep is never enough for a 48 x 48 factor: flagged, and nothing else changes for the other flag
        _, _, _, capped = pkg.fit_basis(F.to(DEV), k, q=6, max_sweeps=1, return_status=True)
        torch.cuda.synchronize()
        capped = capped.cpu().tolist()
        assert capped[0] == pkg.SVDC_FIT_JACOBI_CAPPED
        assert capped[1] & pkg.SVDC_FIT_JACOBI_CAPPED
    shape = pkg.make_shape(F.to(DEV), k)
    assert pkg.svdcache_workspace_bytes(shape) == pkg.svdcache_fit_workspace_bytes(shape) > 0
    assert 0 < pkg.svdcache_fit_status_offset(shape) < pkg.svdcache_workspace_bytes(shape)


def test_fit_status_words_column_block_jacobi():
    """The sweep-cap flag of the Jacobi by column blocks (sketch widths above 138), whose convergence is tracked in
    three rotating counters on the device: caps of 1, 2 and 3 sweeps end on each of the three counters and are all
    too few for a 192 x 192 factor (flag set, the call still succeeds and V is orthonormal); the default cap converges
    (no flag) and gives the basis of the exact decomposition."""
    g = torch.Generator().manual_seed(78)
    N, D, k = 500, 256, 96
    r_all = min(N, D)
    blocks = []
    for _ in range(2):
        left = torch.linalg.qr(torch.randn(N, r_all, generator=g, dtype=torch.float64))[0]
        right = torch.linalg.qr(torch.randn(D, r_all, generator=g, dtype=torch.float64))[0]
        blocks.append(((left * (10.0 / torch.arange(1, r_all + 1, dtype=torch.float64))) @ right.T).to(torch.bfloat16))
    F = torch.stack(blocks).contiguous()
    for cap in (1, 2, 3):
        V, _, _, status = pkg.fit_basis(F.to(DEV), k, q=8, max_sweeps=cap, return_status=True)
        torch.cuda.synchronize()
        assert status.cpu().tolist() == [pkg.SVDC_FIT_JACOBI_CAPPED] * 2, f"cap {cap}: {status.cpu().tolist()}"
        Vd = V.double().cpu()
        for b in range(2):
            # columns of L after any number of rotations, normalised: unit norm, but not yet orthogonal
            assert (Vd[b].norm(dim=0) - 1).abs().max() < 1e-3
    V, sigma, fro2, status = pkg.fit_basis(F.to(DEV), k, q=8, return_status=True)
    torch.cuda.synchronize()
    assert status.cpu().tolist() == [0, 0]
    for b in range(2):
        _fit_checks(F[b], V[b], sigma[b], fro2[b], k, "bf16")


def test_fit_basis_flux_block_full_size():
    """One FLUX-shaped block (4608 x 3072 bf16, k = 32) at full size against the exact decomposition."""
    wl = WORKLOADS["flux1"]
    F = FeatureStream(wl, 0, work=torch.float32).at(0).unsqueeze(0)
    V, sigma, fro2 = pkg.fit_basis(F.to(DEV), wl.k)
    torch.cuda.synchronize()
    _fit_checks(F[0], V[0], sigma[0], fro2[0], wl.k, "bf16")


@pytest.mark.parametrize("B,N,D,k", [(2, 200, 256, 32), (1, 150, 3072, 32), (1, 100, 3072, 64), (1, 140, 512, 128)])
def test_mfma_fast_precision_mode_is_within_the_bf16_tolerance(B, N, D, k):
    """SVDC_FAST: single bf16 operands.  Same parity bar (2e-2 for bf16 storage), larger error than
    the default mode."""
    F, V, S0 = _lowrank_problem(B, N, D, k, seed=N + k)
    Fd, Vd = F.to(DEV), V.to(DEV)
    errs = {}
    for mode in (pkg.SVDC_PRECISE, pkg.SVDC_FAST):
        shape = pkg.make_shape(Fd, k, precision=mode)
        pk = pkg.pack_basis(shape, Vd)
        R, S, Cc, Fh = torch.empty_like(Fd), S0.clone().to(DEV), torch.empty(B, N, k, device=DEV), torch.empty_like(Fd)
        pkg.svdcache_full_step(shape, Fd, Vd, pk, R, S, Cc, 0.5, False)
        pkg.svdcache_forecast(shape, S, Vd, pk, R, Fh)
        torch.cuda.synchronize()
        worst = 0.0
        fast = mode == pkg.SVDC_FAST
        for b in range(B):
            Rr, Sr, Cr = ref_full_step(to_np(F[b]), to_np(V[b]), to_np(S0[b]), 0.5, False, "bf16")
            assert_close(to_np(R[b]), Rr, "bf16", f"R[{b}] mode {mode}", floor_of=to_np(F[b]), fast=fast)
            assert_close(to_np(S[b]), Sr, "bf16", f"S[{b}] mode {mode}", fast=fast)
            assert_close(to_np(Cc[b]), Cr, "bf16", f"C[{b}] mode {mode}", fast=fast)
            assert_close(to_np(Fh[b]), ref_forecast(Sr, to_np(V[b]), Rr, "bf16"), "bf16", f"Fhat[{b}] mode {mode}",
                         fast=fast, scale_of=to_np(F[b]), ulp_of=Rr)
            worst = max(worst, rel_err(to_np(R[b]), Rr))
        errs[mode] = worst
    assert errs[pkg.SVDC_PRECISE] <= 3e-3 and errs[pkg.SVDC_FAST] <= 1.5e-2


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16], ids=["f32", "bf16"])
@pytest.mark.parametrize("B,D,l,N", [(1, 128, 36, 4000), (3, 256, 64, 6001), (2, 384, 128, 5003), (1, 264, 50, 3001)])
def test_fit_basis_partial_gram_matrices_in_several_areas(dtype, B, D, l, N):
    """Many more rows than channels: the partial Gram matrices of Y do not fit into one area of the workspace and lie in three
    (the last case has no operand words, so in two), one block's in two of them."""
    test_fit_basis_at_the_block_edges_of_the_small_matrices(dtype, B, D, l, N - l)


@pytest.mark.parametrize("dtype,B,N,D,k,fast,pad", [
    (torch.float32, 1, 37, 5120, 8, 0, 0), (torch.float32, 3, 333, 4096, 40, 0, 8), (torch.float32, 1, 150, 3072, 128, 0, 0),    # 1 tile per workgroup
    (torch.bfloat16, 1, 101, 3072, 100, 0, 64), (torch.float32, 1, 6131, 1152, 68, 0, 0), (torch.bfloat16, 4, 1031, 2560, 96, 0, 0),    # 2
    (torch.bfloat16, 1, 4609, 3072, 64, 0, 0), (torch.float32, 2, 5001, 1920, 128, 0, 0),                                      # 2, 3
    (torch.float32, 7, 2299, 2048, 100, 0, 0), (torch.bfloat16, 4, 4199, 4096, 68, 0, 0),                                       # 4, 5
    (torch.bfloat16, 3, 6001, 1536, 128, 0, 8), (torch.float32, 3, 7297, 512, 128, 0, 0),                                       # 5, 6
    (torch.bfloat16, 5, 5003, 2560, 120, 1, 0)])
def test_full_step_in_two_launches(dtype, B, N, D, k, fast, pad):
    """A full step with a buffer for C may run as a projection and a reconstruction; without one it is a single launch.  Both add up in the
    same order: R, S and the packed state have the same bits, also in place, and C is the oracle's."""
    g = torch.Generator(device=DEV).manual_seed(N + D + k)
    wide = torch.randn(B, N, D + pad, generator=g, device=DEV).to(dtype)
    F = wide[:, :, :D]
    V = torch.linalg.qr(torch.randn(B, D, k, generator=g, device=DEV))[0].contiguous()
    S0 = torch.randn(B, N, k, generator=g, device=DEV)
    shape = pkg.make_shape(F, k, pkg.SVDC_FAST if fast else pkg.SVDC_PRECISE)
    pk = pkg.pack_basis(shape, V)
    one, two, inplace = (torch.zeros_like(wide)[:, :, :D] for _ in range(3))
    for init in (True, False):
        Sa, Sb, Sc = S0.clone(), S0.clone(), S0.clone()
        C, C2 = torch.empty_like(S0), torch.empty_like(S0)
        Spa, Spb = pkg.alloc_packed_state(shape, DEV), pkg.alloc_packed_state(shape, DEV)
        pkg.svdcache_full_step_packed(shape, F, V, pk, one, Sa, None, Spa, 0.3, init)
        pkg.svdcache_full_step_packed(shape, F, V, pk, two, Sb, C, Spb, 0.3, init)
        inplace.copy_(F)
        pkg.svdcache_full_step(shape, inplace, V, pk, inplace, Sc, C2, 0.3, init)
        torch.cuda.synchronize()
        assert torch.equal(one, two) and torch.equal(Sa, Sb) and torch.equal(Spa, Spb)
        assert torch.equal(inplace, two) and torch.equal(Sc, Sb) and torch.equal(C, C2)
    b = B - 1
    ref, _, Cr = ref_full_step(to_np(F[b, -40:]), to_np(V[b]), to_np(S0[b, -40:]), 0.3, False, "f32" if dtype == torch.float32 else "bf16")
    assert_close(to_np(C[b, -40:]), Cr, "bf16" if fast else "f32", f"C[{b}]", fast=bool(fast))


@pytest.mark.parametrize("dtype,B,N,D,k,fast", [(torch_dtype(c[0]), *c[1:6]) for c in TWO_LAUNCHES if c[0:4] in
                                                (("f32", 1, 6131, 1152), ("bf16", 1, 4609, 3072), ("bf16", 5, 5003, 2560))])
def test_rows_that_are_not_finite_stay_by_themselves_in_both_forms_of_the_full_step(dtype, B, N, D, k, fast):
    """An infinity or a NaN in a row of F: nothing of R is finite in that row, with a buffer for C (two launches) and without (one), C and S are the
    same in both, and all other rows keep the bits that they have without it.  C may also be the buffer S."""
    g = torch.Generator(device=DEV).manual_seed(N + k)
    F = torch.randn(B, N, D, generator=g, device=DEV).to(dtype)
    V = torch.linalg.qr(torch.randn(B, D, k, generator=g, device=DEV))[0].contiguous()
    S0 = torch.randn(B, N, k, generator=g, device=DEV)
    shape = pkg.make_shape(F, k, pkg.SVDC_FAST if fast else pkg.SVDC_PRECISE)
    pk = pkg.pack_basis(shape, V)

    def step(F, with_C):
        R, S, C = torch.empty_like(F), S0.clone(), torch.empty_like(S0) if with_C else None
        pkg.svdcache_full_step(shape, F, V, pk, R, S, C, 0.3, False)
        return R, S, C
    clean, S_clean, C_clean = step(F, True)
    alone = S0.clone()
    pkg.svdcache_full_step(shape, F, V, pk, torch.empty_like(F), alone, alone, 0.3, False)
    assert torch.equal(alone, C_clean)
    bad = [(0, 0), (0, 17), (B - 1, N // 2), (B - 1, N - 1)]
    for i, (b, n) in enumerate(bad):
        F[b, n, (331 * i) % D] = (float("inf"), float("nan"), float("-inf"), float("inf"))[i]
    R1, S1, _ = step(F, False)
    R2, S2, C2 = step(F, True)
    rows = torch.zeros(B, N, dtype=torch.bool, device=DEV)
    for b, n in bad:
        rows[b, n] = True
    for R in (R1, R2):
        assert not torch.isfinite(R[rows].float()).any() and torch.equal(R[~rows], clean[~rows])
    assert torch.equal(S1.nan_to_num(7.0), S2.nan_to_num(7.0)) and torch.equal(S2[~rows], S_clean[~rows])
    assert not torch.isfinite(C2[rows]).any() and torch.equal(C2[~rows], C_clean[~rows])


@pytest.mark.parametrize("dtype,B,N,D,k,fast,pad", [
    (torch.float32, 1, 6150, 3072, 32, 0, 0), (torch.float32, 3, 2777, 1920, 20, 0, 8), (torch.float32, 2, 13001, 256, 8, 0, 0),      # slabs of 6, 5, 2
    (torch.float32, 1, 4403, 3072, 64, 0, 0), (torch.float32, 2, 3333, 2048, 40, 0, 64),                                       # 3, 4
    (torch.float32, 1, 3333, 3072, 128, 0, 0), (torch.float32, 3, 4111, 1152, 100, 0, 0), (torch.float32, 1, 77, 1536, 64, 0, 0),
    (torch.bfloat16, 1, 12100, 3072, 16, 0, 0), (torch.bfloat16, 3, 6007, 1152, 32, 0, 8),                                     # 6 and 12, 3
    (torch.bfloat16, 2, 5003, 2560, 64, 0, 0), (torch.bfloat16, 1, 9007, 3072, 52, 0, 0), (torch.bfloat16, 5, 5555, 256, 48, 0, 0),   # 4 and 5, 4, 2
    (torch.bfloat16, 1, 5001, 3072, 128, 0, 0), (torch.bfloat16, 3, 5003, 1152, 72, 0, 64), (torch.bfloat16, 1, 129, 3072, 128, 0, 0),
    (torch.bfloat16, 1, 7001, 3072, 64, 1, 0), (torch.bfloat16, 2, 6001, 2048, 48, 1, 0),                                      # 6, 8
    (torch.bfloat16, 1, 9001, 3072, 64, 1, 0), (torch.bfloat16, 2, 50003, 3072, 40, 1, 0),                                     # between and beyond the unshared slabs of 12
    (torch.bfloat16, 2, 4999, 2560, 100, 1, 8), (torch.bfloat16, 1, 5005, 1920, 128, 1, 0)])
def test_cached_steps_share_their_coefficients(dtype, B, N, D, k, fast, pad):
    """The waves of a workgroup load and convert a quarter of a row tile's coefficients each and pass the operands on: plain and packed
    state, 2 to 4 states with and without an added tensor, in place.  Every element against float64, and the same bits as a call
    of the last rows alone, whose workgroups have one row tile or share nothing.
    Bound: bf16 has 8 bits, so a coefficient or a basis element is off by 2^-8 of itself as one bf16, by 2^-16 as two (a high and a low part); two
    such factors, and the dropped low x low product, make 2^-7 (1 + 2^-9) or 3 x 2^-16; weighting and adding up in float32 at most (k + 8) 2^-24 < 2^-16 of
    sum |w s v|; then the sum with R and X and the storage rounding."""
    g = torch.Generator(device=DEV).manual_seed(N + D + k)
    wide = torch.randn(B, N, D + pad, generator=g, device=DEV).to(dtype)
    R = wide[:, :, :D]
    X = torch.randn(B, N, D + pad, generator=g, device=DEV).to(dtype)[:, :, :D]
    V = (torch.randn(B, D, k, generator=g, device=DEV) / D ** 0.5).contiguous()
    S = [torch.randn(B, N, k, generator=g, device=DEV) for _ in range(4)]
    shape = pkg.make_shape(R, k, pkg.SVDC_FAST if fast else pkg.SVDC_PRECISE)
    pk = pkg.pack_basis(shape, V)
    n0 = N - min(N, k + 13)
    tail = [s[-1:, n0:].contiguous() for s in S]
    tshape, tpk = pkg.make_shape(R[-1:, n0:], k, pkg.SVDC_FAST if fast else pkg.SVDC_PRECISE), pkg.pack_basis(shape, V)[-pk.numel() // B:]
    unit = 2.0 ** -8 if dtype == torch.bfloat16 else 2.0 ** -24
    product = (2.0 ** -7 * (1 + 2.0 ** -9) if fast and k > 32 else 3 * 2.0 ** -16) + 2.0 ** -16
    empty = lambda: torch.empty_like(wide)[:, :, :D]
    for w, x in (([1.0], False), ([1.5, -0.5], True), ([2.0, -1.0], False), ([0.5, 0.25, -1.25], True), ([0.5, 0.25, -1.25, 2.0], False)):
        out, again, part = empty(), empty(), empty()[-1:, n0:]
        if len(w) == 1:
            pkg.svdcache_forecast(shape, S[0], V, pk, R, out)
            pkg.svdcache_forecast(tshape, tail[0], V[-1:], tpk, R[-1:, n0:], part)
            Sp = pkg.alloc_packed_state(shape, DEV)
            pkg.svdcache_pack_state(shape, S[0], Sp)
            pkg.svdcache_forecast_packed(shape, Sp, pk, R, again)
        else:
            m = len(w)
            pkg.svdcache_forecast_combine(shape, S[:m], w, V, pk, R, X if x else None, out)
            pkg.svdcache_forecast_combine(tshape, tail[:m], w, V[-1:], tpk, R[-1:, n0:], X[-1:, n0:] if x else None, part)
            again.copy_(X if x else R)
            pkg.svdcache_forecast_combine(shape, S[:m], w, V, pk, R if x else again, again if x else None, again)
        torch.cuda.synchronize()
        assert torch.equal(out, again) and torch.equal(out[-1:, n0:], part), (w, x)
        for b in range(B):
            c, size = sum(wi * s[b].double() for wi, s in zip(w, S)), sum(abs(wi) * s[b].double().abs() for wi, s in zip(w, S))
            added = X[b].double() if x else 0.0
            want = c @ V[b].double().T + R[b].double() + added
            size = size @ V[b].double().abs().T
            bound = product * size + 2.0 ** -22 * (size + R[b].double().abs() + abs(added))
            bound = bound + unit * (want.abs() + bound) + 1e-30
            worst = float(((out[b].double() - want).abs() / bound).max())
            assert worst <= 1.0, (w, x, b, worst)


@pytest.mark.parametrize("B,N,D,k,pad", [(1, 85001, 3072, 24, 0), (8, 5206, 1536, 8, 8)])
def test_cached_steps_that_add_a_tensor_in_wide_slabs(B, N, D, k, pad):
    """Two states in a long call, three in three rounds of the narrower slabs: slabs of 12 chunks whose waves share nothing."""
    test_cached_steps_share_their_coefficients(torch.bfloat16, B, N, D, k, 0, pad)


@pytest.mark.parametrize("B,N,D,k", [(1, 308009, 512, 4), (2, 38407, 2048, 16)])
def test_long_cached_steps_of_two_states_that_do_not_share(B, N, D, k):
    """Rows of a power of two of channels, rank <= 16."""
    test_cached_steps_share_their_coefficients(torch.bfloat16, B, N, D, k, 0, 0)


@pytest.mark.parametrize("B,N,D,k", [(1, 273, 1152, 48), (1, 304, 256, 36), (2, 404, 512, 124), (1, 336, 512, 40), (1, 257, 1920, 128)])
def test_short_cached_steps_of_several_float32_states(B, N, D, k):
    """Slabs of one chunk in the place of 2, 3 or 4."""
    test_cached_steps_share_their_coefficients(torch.float32, B, N, D, k, 0, 0)


@pytest.mark.parametrize("B,N,k", [(4, 4090, 32), (4, 3060, 64), (2, 4090, 128)])
def test_full_step_tiles_with_a_row_tile_in_lds(B, N, k):
    """3072 channels and one round of 256 or more workgroup tiles, each block ending in a partly filled tile.  At
    rank 64 these are the launches that keep the third row tile of a workgroup tile in LDS (both operand modes);
    ranks 32 and 128 run the register-only tiles at the same sizes.  Every element is compared, out of place and
    in place (R aliases F), with and without the coefficient output."""
    D = 3072
    F, V, S0 = _lowrank_problem(B, N, D, k, seed=N + k)
    ref = [ref_full_step(to_np(F[b]), to_np(V[b]), to_np(S0[b]), 0.3, False, "bf16") for b in range(B)]
    Vd = V.to(DEV)
    for mode in (pkg.SVDC_PRECISE, pkg.SVDC_FAST):
        coef = "f32" if mode == pkg.SVDC_PRECISE else "bf16"
        fast = mode == pkg.SVDC_FAST
        for inplace in (False, True):
            Fd = F.to(DEV)
            shape = pkg.make_shape(Fd, k, precision=mode)
            pk = pkg.pack_basis(shape, Vd)
            R = Fd if inplace else torch.full_like(Fd, 7.0)
            S = S0.clone().to(DEV)
            Cc = None if inplace else torch.empty(B, N, k, device=DEV)
            pkg.svdcache_full_step(shape, Fd, Vd, pk, R, S, Cc, 0.3, False)
            torch.cuda.synchronize()
            for b in range(B):
                Rr, Sr, Cr = ref[b]
                assert_close(to_np(R[b]), Rr, "bf16", f"R[{b}] mode {mode} inplace {inplace}", floor_of=to_np(F[b]),
                             fast=fast)
                assert_close(to_np(S[b]), Sr, coef, f"S[{b}] mode {mode}", fast=fast)
                if Cc is not None:
                    assert_close(to_np(Cc[b]), Cr, coef, f"C[{b}] mode {mode}", fast=fast)
                assert rel_err(to_np(R[b]), Rr) <= (3e-3 if mode == pkg.SVDC_PRECISE else 1.5e-2)


# ---------------------------------------------------------------------------------------------
# full-size launches (the configurations bench.py times), checked on sampled rows
# ---------------------------------------------------------------------------------------------

def _full_size_fit_check(F_block, V_b, sigma_b, fro2_b, k, store):
    """The fitted basis of one full-size block against the exact truncated SVD (Sec. 3.2, Eq. 4-5; the oracle takes
    the Gram route at these sizes): singular values, the energy the fitted directions capture relative to the
    optimum, and that the reported sigma_j are the norms of F v_j.  Unlike "the cached step right after the first
    full step returns F", which holds for any orthonormal V, these say WHICH subspace was found.

    Subspace iteration with a sketch of width l and q applications of F^T F finds sigma_j to a relative error of
    about (sigma_{l+1} / sigma_j)^(2 (2q + 1)): the values above the flat bulk of the synthetic residual are compared
    at the parity bar, those inside it (where sigma_{l+1} / sigma_j is close to one and no number of iterations
    separates them: rank 64 of the FLUX-shaped stream) by what still holds there -- a Rayleigh-Ritz value never
    exceeds the exact one, and the energy captured by all k directions is within 1e-3 of the optimum."""
    tol = TOL[store]
    Fd = to_np(F_block)
    l = min(2 * k, min(Fd.shape), 256)                  # the fit's defaults: p = k, q = 3 (bf16) / 5 (f32)
    q = 3 if store == "bf16" else 5
    _, s_more, fr = ref_fit_basis(Fd, min(l + 1, min(Fd.shape)))
    sr = s_more[:k]
    Vg, sg = to_np(V_b), to_np(sigma_b)
    assert np.abs(Vg.T @ Vg - np.eye(k)).max() <= 1e-5
    conv = (s_more[-1] / sr) ** (2 * (2 * q + 1)) if l + 1 <= min(Fd.shape) else np.zeros(k)
    err = np.abs(sg / sr - 1)
    resolved = 30 * conv <= tol
    assert resolved[: max(1, k // 2)].all(), "the leading half of the spectrum must be resolvable at the default q"
    assert err[resolved].max() <= tol, f"sigma rel err {err[resolved].max():.2e} on the resolved values"
    assert np.all(sg <= sr * (1 + 1e-5)) and np.all(sg >= 0.8 * sr), f"sigma outside [0.8, 1] x exact: {err.max():.2e}"
    assert abs(float(fro2_b) / fr - 1) <= 1e-5
    proj = Fd @ Vg
    deficit = 1 - np.sum(proj ** 2) / np.sum(sr ** 2)
    assert deficit <= 1e-3, f"captured-energy deficit {deficit:.2e}"      # measured: a few 1e-6 at the default q
    assert np.abs(np.linalg.norm(proj, axis=0) / sg - 1).max() <= 1e-4


def _sampled_row_parity(wl, B, blocks_to_check, n_rows, precision=0, fit_check_block=None):
    """Run fit + pack + two full steps + one cached step at full size on GPU-generated features and
    recompute sampled token rows with the oracle (rows are independent given V and S).  Nothing the GPU
    computed is handed to the oracle: it gets the generated features, the generator's basis and its own state."""
    store = wl.dtype
    feats = [torch.empty(B, wl.N, wl.D, device=DEV, dtype=torch_dtype(store)) for _ in range(2)]
    Vgen = torch.empty(B, wl.D, wl.k, device=DEV)
    for b in range(B):
        fs = FeatureStream(wl, b, device=DEV)
        feats[0][b], feats[1][b] = fs.at(0), fs.at(wl.interval)
        Vgen[b] = fs.V[:, :wl.k].float()          # the generator's leading directions: the basis of both sides
        del fs
    shape = pkg.make_shape(feats[0], wl.k, precision=precision)
    assert pkg.svdcache_has_mfma_path(shape)
    R = torch.empty_like(feats[0])
    S = torch.empty(B, wl.N, wl.k, device=DEV)
    Cc = torch.empty_like(S)
    Fh = torch.empty_like(R)
    # fit + pack + step with the FITTED basis, checked by an identity that needs no oracle: right after the
    # first full step the cached step gives the feature back (up to the rounding of R and Fhat)
    V, sigma, fro2 = pkg.fit_basis(feats[0], wl.k)
    pk = pkg.pack_basis(shape, V)
    pkg.svdcache_full_step(shape, feats[0], V, pk, R, S, None, wl.alpha, True)
    pkg.svdcache_forecast(shape, S, V, pk, R, Fh)
    torch.cuda.synchronize()
    back = 1e-5 if store == "f32" else (6e-3 if precision == 0 else 2e-2)
    for b in blocks_to_check:
        Vb = to_np(V[b])
        assert np.abs(Vb.T @ Vb - np.eye(wl.k)).max() <= 1e-5
        assert rel_err(to_np(Fh[b][:512]), to_np(feats[0][b][:512])) <= back
    if fit_check_block is not None:
        b = fit_check_block
        _full_size_fit_check(feats[0][b], V[b], sigma[b], fro2[b], wl.k, store)
    # parity of the steps against the oracle, both sides on the generator's basis
    pk = pkg.pack_basis(shape, Vgen)
    pkg.svdcache_full_step(shape, feats[0], Vgen, pk, R, S, None, wl.alpha, True)
    S0 = S.clone()
    pkg.svdcache_full_step(shape, feats[1], Vgen, pk, R, S, Cc, wl.alpha, False)
    pkg.svdcache_forecast(shape, S, Vgen, pk, R, Fh)
    # the same two calls with the state handed over in packed form: identical results at full size
    Sp = pkg.alloc_packed_state(shape, DEV)
    S2, R2, Fh2 = S0.clone(), torch.empty_like(R), torch.empty_like(R)
    pkg.svdcache_full_step_packed(shape, feats[1], Vgen, pk, R2, S2, None, Sp, wl.alpha, False)
    pkg.svdcache_forecast_packed(shape, Sp, pk, R2, Fh2)
    torch.cuda.synchronize()
    for b in blocks_to_check:
        assert torch.equal(S2[b], S[b]) and torch.equal(R2[b], R[b]) and torch.equal(Fh2[b], Fh[b])
    del S2, R2, Fh2, Sp
    g = torch.Generator().manual_seed(wl.config_id)
    fast = precision != 0
    for b in blocks_to_check:
        assert torch.isfinite(R[b].float()).all() and torch.isfinite(Fh[b].float()).all() and torch.isfinite(S[b]).all()
        rows = torch.cat([torch.tensor([0, 1, 15, 16, 31, 32, wl.N - 17, wl.N - 16, wl.N - 1]),
                          torch.randint(0, wl.N, (n_rows,), generator=g)]).unique()
        Vb = to_np(Vgen[b])
        F0r, F1r = to_np(feats[0][b][rows]), to_np(feats[1][b][rows])
        _, S0r, _ = ref_full_step(F0r, Vb, None, wl.alpha, True, store)
        coef_store = "f32" if precision == 0 else "bf16"   # SVDC_FAST rounds V to bf16 in the projection
        assert_close(to_np(S0[b][rows]), S0r, coef_store, f"S after init, block {b}", fast=fast)
        Rr, S1r, C1r = ref_full_step(F1r, Vb, S0r, wl.alpha, False, store)       # the oracle's own state
        assert_close(to_np(R[b][rows]), Rr, store, f"R block {b}", floor_of=F1r, fast=fast)
        assert_close(to_np(S[b][rows]), S1r, coef_store, f"S block {b}", fast=fast)
        assert_close(to_np(Cc[b][rows]), C1r, coef_store, f"C block {b}", fast=fast)
        Fr = ref_forecast(S1r, Vb, Rr, store)
        assert_close(to_np(Fh[b][rows]), Fr, store, f"Fhat block {b}", fast=fast, scale_of=F1r, ulp_of=Rr)
    return sigma, fro2, feats


def test_flux57_full_size_launch_sampled_rows():
    """Config 3 as bench.py launches it: 57 blocks x 4608 x 3072 bf16, k = 32, one launch per kernel."""
    wl = WORKLOADS["flux57"]
    sigma, fro2, feats = _sampled_row_parity(wl, wl.B, blocks_to_check=[0, 28, 56], n_rows=96)
    # the fitted singular values of one block against the exact ones
    _, sr, fr = ref_fit_basis(to_np(feats[0][56]), wl.k)
    assert np.abs(to_np(sigma[56]) / sr - 1).max() <= TOL["bf16"]
    assert abs(float(fro2[56]) / fr - 1) <= 1e-5


@pytest.mark.parametrize("k", [16, 64])
def test_flux57_full_size_launch_other_ranks(k):
    """Config 3 lists the ranks 16, 32 and 64: the same 57-block launches at the other two ranks (rank 64 runs the
    full step with 48-row tiles whose third row tile sits in LDS, over 22 rounds of the persistent grid)."""
    wl = WORKLOADS["flux57"].with_(k=k)
    _sampled_row_parity(wl, wl.B, blocks_to_check=[0, 31, 56], n_rows=64, fit_check_block=31)


def test_flux57_full_size_launch_fast_mode():
    wl = WORKLOADS["flux57"].with_(B=8)
    _sampled_row_parity(wl, wl.B, blocks_to_check=[0, 7], n_rows=64, precision=pkg.SVDC_FAST)


def test_hunyuan_shape_offsets_beyond_2_to_31_sampled_rows():
    """Config 4 shape (119056 tokens x 3072, k = 64) on 7 of its 60 blocks: the last block starts 2.19e9 elements
    (4.4e9 bytes) into the tensors, beyond what 32-bit element or byte offsets reach.  First and last block are
    compared with the oracle on sampled rows; the fitted basis of the last block against the exact decomposition."""
    wl = WORKLOADS["hyv60"]
    assert 6 * wl.N * wl.D > 2 ** 31
    _sampled_row_parity(wl, 7, blocks_to_check=[0, 6], n_rows=96, fit_check_block=6)


def test_hunyuan_60_block_launch_first_middle_and_last_block():
    """Config 4 at its real size, the launch bench.py times: 60 blocks x 119056 x 3072 bf16 (43.9 GB per tensor),
    k = 64.  Blocks 0 and 59 hold generated features; to keep the generation short the blocks between hold copies
    of them (even blocks of block 0, odd ones of block 59) with the matching basis.  Sampled rows of the first
    and last block are recomputed by the oracle; a middle block must equal, bit for bit, the block it copies (every
    element of it is thereby compared with a block whose rows were sampled against the oracle)."""
    wl = WORKLOADS["hyv60"]
    B, N, D, k = wl.B, wl.N, wl.D, wl.k
    F = torch.empty(B, N, D, device=DEV, dtype=torch.bfloat16)
    Vgen = torch.empty(B, D, k, device=DEV)
    for b in (0, B - 1):
        fs = FeatureStream(wl, b, device=DEV)
        F[b] = fs.at(0)
        Vgen[b] = fs.V[:, :k].float()
        del fs
    for b in range(1, B - 1):
        src = 0 if b % 2 == 0 else B - 1
        F[b].copy_(F[src])
        Vgen[b].copy_(Vgen[src])
    shape = pkg.make_shape(F, k)
    pk = pkg.pack_basis(shape, Vgen)
    R = torch.empty_like(F)
    S = torch.empty(B, N, k, device=DEV)
    pkg.svdcache_full_step(shape, F, Vgen, pk, R, S, None, wl.alpha, True)
    torch.cuda.synchronize()
    mid = 30
    assert torch.equal(R[mid], R[0]) and torch.equal(S[mid], S[0])
    assert torch.equal(R[mid + 1], R[B - 1]) and torch.equal(S[mid + 1], S[B - 1])
    g = torch.Generator().manual_seed(wl.config_id + 60)
    ref = {}
    for b in (0, B - 1):
        rows = torch.cat([torch.tensor([0, 15, 16, 47, 48, N - 17, N - 1]),
                          torch.randint(0, N, (64,), generator=g)]).unique()
        Fr = to_np(F[b][rows])
        Rr, Sr, _ = ref_full_step(Fr, to_np(Vgen[b]), None, wl.alpha, True, "bf16")
        assert_close(to_np(R[b][rows]), Rr, "bf16", f"R block {b}", floor_of=Fr)
        assert_close(to_np(S[b][rows]), Sr, "f32", f"S block {b}")
        ref[b] = (rows, Fr, Rr, Sr)
    # the cached step in place (Fhat takes the buffer of R), same launch size
    pkg.svdcache_forecast(shape, S, Vgen, pk, R, R)
    torch.cuda.synchronize()
    assert torch.equal(R[mid], R[0]) and torch.equal(R[mid + 1], R[B - 1])
    for b in (0, B - 1):
        rows, Fr, Rr, Sr = ref[b]
        assert_close(to_np(R[b][rows]), ref_forecast(Sr, to_np(Vgen[b]), Rr, "bf16"), "bf16", f"Fhat block {b}",
                     scale_of=Fr, ulp_of=Rr)


def test_rank_sweep_at_stacked_prompt_shape():
    """Config 5 shape: 4 prompts stacked along N with one shared basis, k in {16, 64, 128}."""
    for k in (16, 64, 128):
        wl = WORKLOADS["sweep"].with_(k=k)
        _sampled_row_parity(wl, 1, blocks_to_check=[0], n_rows=64)


@pytest.mark.parametrize("k", [8, 32, 128])
def test_rank_sweep_float32_at_stacked_prompt_shape(k):
    """The float32 half of config 5 at its real size (18432 x 3072): the matrix-core kernels with float32 features
    split into bf16 high + low parts on the fly, sampled rows against the oracle at the float32 bar."""
    wl = WORKLOADS["sweep"].with_(k=k, dtype="f32")
    _sampled_row_parity(wl, 1, blocks_to_check=[0], n_rows=64, fit_check_block=0 if k == 32 else None)


# ---------------------------------------------------------------------------------------------
# float32 features on the matrix cores (operands split into bf16 high + low parts)
# ---------------------------------------------------------------------------------------------

@pytest.mark.parametrize("B,N,D,k", [(2, 200, 256, 32), (1, 77, 512, 8), (1, 131, 512, 128), (1, 150, 3072, 32),
                                     (1, 70, 3072, 64), (2, 49, 256, 20), (1, 60, 1024, 32), (1, 50, 1536, 16),
                                     (1, 70, 2048, 64), (1, 40, 4096, 32), (1, 50, 1152, 32), (1, 70, 1920, 64),
                                     (1, 40, 2560, 16), (1, 36, 5120, 32), (1, 129, 5120, 128)])
def test_mfma_float32_features(B, N, D, k):
    Fb, V, S0 = _lowrank_problem(B, N, D, k, seed=N * 3 + k)
    g = torch.Generator().manual_seed(N)
    F = Fb.float() + 1e-3 * torch.randn(B, N, D, generator=g)      # not bf16-representable
    shape = pkg.make_shape(F, k)
    assert pkg.svdcache_has_mfma_path(shape)
    for init in (True, False):
        R, S, Cc, shape, pk = _run_full(F, D, V, S0, 0.5, init)
        assert pk is not None
        Fh = torch.empty_like(R)
        pkg.svdcache_forecast(shape, S, V.to(DEV), pk, R, Fh)
        torch.cuda.synchronize()
        for b in range(B):
            Rr, Sr, Cr = ref_full_step(to_np(F[b]), to_np(V[b]), to_np(S0[b]), 0.5, init, "f32")
            assert_close(to_np(R[b]), Rr, "f32", f"R[{b}]", floor_of=to_np(F[b]))
            assert_close(to_np(S[b]), Sr, "f32", f"S[{b}]")
            assert_close(to_np(Cc[b]), Cr, "f32", f"C[{b}]")
            Fr = ref_forecast(Sr, to_np(V[b]), Rr, "f32")       # the oracle's own state
            assert_close(to_np(Fh[b]), Fr, "f32", f"Fhat[{b}]", scale_of=to_np(F[b]))


def test_step_kernels_are_bitwise_deterministic():
    """No atomics on the output path of the step kernels: two runs on the same inputs give the same bits
    (matrix-core path at FLUX width and the general path)."""
    for (B, N, D, k) in [(3, 300, 3072, 32), (2, 130, 200, 17)]:
        Fbuf, V, S0 = _rand_problem(B, N, D, k, torch.bfloat16, seed=N)
        runs = []
        for _ in range(2):
            R, S, Cc, shape, pk = _run_full(Fbuf, D, V, S0, 0.4, False)
            Fh = torch.empty_like(R)
            pkg.svdcache_forecast(shape, S, V.to(DEV), pk, R, Fh)
            torch.cuda.synchronize()
            runs.append((R.clone(), S.clone(), Cc.clone(), Fh.clone()))
        for a, b in zip(*runs):
            assert torch.equal(a, b)


def test_flux57_fit_is_bitwise_reproducible():
    """At the batch size of the benchmark no step of the fit sums in an order that depends on scheduling
    (back-projection with one row group per block, Gram matrices from ordered partial sums): two fits of the
    same features give the same basis, bit for bit."""
    wl = WORKLOADS["flux57"]
    F = torch.empty(wl.B, wl.N, wl.D, device=DEV, dtype=torch.bfloat16)
    for b in range(wl.B):
        F[b] = FeatureStream(wl, b, device=DEV).at(0)
    V1, s1, _ = pkg.fit_basis(F, wl.k)
    V2, s2, _ = pkg.fit_basis(F, wl.k)
    torch.cuda.synchronize()
    assert torch.equal(V1, V2) and torch.equal(s1, s2)


def test_flux_block_trajectory_against_a_free_running_oracle():
    """Config 2 (one FLUX-sized block, bf16, k = 32, full step every 5) over 16 timesteps on the matrix-core
    path.  The oracle keeps its OWN state on 80 sampled token rows (rows are independent given V), so errors of
    the GPU path would have to stay small over four EMA updates, not just within one call."""
    wl = WORKLOADS["flux1"].with_(T=16)
    fs = FeatureStream(wl, 0, device=DEV)
    F0 = fs.at(0).unsqueeze(0).contiguous()
    shape = pkg.make_shape(F0, wl.k)
    V = fs.V[:, :wl.k].float().unsqueeze(0).contiguous()          # the generator's leading directions
    pk = pkg.pack_basis(shape, V)
    assert pk is not None
    Vn = to_np(V[0])
    rows = torch.cat([torch.tensor([0, 15, 16, 47, 48, wl.N - 1]),
                      torch.randint(0, wl.N, (74,), generator=torch.Generator().manual_seed(4))]).unique()
    R = torch.empty_like(F0)
    S = torch.empty(1, wl.N, wl.k, device=DEV)
    Fh = torch.empty_like(F0)
    Rr = Sr = None
    for t in range(wl.T):
        if is_full_step(t, wl.interval):
            Ft = fs.at(t).unsqueeze(0).contiguous()
            pkg.svdcache_full_step(shape, Ft, V, pk, R, S, None, wl.alpha, t == 0)
            torch.cuda.synchronize()
            Frows = to_np(Ft[0][rows])
            Rr, Sr, _ = ref_full_step(Frows, Vn, Sr, wl.alpha, t == 0, "bf16")
            assert_close(to_np(R[0][rows]), Rr, "bf16", f"t={t} R", floor_of=Frows)
            assert_close(to_np(S[0][rows]), Sr, "f32", f"t={t} S")
        else:
            pkg.svdcache_forecast(shape, S, V, pk, R, Fh)
            torch.cuda.synchronize()
            assert_close(to_np(Fh[0][rows]), ref_forecast(Sr, Vn, Rr, "bf16"), "bf16", f"t={t} Fhat", scale_of=Frows,
                         ulp_of=Rr)


@pytest.mark.parametrize("dtype,D,k", [(torch.float32, 64, 8), (torch.bfloat16, 256, 32)])
def test_step_calls_by_both_routes_of_the_binding(dtype, D, k, monkeypatch):
    """The compiled step calls and the ctypes ones make the same calls, on the current stream, and refuse the same arguments
    with the same errors: other strides, types, sizes and devices, buffers that are too small, numbers out of range."""
    from paper_2601_07396_amd import binding
    pkg.load_library()
    fast = binding._fast
    assert fast is not None
    answers = {}                                     # what the module said, by function: 0 made, None not ordinary

    class Recorder:
        def __getattr__(self, name):
            def call(*args):
                answers.setdefault(name, []).append(getattr(fast, name)(*args))
                return answers[name][-1]
            return call

    monkeypatch.setattr(binding, "_fast", Recorder())
    B, N = 2, 50
    Fbuf, V, S0 = _rand_problem(B, N, D, k, dtype, seed=D)
    F, V, Rp = Fbuf.to(DEV), V.to(DEV), Fbuf.flip(1).contiguous().to(DEV)
    shape = pkg.make_shape(F, k)
    packed = pkg.pack_basis(shape, V)
    Sp = pkg.alloc_packed_state(shape, F.device) if packed is not None else None

    def good():
        S, Cc, R, Fh = S0.to(DEV), torch.empty(B, N, k, device=DEV), torch.empty_like(F), torch.empty_like(F)
        out = []
        pkg.svdcache_full_step(shape, F, V, packed, R, S, Cc, 0.3, False)
        pkg.svdcache_forecast(shape, S, V, packed, R, Fh)
        out += [R.clone(), S.clone(), Cc, Fh.clone()]
        pkg.svdcache_full_step_residual_ema(shape, F, V, packed, Rp, R, S, None, 0.5, 0.25, False)
        pkg.svdcache_forecast_combine(shape, [S, Cc], [1.5, -0.5], V, packed, R, F, Fh)
        out += [R.clone(), S.clone(), Fh.clone()]
        if Sp is not None:
            pkg.svdcache_full_step_packed(shape, F, V, packed, R, S, None, Sp, 0.5, False)
            pkg.svdcache_forecast_packed(shape, Sp, packed, R, Fh)
            out += [R.clone(), S.clone(), Fh.clone(), Sp.clone()]
        return out

    S, R, Fh = S0.to(DEV), torch.empty_like(F), torch.empty_like(F)
    wide = torch.empty(B, N, D + 8, device=DEV, dtype=dtype)[:, :, :D]
    other = torch.float64 if dtype == torch.float32 else torch.float32
    full = lambda **kw: pkg.svdcache_full_step(*[{**dict(shape=shape, F=F, V=V, P=packed, R=R, S=S, C=None, a=0.5, i=False), **kw}[n]
                                                for n in ("shape", "F", "V", "P", "R", "S", "C", "a", "i")])
    bad = [lambda: full(R=wide), lambda: full(F=F.to(other)), lambda: full(V=V[:, :, :-1]), lambda: full(S=S.double()),
           lambda: full(S=S.transpose(1, 2)), lambda: full(C=S[:1]), lambda: full(F=F.cpu()), lambda: full(a=0.0), lambda: full(a=1.5),
           lambda: full(a=float("nan")), lambda: full(a="x"), lambda: full(V=None), lambda: full(P=torch.empty(8, device=DEV)),
           lambda: pkg.svdcache_forecast(shape, S, V, packed, R[:1], Fh), lambda: pkg.svdcache_forecast(shape, S, V, packed, R, wide),
           lambda: pkg.svdcache_forecast_combine(shape, [S], [1.0, 2.0], V, packed, R, None, Fh),
           lambda: pkg.svdcache_forecast_combine(shape, [S] * 5, [1.0] * 5, V, packed, R, None, Fh),
           lambda: pkg.svdcache_forecast_combine(shape, [S], [float("nan")], V, packed, R, None, Fh),
           lambda: full(shape=bytes(shape)), lambda: full(shape=np.frombuffer(bytes(shape), np.uint8)),
           lambda: pkg.svdcache_forecast(bytes(shape), S, V, packed, R, Fh)]

    def refusals():
        texts = []
        for call in bad:
            with pytest.raises(Exception) as e:
                call()
            texts.append((type(e.value).__name__, str(e.value)))
        return texts

    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        by_module = good()
        made = {name: set(v) for name, v in answers.items()}
        answers.clear()
        said_module = refusals()
    assert made == {name: {0} for name in ("full_step", "forecast", "full_step_residual_ema", "forecast_combine") +
                    (("full_step_packed", "forecast_packed") if Sp is not None else ())}
    # a number out of range, or a state too many, is for the library to refuse; all other refusals are Python's
    assert sorted(answers) == ["forecast", "forecast_combine", "full_step"]
    assert answers["forecast"] == [None] * 3 and answers["forecast_combine"] == [None, None, -5]
    assert answers["full_step"] == [None] * 7 + [-5] * 3 + [None] * 5
    monkeypatch.setattr(binding, "_fast", None)
    with torch.cuda.stream(side):
        by_ctypes, said_ctypes = good(), refusals()
    torch.cuda.synchronize()
    assert said_module == said_ctypes
    assert all(torch.equal(x, y) for x, y in zip(by_module, by_ctypes)) and len(by_module) == len(by_ctypes)
    # what is only another way to hand over the same arguments still works
    monkeypatch.setattr(binding, "_fast", fast)
    two = pkg.make_shape(F[0], k)
    pkg.svdcache_full_step(two, F[0], V[:1], None, R[0], S[:1].contiguous(), None, np.float32(0.5), 1)
    pkg.svdcache_forecast_combine(shape, (S, S), (0.5, 0.5), V, packed, R, None, Fh)
    # a weight whose conversion takes the other weights away
    class Greedy:
        def __float__(self):
            del weights[1:]
            return 0.5

    weights = [Greedy()] + [0.5] * 3
    assert fast.forecast_combine(shape, [S] * 4, weights, V, packed, R, None, Fh) is None and len(weights) == 4
    torch.cuda.synchronize()
