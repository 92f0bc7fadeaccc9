"""recon_apply over the batch sizes of its kernels and the row alignments they take."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _check(M, N, off, B, noalloc):
    """Rows that start off floats past an allocation: each sum is within N rounding errors of
    2^-24 of the sum of |R s|, plus alpha, beta and the few sums of partial sums."""
    import torch
    import paper_1608_00386_amd as W
    rng = np.random.default_rng(M + 7 * N + 31 * B)
    R = rng.standard_normal((M, N)).astype(np.float32)
    S = rng.standard_normal((B, N)).astype(np.float32)
    C0 = rng.standard_normal((B, M)).astype(np.float32)

    def put(a):
        t = torch.empty(a.size + off, device="cuda")
        t[off:] = torch.from_numpy(a.ravel()).cuda()
        return t[off:].view(a.shape)

    Rt, St, Ct = put(R), put(S), torch.from_numpy(C0.copy()).cuda()
    W.recon_apply(Rt, St, Ct, alpha=0.7, beta=0.5, noalloc=noalloc)
    again = torch.from_numpy(C0.copy()).cuda()
    W.recon_apply(Rt, St, again, alpha=0.7, beta=0.5, noalloc=noalloc)
    assert torch.equal(Ct, again)
    R64, S64, C64 = R.astype(np.float64), S.astype(np.float64), C0.astype(np.float64)
    a, b = float(np.float32(0.7)), float(np.float32(0.5))
    ref = a * (S64 @ R64.T) + b * C64
    scale = a * (np.abs(S64) @ np.abs(R64).T) + np.abs(b * C64)
    err = np.abs(Ct.cpu().numpy() - ref)
    assert np.all(err <= (N + 4) * 2.0 ** -24 * scale)


@pytest.mark.parametrize("noalloc", [False, True])
@pytest.mark.parametrize("B", [1, 2, 5, 8, 9, 16, 17, 32, 33, 49])
@pytest.mark.parametrize("M,N,off", [(1, 1, 0), (63, 127, 0), (65, 130, 1), (64, 128, 0),
                                     (130, 1029, 3), (200, 3000, 2)])
def test_recon_batches_match_fp64(M, N, off, B, noalloc):
    _check(M, N, off, B, noalloc)


@pytest.mark.parametrize("M,B", [(262145, 17), (140000, 40)])
def test_recon_noalloc_many_rows(M, B):
    """More rows than the fixed array holds tiles of 16 (one realisation a pass; unaligned rows
    only) or of 32 realisations."""
    _check(M, 3, 1, B, True)


@pytest.mark.parametrize("M,N,Bs", [
    (5400, 55607, (8, 16, 24)), (5400, 55608, (16,)), (5400, 8001, (8, 20)),
    (3000, 1001, (2, 9, 16, 24)), (3000, 515, (8, 16, 20)), (64, 20001, (8, 12, 32))])
def test_recon_sums_are_as_exact_as_a_gemv(M, N, Bs):
    """The rms error over all sums is within that of a GEMV per realisation: 64 lanes add every
    64th product of a split one after the other, (L + 1) / 2 roundings of the variance of all N
    products for chains of L, then a tree of 6 levels and the splits in order, half a rounding
    each.  The splits: as many as 8,192 waves of two rows hold, of at least 256 columns, whole
    groups of 64.  A rounding is at most 2^-24 of its value, uniformly distributed (1 / 3)."""
    import torch
    import paper_1608_00386_amd as W
    gen = torch.Generator(device="cuda").manual_seed(M + N)
    R = torch.randn(M, N, device="cuda", generator=gen)
    S = torch.randn(max(Bs), N, device="cuda", generator=gen)
    ref = torch.empty(max(Bs), M, dtype=torch.float64, device="cuda")
    rss = torch.empty_like(ref)
    for i in range(0, M, 600):
        r = R[i:i + 600].double()
        ref[:, i:i + 600] = S.double() @ r.T
        rss[:, i:i + 600] = ((S.double() ** 2) @ (r ** 2).T).sqrt()
    splits = max(1, min(8192 // ((M + 1) // 2), N // 256))
    chunk = -(-(-(-N // splits)) // 64) * 64
    splits = -(-N // chunk)
    bound = 2.0 ** -24 * (((chunk / 64 + 1) / 2 + 6 + splits / 2) / 3) ** 0.5
    for B in Bs:
        for noalloc in (False, True):
            C = torch.empty(B, M, device="cuda")
            W.recon_apply(R, S[:B], C, noalloc=noalloc)
            rms = float(((C.double() - ref[:B]) / rss[:B]).square().mean().sqrt())
            assert rms <= bound, (B, noalloc, rms / bound)
