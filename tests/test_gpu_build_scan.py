"""The scanning build of Algorithm 1 (closed-form sums, certified signs and
certified rows of P) against the build that rebuilds every residual in the
reference arithmetic, which runs on a workspace too small for the former: the
same P, codes, errors and fragile counts bit for bit.  (Both are checked
against the oracle in test_gpu_parity.py and test_gpu_fullsize.py.)"""
import math

import numpy as np
import pytest
import torch

import oracle
import paper_2608_04405_amd as bpc
from _helpers import bits_of

pytestmark = pytest.mark.gpu
DEV = "cuda"


def small_workspace(B, H, N, L):
    """The bytes the residual-rebuilding build needs: one fp64 sum per
    128-key chunk and coordinate (and per 32 chunks when there are more than
    256), P and G in fp64."""
    nch = -(-N // 128)
    nfold = -(-nch // 32) if nch > 256 else 0
    return 1024 * (B * H * (nch + nfold + L) + L)


def both(K, G, N, codes_stride_rows=0):
    B, H = K.shape[:2]
    L = G.shape[0]
    res = []
    sizes = [bpc.build_workspace_bytes(B, H, N, L), small_workspace(B, H, N, L)]
    for size in sizes:
        ws = torch.randint(0, 256, (size,), dtype=torch.uint8, device=DEV)
        codes = torch.full((B, H, N + codes_stride_rows, L // 32), 0x5A5A5A5A, dtype=torch.int32, device=DEV)
        err = torch.empty(B, H, N, device=DEV)
        frag = torch.zeros(1, dtype=torch.int64, device=DEV)
        P, codes, err = bpc.build_hash(K, G, N=N, codes_out=codes, err_out=err, fragile=frag, workspace=ws)
        torch.cuda.synchronize()
        assert (codes[:, :, N:] == 0x5A5A5A5A).all()
        res.append((P, codes, err, int(frag)))
    if sizes[1] >= sizes[0]:  # a few keys: any accepted workspace holds the scanning build
        res[1] = by_oracle(K, G, N)
    return res


def by_oracle(K, G, N):
    B, H = K.shape[:2]
    out = [oracle.build_binary_pcs(bits_of(K)[b, h, :N], G.cpu().numpy()) for b in range(B) for h in range(H)]
    P, codes, err = (np.stack([o[i] for o in out]) for i in range(3))
    return (torch.from_numpy(P).reshape(B, H, -1, 128).to(DEV),
            torch.from_numpy(codes.view(np.int32)).reshape(B, H, N, -1).to(DEV),
            torch.from_numpy(err.astype(np.float32)).reshape(B, H, N).to(DEV), sum(int(o[3]) for o in out))


def assert_same(res):
    (P, c, e, f), (P2, c2, e2, f2) = res
    c = c[:, :, :e.shape[2]]
    c2 = c2[:, :, :e.shape[2]]
    assert torch.equal(c, c2)
    same = (P.view(torch.int32) == P2.view(torch.int32)) | (P.isnan() & P2.isnan())
    assert bool(same.all()), int((~same).sum())
    assert bool(((e == e2) | (e.isnan() & e2.isnan())).all())
    assert f == f2


def keys(N, B=1, H=2, seed=0, rank=8, noise=0.1):
    g = torch.Generator(device=DEV).manual_seed(seed)
    A = torch.randn(H, rank, 128, generator=g, device=DEV)
    Z = torch.randn(B, H, N, rank, generator=g, device=DEV)
    x = torch.randn(B, H, N, 128, generator=g, device=DEV) * noise
    for r in range(rank):
        x += Z[..., r:r + 1] * A[:, r:r + 1]
    return x.to(torch.bfloat16)


def directions(L, seed=1):
    return torch.randn(L, 128, generator=torch.Generator(device=DEV).manual_seed(seed), device=DEV)


# one key; one short, one whole, one whole and a bit 64-key tile; a 128-key
# chunk and a bit; a wavefront's and a workgroup's share and a bit; more than
# one block per wavefront
# (more than 256 chunks in all, or long heads, below which the rebuilding passes
# run anyway, as they do up to 128 keys per head but for L = 64)
@pytest.mark.parametrize("L,N,B,H", [(32, 1, 8, 5200), (64, 1, 8, 5200), (64, 63, 8, 96), (64, 64, 8, 96),
                                     (64, 65, 8, 96), (128, 65, 8, 96), (128, 129, 8, 96), (32, 129, 8, 48),
                                     (64, 257, 8, 24), (128, 1025, 8, 8), (64, 40961, 1, 8), (32, 6150, 1, 2)])
def test_sizes(L, N, B, H):
    print(f"[build scan] L={L} N={N} B={B} H={H}", flush=True)
    assert_same(both(keys(N, B, H, seed=N), directions(L), N, codes_stride_rows=3))


FORMS = ["zero_columns", "negative_zero_columns", "cancelling", "tiny_and_huge", "outlier_key", "denormal", "constant",
         "zero", "infinite", "strided"]


@pytest.mark.parametrize("L", [32, 64, 128])
@pytest.mark.parametrize("form", FORMS)
def test_forms(form, L):
    N = 640 if form != "strided" else 700
    print(f"[build scan] {form} L={L}", flush=True)
    K = keys(N, H=72, seed=L)
    if form == "zero_columns":  # heads of 64 padded to 128: those columns of P are zero
        K[..., 64:] = 0
    elif form == "negative_zero_columns":
        K[..., 5] = 0
        K[..., 5] = -K[..., 5]
        K[:, :, ::2, 9] = 0
        K[:, :, 1::2, 9] = -torch.zeros_like(K[:, :, 1::2, 9])
    elif form == "cancelling":  # u k = the same for k and -k: residuals cancel exactly
        K[:, :, N // 2:] = -K[:, :, :N // 2]
    elif form == "tiny_and_huge":  # magnitudes span more than fp64 sums hold exactly
        K[:, :, ::3] *= 2.0 ** -60
        K[:, :, 1::7] *= 2.0 ** 20
    elif form == "outlier_key":  # one key's norm far above the others'
        K[:, :, 11] *= 2.0 ** 12
    elif form == "denormal":
        K = (K.float() * 2.0 ** -128).to(torch.bfloat16)
    elif form == "constant":
        K[:] = K[:, :, :1]
    elif form == "zero":
        K.zero_()
    elif form == "infinite":
        K[0, 0, 17, 3] = float("inf")
        K[0, 1, 100, 77] = float("nan")
    elif form == "strided":  # rows of 136 elements, heads interleaved
        K = torch.zeros(1, N, 72, 136, dtype=torch.bfloat16, device=DEV).transpose(1, 2)[..., :128].copy_(K)
    assert_same(both(K, directions(L), N if form != "strided" else N - 57))


def test_small_integers():
    """Sums that are exact and often lie halfway between two floats, which is
    where a bound other than zero would not certify them."""
    N, L = 2048, 64
    g = torch.Generator(device=DEV).manual_seed(3)
    K = torch.randint(-4, 5, (1, 24, N, 128), generator=g, device=DEV).to(torch.bfloat16)
    K[:, :, ::2] = -K[:, :, 1::2]
    assert_same(both(K, directions(L), N))


def test_uncertified_columns():
    """Columns that cannot certify, few enough for the scan to go on: the sum of
    u_j R_jd cancels while its terms span more than 53 bits, so that nothing is
    known of its sign.  Three cancel at the first bit, three at the second (with
    the first row of P removed); 27 chunks, the last of four keys."""
    N, L = 26 * 128 + 4, 64
    rng = np.random.default_rng(8)
    u0, u1 = np.array([[1, 1], [1, -1], [-1, 1], [-1, -1]] * (N // 4)).T[:, rng.permutation(N)]
    to = lambda x: torch.from_numpy(np.ascontiguousarray(x)).float().to(torch.bfloat16)
    K = keys(N, H=2, seed=9).cpu()
    K[..., 0], K[..., 1] = to(u0 * rng.uniform(1, 2, N)), to(u1 * rng.uniform(1, 2, N))
    for d in (10, 11, 12, 20, 21, 22):
        x = to(2.0 ** rng.uniform(-60, 0, N // 2)).float().numpy().astype(np.float64)
        x[0], x[1] = 1.0, 2.0 ** -60
        k = np.zeros(N)
        if d < 20:  # pairs of one u0, opposite values
            order = np.concatenate([rng.permutation(np.flatnonzero(u0 == s)) for s in (1, -1)])
        else:       # pairs of one u1 and both u0: the sum of u0 k does not cancel
            order = np.stack([np.concatenate([rng.permutation(np.flatnonzero((u1 == s) & (u0 == t))) for s in (1, -1)])
                              for t in (1, -1)], 1).reshape(-1)
        k[order[::2]], k[order[1::2]] = x, -x
        u = u0 if d < 20 else u1
        # what the certificate needs does not hold: the sum is 0 (with equally
        # many u0 = u1 and u0 = -u1 also after the first bit) and cannot be exact
        assert math.fsum(u * k) == 0.0 and (u0 * u1).sum() == 0
        assert N * np.abs(k).max() >= 2.0 ** 53 * np.abs(k).min() * 2.0 ** -7
        assert d < 20 or math.fsum(u0 * k) > 1.0
        K[..., d] = to(k)
    G = directions(L)
    G[:2] = 0
    G[0, 0], G[1, 1] = 1.0, 1.0
    res = both(K.to(DEV), G, N)
    assert_same(res)
    assert_same((res[0], by_oracle(K, G, N)))


@pytest.mark.parametrize("L", [32, 64, 128])
def test_sign_of_a_vanished_column(L):
    """A column whose residual has become exactly zero sums to -0 where every
    term is -0: all u = -1 and no padding row (N a multiple of 128)."""
    N = 640
    K = torch.zeros(1, 72, N, 128, dtype=torch.bfloat16, device=DEV)
    K[..., 0] = 1.0
    K[:, :, 1::2, 0] = -1.0
    K[..., 1] = -1.0
    K[:, 36:, :, 2:] = keys(N, H=36, seed=3)[..., 2:]
    G = directions(L)
    G[0], G[1] = 0, 0
    G[0, 0], G[1, 1] = 1.0, 1.0
    res = both(K, G, N)
    assert bool((res[1][0][:, :36, 1, 0].view(torch.int32) == -2 ** 31).all())  # the case arises
    assert_same(res)
    assert_same(both(K, G, N - 1))


# A (b, h) whose columns or signs certify too rarely leaves the scan for the
# residuals, one bit behind the others: few different keys, a NaN, every sign
# uncertain, beside heads that go on scanning; one chunk, one fold of chunks and
# several, whole and ragged.
@pytest.mark.parametrize("L,N,H", [(64, 100, 420), (64, 643, 72), (128, 640, 72), (64, 2049, 24), (32, 5000, 12),
                                   (64, 70001, 3)])
@pytest.mark.parametrize("form", ["two_keys", "few_keys", "nan", "negative_zeros", "rank_one"])
def test_leaving_the_scan(form, L, N, H):
    print(f"[build scan] leaving: {form} L={L} N={N} H={H}", flush=True)
    K = keys(N, H=H, seed=L + N)
    part = K[:, ::3]
    if form == "two_keys":
        part[:] = part[:, :, :1].clone()
        part[:, :, ::3] = -0.5 * part[:, :, :1].clone() + 1
    elif form == "few_keys":
        part[:] = part[:, :, :16].repeat(1, 1, -(-N // 16), 1)[:, :, :N].clone()
    elif form == "nan":
        part[:, :, N // 3, 5] = float("nan")
    elif form == "negative_zeros":
        part[..., 64:] = 0
        part[:, :, ::2, 64:] = -part[:, :, ::2, 64:]
    elif form == "rank_one":
        part[:] = (part[:, :, :1].float() * torch.randint(-3, 4, (1, 1, N, 1), device=DEV)).to(torch.bfloat16)
    assert_same(both(K, directions(L), N))


# either side of the bounds between the scan, the rebuilding passes and those
# with a checkpoint
@pytest.mark.parametrize("L,N,H", [(32, 6143, 1), (32, 6144, 1), (64, 3071, 2), (64, 3072, 2), (64, 8192, 1),
                                   (128, 1535, 4), (128, 1536, 4), (128, 12288, 1), (64, 128, 256), (64, 128, 257),
                                   (128, 128, 257), (128, 129, 129), (32, 256, 129), (128, 1000, 70),
                                   (64, 600, 70), (64, 1000, 70)])
def test_paths(L, N, H):
    """Three sizes of workspace: the same results, whichever path each takes."""
    print(f"[build scan] paths L={L} N={N} H={H}", flush=True)
    K, G = keys(N, H=H, seed=L + N), directions(L)
    sizes = {small_workspace(1, H, N, L), small_workspace(1, H, N, L) + 1024 * 128 * H * -(-N // 128),
             bpc.build_workspace_bytes(1, H, N, L), bpc.build_checkpoint_workspace_bytes(1, H, N, L)}
    res = []
    for size in sorted(sizes):
        ws = torch.randint(0, 256, (size,), dtype=torch.uint8, device=DEV)
        err = torch.empty(1, H, N, device=DEV)
        frag = torch.zeros(1, dtype=torch.int64, device=DEV)
        P, codes, err = bpc.build_hash(K, G, err_out=err, fragile=frag, workspace=ws)
        res.append((P, codes, err, int(frag)))
    for r in res[1:]:
        assert_same((res[0], r))
