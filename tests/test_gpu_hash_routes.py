"""hash_keys (over many keys: codes on the matrix cores with certified signs,
residual norms apart; over few, in the reference arithmetic throughout) and
hash_keys_mm against the kernel of decode-time append, which keeps
the residual of Algorithm 2 and decides every bit in the reference arithmetic:
the same codes, norms and fragile counts bit for bit, over the forms in which
certified decisions are rare.  (The append kernel is checked against the oracle
in test_gpu_append.py.)"""
import pytest
import torch

import paper_2608_04405_amd as bpc

pytestmark = pytest.mark.gpu
DEV = "cuda"


def reference(K, P, N):
    B, H, _, _ = K.shape
    L = P.shape[-2]
    kn = K[:, :, :N].contiguous()
    Kc, Vc = torch.zeros_like(kn), torch.zeros_like(kn)
    codes = torch.zeros(B, H, N, L // 32, dtype=torch.int32, device=DEV)
    err = torch.empty(B, H, N, device=DEV)
    frag = torch.zeros(1, dtype=torch.int64, device=DEV)
    bpc.append_kv(kn, kn, Kc, Vc, codes, P, 0, err_out=err, fragile=frag)
    return codes, err, int(frag)


def check(K, P, N):
    B, H = K.shape[:2]
    L = P.shape[-2]
    want, err0, frag0 = reference(K, P, N)
    for mm in (False, True):
        codes = torch.full((B, H, N + 2, L // 32), 0x5A5A5A5A, dtype=torch.int32, device=DEV)
        err = torch.empty(B, H, N, device=DEV)
        frag = torch.zeros(1, dtype=torch.int64, device=DEV)
        fall = torch.zeros(1, dtype=torch.int64, device=DEV)
        if mm:
            bpc.hash_keys_mm(K, P, N=N, codes_out=codes, fragile=frag, fallbacks=fall)
            assert 0 <= int(fall) <= B * H * N * L
        else:
            bpc.hash_keys(K, P, N=N, codes_out=codes, err_out=err, fragile=frag)
            assert bool(((err == err0) | (err.isnan() & err0.isnan())).all())
        assert torch.equal(codes[:, :, :N], want)
        assert (codes[:, :, N:] == 0x5A5A5A5A).all()
        assert int(frag) == frag0


def inputs(N, L, B=1, H=2, seed=0):
    g = torch.Generator(device=DEV).manual_seed(seed + L)
    A = torch.randn(H, 8, 128, generator=g, device=DEV)
    K = (torch.randn(B, H, N, 8, generator=g, device=DEV) @ A
         + 0.1 * torch.randn(B, H, N, 128, generator=g, device=DEV)).to(torch.bfloat16)
    P = torch.randn(B, H, L, 128, generator=g, device=DEV) * torch.linspace(1.0, 0.05, L, device=DEV).view(-1, 1)
    return K, P


# one key, a tile and its edges, a 256-key workgroup of the norms and its edges,
# several workgroups (each wavefront decides one tile here: second_tiles below)
# (calls of 8 heads take the reference arithmetic with norms; with more than 512
# groups of 64 keys, and more than one per head, the norms are apart)
@pytest.mark.parametrize("L,N,B", [(32, 1, 2), (64, 63, 2), (128, 65, 2), (64, 256, 2), (128, 257, 2), (32, 255, 2),
                                   (64, 1500, 2), (64, 64, 260), (64, 65, 128), (128, 65, 129), (32, 255, 70),
                                   (64, 256, 65), (128, 257, 60), (64, 1500, 12)])
def test_sizes(L, N, B):
    print(f"[hash routes] L={L} N={N} B={B}", flush=True)
    check(*inputs(N, L, B=B), N)


@pytest.mark.parametrize("B", [1, 60])
@pytest.mark.parametrize("L", [32, 64, 128])
@pytest.mark.parametrize("form", ["zero_rows", "zero_projection", "zero_keys", "exact_fit", "few_uncertain", "non_finite",
                                  "huge", "tiny", "strided", "shared"])
def test_forms(form, L, B):
    print(f"[hash routes] {form} L={L} B={B}", flush=True)
    N = 300
    K, P = inputs(N, L, B=B, seed=7)
    if form == "zero_rows":  # a head whose keys ran out of directions
        P[:, :, L // 2:] = 0
        P[:, :, 3] = 0
    elif form == "zero_projection":
        P.zero_()
    elif form == "zero_keys":  # padding inside a cache
        K[:, :, 40:200] = 0
    elif form == "exact_fit":  # every residual reaches 0 and most decisions are exactly 0
        P[:] = 0
        P[:, :, 0, :64] = 1.5
        P[:, :, 1, 64:] = 0.25
        K = torch.cat([P[:, :, :1, :64].expand(B, 2, N, 64), P[:, :, 1:2, 64:].expand(B, 2, N, 64)], -1)
        K = K.to(torch.bfloat16).contiguous()
        P[:, :, 2:] = torch.randn_like(P[:, :, 2:])
        P[:, :, 2:, ::2] = -P[:, :, 2:, 1::2]
    elif form == "few_uncertain":  # single keys at zero among certain ones
        K[:, :, ::50] = 0
    elif form == "non_finite":
        K[0, 0, 5, 1] = float("inf")
        K[0, 1, 64, 127] = float("nan")
        P[0, 1, 9, 0] = float("inf")
    elif form == "huge":
        K = (K.float() * 2.0 ** 100).to(torch.bfloat16)
        P = P * 2.0 ** 20
    elif form == "tiny":
        K = (K.float() * 2.0 ** -120).to(torch.bfloat16)
    elif form == "strided":
        K = torch.zeros(B, N, 2, 144, dtype=torch.bfloat16, device=DEV).transpose(1, 2)[..., :128].copy_(K)
    elif form == "shared":
        P = P[0, 0].contiguous()
    check(K, P, N - 13 if form == "strided" else N)


# Calls of more than 524288 keys give every wavefront a second tile, whose keys
# are loaded while the first is decided: a workgroup covers 512 keys at L = 32
# (256 at a time) and 1024 above (512 at a time).  Here the last workgroup's
# first wavefront goes from a whole tile to one of 10 keys.
SECOND = [(32, 4096 + 256 + 10), (64, 4096 + 512 + 10), (128, 4096 + 512 + 10)]


@pytest.mark.parametrize("L,N", SECOND)
@pytest.mark.parametrize("form", ["plain", "zero_tiles", "cancelling_tiles", "few_zero_keys", "late_zeros"])
def test_second_tiles(form, L, N):
    """A whole tile decided in the reference arithmetic (its keys' products with
    a row of P cancel) must leave the keys of the wavefront's next tile loaded,
    whichever block of bits it was found in.  Zero keys need no such tile."""
    print(f"[hash routes] second tiles {form} L={L} N={N}", flush=True)
    K, P = inputs(N, L, B=16, H=8, seed=11)
    if form == "zero_tiles":
        K[:, ::2, 4096:4160] = 0  # before the 10-key tail
        K[:, :, 1024:1088] = 0    # before an ordinary tile
        K[:, 1::4, :2048] = 0     # half of a head, as left padding
    elif form == "cancelling_tiles":  # a_0 = 0: uncertain in the first block
        P[:, :, 0, ::2] = -P[:, :, 0, 1::2]
        K[:, ::2, 4096:4160] = 1.0
        K[:, :, 1024:1088] = 1.0
        K[:, 1::4, :2048] = 1.0
    elif form == "few_zero_keys":  # stays with single decisions
        K[:, :, 4096:4116] = 0
    elif form == "late_zeros":  # residuals reach 0 after the first block of bits
        P[:, :, 16:, ::2] = -P[:, :, 16:, 1::2]
        P[:, :, :16] = 0
        P[:, :, 0] = 1.0
        K[:, :, 4096:4160] = 1.0
    check(K, P, N)


@pytest.mark.parametrize("L", [32, 64, 128])
@pytest.mark.parametrize("N", [20, 64, 84])
@pytest.mark.parametrize("other", ["infinite", "huge", "plain"])
def test_zero_rows_beside(other, N, L):
    """Zero rows of P are counted as fragile once per key, also where another
    row takes the bounds out of range and single decisions are recomputed (at
    most 24 keys of a tile)."""
    print(f"[hash routes] zero rows beside {other} rows N={N} L={L}", flush=True)
    K, P = inputs(N, L, seed=5)
    P[:, :, 3] = 0
    P[:, 1, 20:25] = 0
    if other == "infinite":
        P[:, :, 9, 4] = float("inf")
    elif other == "huge":
        P[:, :, 9] *= 1e32
    check(K, P, N)


@pytest.mark.parametrize("L", [32, 64, 128])
@pytest.mark.parametrize("lead", [0, 1, 17, 31, "all"])
def test_zero_keys(lead, L):
    """Zero keys (of either sign), and keys whose squares vanish in fp32, among
    ordinary ones: up to the first row of P that is not zero, whichever block it
    lies in, their decisions are exact zeros."""
    print(f"[hash routes] zero keys after {lead} zero rows L={L}", flush=True)
    N = 200
    K, P = inputs(N, L, B=70, seed=3)
    P[:, :, : L if lead == "all" else lead] = 0
    K[:, :, 64:128] = 0
    K[:, :, 64:128:3] = -K[:, :, 64:128:3]
    K[:, :, 130] = 0
    K[:, :, 150, :] = 0
    K[:, :, 150, 7] = 2.0 ** -80  # not zero
    K[:, :, 64, 9] = 2.0 ** -126
    check(K, P, N)
    P[:, 1, L - 1, 5] = float("inf")  # no usable bound
    check(K[:1], P[:1], 20)
    check(K, P, N)
