"""Appends of a few tokens (a wavefront per key) against one append of all of
them (four lanes per key, every dot product in the reference order): the same
cache rows, codes, norms and fragile counts bit for bit, also where decisions
cannot be certified."""
import pytest
import torch

import paper_2608_04405_amd as bpc

pytestmark = pytest.mark.gpu
DEV = "cuda"


def run(k, v, P, T):
    B, H, N, _ = k.shape
    L = P.shape[-2]
    K = torch.zeros(B, H, N + 5, 128, dtype=torch.bfloat16, device=DEV)
    V = torch.zeros_like(K)
    codes = torch.zeros(B, H, N + 5, L // 32, dtype=torch.int32, device=DEV)
    frag = torch.zeros(1, dtype=torch.int64, device=DEV)
    errs = []
    for t in range(0, N, T):
        err = torch.empty(B, H, min(T, N - t), device=DEV)
        bpc.append_kv(k[:, :, t:t + T], v[:, :, t:t + T], K, V, codes, P, 2 + t, err_out=err, fragile=frag)
        errs.append(err)
    torch.cuda.synchronize()
    return K, V, codes, torch.cat(errs, -1), int(frag)


@pytest.mark.parametrize("L", [32, 64, 128])
@pytest.mark.parametrize("form", ["plain", "zero_keys", "zero_rows", "exact_fit", "non_finite", "huge", "tiny"])
def test_chunks(form, L):
    print(f"[append wave] {form} L={L}", flush=True)
    N = 48
    g = torch.Generator(device=DEV).manual_seed(L)
    A = torch.randn(8, 128, generator=g, device=DEV)
    k = (torch.randn(2, 2, N, 8, generator=g, device=DEV) @ A).to(torch.bfloat16)
    v = torch.randn(2, 2, N, 128, generator=g, device=DEV).to(torch.bfloat16)
    P = torch.randn(2, 2, L, 128, generator=g, device=DEV)
    if form == "zero_keys":
        k[:, :, 10:30] = 0
    elif form == "zero_rows":
        P[:, :, 1::3] = 0
    elif form == "exact_fit":  # residuals reach 0, later decisions are exact zeros or cancel
        P[:, :, 0] = 1.0
        k[:] = 1.0
        P[:, :, 2:, ::2] = -P[:, :, 2:, 1::2]
    elif form == "non_finite":
        k[0, 0, 3, 5] = float("inf")
        k[1, 1, 7, 0] = float("nan")
        P[1, 0, L - 1, 127] = float("inf")
    elif form == "huge":
        k, P = (k.float() * 2.0 ** 110).to(torch.bfloat16), P * 2.0 ** 60
    elif form == "tiny":
        k, P = (k.float() * 2.0 ** -125).to(torch.bfloat16), P * 2.0 ** -20
    want = run(k, v, P, N)
    for T in (1, 7, 32):
        for a, b in zip(run(k, v, P, T), want):
            if isinstance(a, int):
                assert a == b
            elif a.dtype == torch.float32:
                assert bool(((a == b) | (a.isnan() & b.isnan())).all())
            else:
                assert torch.equal(a.view(torch.int16), b.view(torch.int16))


@pytest.mark.parametrize("L", [32, 64, 128])
@pytest.mark.parametrize("T,H", [(16, 300), (17, 240), (17, 300), (32, 128), (32, 129)])
def test_counts(T, H, L):
    """The number of new keys and heads at which a wavefront per key stops: the
    same results on either side as with four lanes per key."""
    print(f"[append wave] T={T} H={H} L={L}", flush=True)
    g = torch.Generator(device=DEV).manual_seed(L + T)
    k = torch.randn(1, H, 2 * T, 128, generator=g, device=DEV).to(torch.bfloat16)
    v = torch.randn(1, H, 2 * T, 128, generator=g, device=DEV).to(torch.bfloat16)
    P = torch.randn(1, H, L, 128, generator=g, device=DEV)
    wide = lambda x: torch.cat([x, x, x], 2)[:, :, :33].contiguous()  # 33 keys: four lanes per key
    want = run(wide(k[:, :, :T]), wide(v[:, :, :T]), P, 33)
    got = run(k[:, :, :T].contiguous(), v[:, :, :T].contiguous(), P, T)
    for a, b in zip(got[:3], want[:3]):
        assert torch.equal(a[:, :, 2:2 + T], b[:, :, 2:2 + T])
    assert torch.equal(got[3], want[3][:, :, :T])
