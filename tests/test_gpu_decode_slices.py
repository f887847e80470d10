"""The decode step on 2048- and 4096-key slices at their edges (one key, one
short of a slice, one more, the last length of each size) against the
three-launch path: the same scores, selections and packed queries bit for bit,
the outputs to fp32 sums in another order (at most a few hundred terms of
relative size 2^-24, and probabilities split to 16 bits: 1e-4 of the largest
value); and with a workspace sized for the larger slices."""
import pytest
import torch

import paper_2608_04405_amd as bpc

pytestmark = pytest.mark.gpu
DEV = "cuda"


def step(B, G, H, N, L, k, ws_bytes=None, m=0):
    g = torch.Generator(device=DEV).manual_seed(N + L)
    q = torch.randn(B, G * H, 128, generator=g, device=DEV).to(torch.bfloat16)
    K = torch.randn(B, H, N + 3, 128, generator=g, device=DEV).to(torch.bfloat16)
    V = torch.randn(B, H, N + 3, 128, generator=g, device=DEV).to(torch.bfloat16)
    P = torch.randn(B, H, L, 128, generator=g, device=DEV)
    codes = torch.randint(-2 ** 31, 2 ** 31, (B, H, N + 3, L // 32), generator=g, device=DEV).int()
    size = bpc.decode_workspace_bytes(B, G * H, H, N, L, k) if ws_bytes is None else ws_bytes
    ws = torch.zeros(size, dtype=torch.uint8, device=DEV)
    idx = torch.empty(B, H, k, dtype=torch.int32, device=DEV)
    sc = torch.empty(B, H, N, dtype=torch.int32, device=DEV)
    qc = torch.empty(B, H, 8, L // 32, dtype=torch.int32, device=DEV)
    outs = []
    for _ in range(2):  # the second call finds the counters as the first left them
        outs.append(bpc.decode_attention(q, K, V, codes, P, k, N=N, idx_out=idx, score_out=sc, qcode_out=qc,
                                         workspace=ws))
    torch.cuda.synchronize()
    assert torch.equal(outs[0], outs[1])
    return outs[0], idx, sc, qc


@pytest.mark.parametrize("L,G", [(32, 1), (64, 4), (64, 8)])
@pytest.mark.parametrize("N,k", [(1, 1), (64, 7), (2047, 41), (2048, 2048), (2049, 41), (4096, 82), (4097, 90),
                                 (32768, 656), (32769, 656)])
def test_edges(N, k, L, G):
    print(f"[decode slices] N={N} k={k} L={L} G={G}", flush=True)
    B, H = 1, 4
    want_slice = 2048 if N <= 32768 else 4096
    assert bpc.decode_slice_keys(B, G * H, H, N, L) == want_slice
    got = step(B, G, H, N, L, k)
    try:
        bpc.set_decode_path(1)
        want = step(B, G, H, N, L, k)
    finally:
        bpc.set_decode_path(0)
    for a, b in zip(got[1:], want[1:]):
        assert torch.equal(a, b)
    assert float((got[0] - want[0]).abs().max()) <= 1e-4 * float(want[0].abs().max())


def test_workspace_of_larger_slices():
    B, G, H, N, L, k = 1, 4, 8, 32768, 64, 656
    full = bpc.decode_workspace_bytes(B, G * H, H, N, L, k)
    # 128 slices of 2048 keys; of 4096, half the records and partials
    per_slice = 4 * (68 + 4 + 132 + 128) + 4 * G * 130
    small = full - 64 * per_slice
    a, b = step(B, G, H, N, L, k), step(B, G, H, N, L, k, ws_bytes=small + 512)
    assert torch.equal(a[1], b[1]) and float((a[0] - b[0]).abs().max()) < 1e-4
    with pytest.raises(bpc.BPCError):
        step(B, G, H, N, L, k, ws_bytes=small // 2)


def test_per_head_workspace_of_larger_slices():
    B, G, H, N, L, k = 1, 4, 8, 16384, 64, 328
    g = torch.Generator(device=DEV).manual_seed(5)
    q = torch.randn(B, G * H, 128, generator=g, device=DEV).to(torch.bfloat16)
    K = torch.randn(B, H, N, 128, generator=g, device=DEV).to(torch.bfloat16)
    P = torch.randn(B, H, L, 128, generator=g, device=DEV)
    codes = torch.randint(-2 ** 31, 2 ** 31, (B, H, N, L // 32), generator=g, device=DEV).int()
    full = bpc.decode_per_head_workspace_bytes(B, G * H, H, N, L, k)
    # 256 slices of 2048 keys; of 4096, half the records and partials
    small = full - 128 * (4 * (68 + 4 + 132 + 128) + 4 * 130)
    got = []
    for size in (full, small + 512):
        idx = torch.empty(B, G * H, k, dtype=torch.int32, device=DEV)
        ws = torch.zeros(size, dtype=torch.uint8, device=DEV)
        got.append((bpc.decode_attention_per_head(q, K, K, codes, P, k, idx_out=idx, workspace=ws), idx))
    assert torch.equal(got[0][1], got[1][1]) and float((got[0][0] - got[1][0]).abs().max()) < 1e-4
    with pytest.raises(bpc.BPCError):
        bpc.decode_attention_per_head(q, K, K, codes, P, k, workspace=ws[: small // 2])
