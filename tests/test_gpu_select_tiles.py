"""select_hard by segments against a sort in the same order (IEEE total order
of float32, lowest index first among equals), at the edges of a segment, of
the levels and of m, with ties, negative and non-finite errors."""
import numpy as np
import pytest
import torch

import paper_2608_04405_amd as bpc

pytestmark = pytest.mark.gpu
DEV = "cuda"


def expected(e, m):
    u = e.view(np.uint32).astype(np.int64)
    key = np.where(u & 0x80000000, 0xFFFFFFFF - u, u + 0x80000000)
    return np.sort(np.lexsort((np.arange(len(e)), -key))[:m]).astype(np.int32)


# one segment exactly and one key more; m of a whole small input; the last length
# of the one-workgroup kernel and the first of a segment; the largest m of the
# segments and the first beyond; three levels
@pytest.mark.parametrize("N,m", [(16384, 1), (16384, 4096), (1000, 1000), (6144, 61), (6145, 61), (7000, 1), (16385, 66), (16385, 4096), (16385, 4097),
                                 (40000, 800), (140001, 4096), (600000, 3000), (65536, 1)])
@pytest.mark.parametrize("values", ["norms", "ties", "wide"])
def test_segments(N, m, values):
    print(f"[select tiles] N={N} m={m} {values}", flush=True)
    rng = np.random.default_rng(N + m)
    if values == "norms":
        e = (6 + 0.6 * rng.standard_normal((1, 2, N))).astype(np.float32)
    elif values == "ties":
        e = rng.integers(0, 5, (1, 2, N)).astype(np.float32)
        e[0, 1] = 2.5  # every key equal
    else:
        e = rng.integers(0, 2 ** 32, (1, 2, N), dtype=np.uint64).astype(np.uint32).view(np.float32)
        e[0, 0, : N // 3] = rng.standard_normal(N // 3) * 1e-30
    t = torch.from_numpy(np.concatenate([e, e[..., :3]], -1)).to(DEV)  # rows of N + 3
    got = bpc.select_hard(t, m, N=N)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    got2 = bpc.select_hard(t, m, N=N, stream=side)
    torch.cuda.synchronize()
    for h in range(2):
        want = expected(e[0, h], m)
        assert np.array_equal(got[0, h].cpu().numpy(), want)
        assert np.array_equal(got2[0, h].cpu().numpy(), want)


@pytest.mark.parametrize("N,m", [(9000, 7), (12, 3)])
def test_many_rows(N, m):
    """More (b, h) than a grid's y dimension takes (65536)."""
    B, H = 8193, 8
    print(f"[select tiles] {B} x {H} rows N={N} m={m}", flush=True)
    g = torch.Generator(device=DEV).manual_seed(N)
    e = torch.rand(B, 1, N, generator=g, device=DEV)
    t = e.expand(B, H, N)  # head stride 0
    got = bpc.select_hard(t, m)
    want = e.sort(dim=-1, descending=True, stable=True).indices[..., :m].sort(-1).values.int()
    assert torch.equal(got, want.expand(B, H, m))


def test_workspace_and_capture():
    """A given workspace is used; a captured call allocates nothing (a graph
    would outlive the allocation); any stream object with a handle is taken."""
    N, m = 40000, 800
    e = torch.rand(2, 2, N, generator=torch.Generator(device=DEV).manual_seed(1), device=DEV)
    want = torch.from_numpy(np.stack([expected(r, m) for r in e.cpu().numpy().reshape(4, N)])).reshape(2, 2, m).to(DEV)
    size = bpc.select_hard_workspace_bytes(2, 2, N, m)
    assert size > 0 and bpc.select_hard_workspace_bytes(2, 2, 4096, 40) == 0
    ws = torch.randint(0, 256, (size,), dtype=torch.uint8, device=DEV)
    out = torch.empty(2, 2, m, dtype=torch.int32, device=DEV)

    def allocations():
        return torch.cuda.memory_stats()["allocation.all.allocated"]

    before = allocations()
    bpc.select_hard(e, m, serr_out=out, workspace=ws)
    assert allocations() == before
    assert torch.equal(out, want)
    with pytest.raises(bpc.BPCError):
        bpc.select_hard(e, m, serr_out=out, workspace=ws[: size // 2])

    class Handle:
        cuda_stream = torch.cuda.current_stream().cuda_stream

    assert torch.equal(bpc.select_hard(e, m, stream=Handle()), want)

    side = torch.cuda.Stream()
    for given in (None, ws):
        with torch.cuda.stream(side):
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=side):
                before = allocations()
                bpc.select_hard(e, m, serr_out=out, workspace=given)
                assert allocations() == before
        for _ in range(3):
            out.fill_(-1)
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(out, want)
