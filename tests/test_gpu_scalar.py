"""GPU parity of the scalar uniform-grid representation (App. K): dequantise and the
round-to-nearest V step, bit-exact against the CPU oracle, with targets and selection taken
through the ordinary calls at group size 1."""
import numpy as np
import pytest
import torch

import oracle
import workloads
from gpu_util import DEV, dev_f32, dev_i32
from paper_2405_14852_amd import Layout, PVContext, PVError

pytestmark = pytest.mark.gpu


def dev_u8(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.uint8)).to(DEV)


@pytest.mark.parametrize("shape,block,nbits", [((64, 512), 128, 2), ((33, 96), 16, 3), ((7, 60), 6, 4),
                                               ((16, 256), 8, 8), ((5, 7), 7, 1)])
@pytest.mark.parametrize("frac", [0.05, 1.0])
def test_scalar_v_step_matches_oracle(shape, block, nbits, frac):
    W0, G, codes, sc, zp = workloads.make_scalar(shape[0], shape[1], block, nbits, seed=95)
    ctx = PVContext(0)
    o, i = shape
    n = o * i
    k = max(1, int(frac * n))
    lay1 = Layout(o, i, 1, 1, 8)                       # group size 1: the unit is a weight
    cd, sd, zd = dev_u8(codes), dev_f32(sc), dev_f32(zp)
    Wd = torch.empty(o, i, dtype=torch.float32, device=DEV)
    ctx.pv_dequantize_scalar(o, i, block, nbits, cd, sd, zd, Wd)
    W_ref = oracle.dequantize_scalar(codes, sc, zp, block, nbits)
    assert np.array_equal(Wd.cpu().numpy().view(np.uint32), W_ref.view(np.uint32))
    Gd = dev_f32(G * 20)
    Td = torch.empty_like(Wd)
    idx = torch.empty(k, dtype=torch.int32, device=DEV)
    ctx.pv_encode_targets_select(lay1, Wd, Gd, 1.0, Td, k, idx)
    T_ref = oracle.encode_targets(W_ref, G * 20, 1.0)
    idx_ref = oracle.select_topk_groups(T_ref, W_ref, 1, k)
    assert np.array_equal(idx.cpu().numpy(), idx_ref)
    nch = torch.full((1,), -3, dtype=torch.int64, device=DEV)
    ctx.pv_reencode_scalar(o, i, block, nbits, Td, sd, zd, idx, k, cd, nch)
    torch.cuda.synchronize()
    want, changed = oracle.reencode_scalar(T_ref, sc, zp, idx_ref, codes, block, nbits)
    assert np.array_equal(cd.cpu().numpy(), want)
    assert int(nch.item()) == changed
    assert changed > 0 or n < 100
    ctx.pv_dequantize_scalar(o, i, block, nbits, cd, sd, zd, Wd)
    assert np.array_equal(Wd.cpu().numpy(), oracle.dequantize_scalar(want, sc, zp, block, nbits))
    ctx.close()


def test_scalar_tie_rule_empty_list_and_errors():
    ctx = PVContext(0)
    sc, zp = dev_f32(np.array([[1.0]], np.float32)), dev_f32(np.array([[0.0]], np.float32))
    codes = dev_u8(np.array([[2, 1, 0, 3]], np.uint8))
    T = dev_f32(np.array([[1.5, 1.5, 7.0, 100.0]], np.float32))
    nch = torch.zeros(1, dtype=torch.int64, device=DEV)
    ctx.pv_reencode_scalar(1, 4, 4, 2, T, sc, zp, dev_i32(np.array([0, 1, 2], np.int32)), 3, codes, nch)
    torch.cuda.synchronize()
    assert list(codes.cpu().numpy()[0]) == [2, 1, 3, 3] and int(nch.item()) == 1
    ctx.pv_reencode_scalar(1, 4, 4, 2, T, sc, zp, None, 0, codes, nch)          # k = 0: a no-op
    torch.cuda.synchronize()
    assert int(nch.item()) == 0
    for args in ((1, 4, 3, 2), (1, 4, 4, 9), (1, 4, 4, 0)):                      # bad block size / bits
        with pytest.raises(PVError):
            ctx.pv_reencode_scalar(*args, T, sc, zp, dev_i32(np.array([0], np.int32)), 1, codes, nch)
    with pytest.raises(PVError):
        ctx.pv_reencode_scalar(1, 4, 4, 2, T, sc, zp, dev_i32(np.array([0], np.int32)), 5, codes, nch)
    ctx.close()


def test_scalar_first_call_of_a_context_can_be_captured():
    """The search needs no scratch memory of a context for the caller's count: a first call may be captured,
    and calls outside the graph that count otherwise leave its replays as they are."""
    o, i, block, nbits = 64, 512, 128, 2
    W0, G, codes, sc, zp = workloads.make_scalar(o, i, block, nbits, seed=96)
    side = torch.cuda.Stream(device=DEV)
    ctx = PVContext(0, stream=side)
    T_np = oracle.encode_targets(oracle.dequantize_scalar(codes, sc, zp, block, nbits), G * 20, 1.0)
    ids = np.arange(0, o * i, 3, dtype=np.int32)
    T, sd, zd, cd, idx = dev_f32(T_np), dev_f32(sc), dev_f32(zp), dev_u8(codes), dev_i32(ids)
    before, nch = cd.clone(), torch.zeros(1, dtype=torch.int64, device=DEV)
    want, changed = oracle.reencode_scalar(T_np, sc, zp, ids, codes, block, nbits)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        ctx.pv_reencode_scalar(o, i, block, nbits, T, sd, zd, idx, len(ids), cd, nch)
    for replay in (True, True, False, True):
        cd.copy_(before)
        nch.fill_(-3)
        torch.cuda.synchronize()
        if replay:
            graph.replay()
        else:
            ctx.pv_reencode_scalar(o, i, block, nbits, T, sd, zd, idx, len(ids), cd, nch)
        torch.cuda.synchronize()
        assert np.array_equal(cd.cpu().numpy(), want) and int(nch.item()) == changed > 0
    ctx.close()


def test_scalar_replays_beside_one_another_and_beside_a_call():
    """Graphs of one context's scalar searches share nothing but what the caller gives them: two of them replayed side
    by side, and one beside a call, all count right, as does every call after them."""
    o, i, block, nbits = 8192, 4096, 128, 2
    gen = torch.Generator(device=DEV)
    gen.manual_seed(97)
    T = torch.randn(o, i, generator=gen, device=DEV)
    sc, zp = (torch.rand(o, i // block, generator=gen, device=DEV) + 0.2 for _ in range(2))
    before = torch.randint(0, 4, (o, i), generator=gen, device=DEV, dtype=torch.uint8)
    idx = torch.arange(o * i, dtype=torch.int32, device=DEV)
    streams = [torch.cuda.Stream(device=DEV) for _ in range(3)]
    ctx = PVContext(0, stream=streams[0])
    codes = [before.clone() for _ in range(3)]
    nch = [torch.zeros(1, dtype=torch.int64, device=DEV) for _ in range(3)]
    torch.cuda.synchronize()

    def call(n):
        ctx.pv_reencode_scalar(o, i, block, nbits, T, sc, zp, idx, o * i, codes[n], nch[n])

    call(0)                             # the context has counted before
    torch.cuda.synchronize()
    want, changed = codes[0].clone(), int((codes[0] != before).sum())
    graphs = [torch.cuda.CUDAGraph() for _ in range(2)]
    for n, graph in enumerate(graphs):
        with torch.cuda.graph(graph, stream=streams[0]):
            call(n + 1)
    for _ in range(4):
        for n in range(3):
            codes[n].copy_(before)
            nch[n].fill_(-3)
        torch.cuda.synchronize()
        for n, graph in enumerate(graphs):
            with torch.cuda.stream(streams[n + 1]):
                graph.replay()
        call(0)
        torch.cuda.synchronize()
        for n in range(3):
            assert int(nch[n].item()) == changed > 0 and torch.equal(codes[n], want)
    ctx.close()


def sampled_vectors(n):
    """The vectors of four weights that the sweep of many single weights samples its scores from."""
    i, u32 = np.arange(16384, dtype=np.uint64), np.uint64(0xFFFFFFFF)
    h = (i * np.uint64(0x9E3779B9)) & u32
    h = ((h ^ (h >> np.uint64(15))) * np.uint64(0x2C1B3C6D)) & u32
    h ^= h >> np.uint64(13)
    nvec = np.uint64(n // 4)
    return ((i * nvec) // np.uint64(16384) + ((h * (nvec // np.uint64(16384))) >> np.uint64(32))).astype(np.int64)


@pytest.mark.parametrize("shape", [(3072, 4096), (4001, 3777)])      # the fewest that the sweep collects from; a ragged end
@pytest.mark.parametrize("kind", ["normal", "equal", "rows", "columns", "zeros", "not_finite", "sampled", "sampled_few",
                                  "half_alike"])
def test_selection_among_many_single_weights(shape, kind):
    """The sweep that keeps keys from a sampled digit on, against a partition of all scores: spread scores, all
    alike, rows and columns of their own size (cells and regions whose lists do not fit), mostly zeros, NaN
    and infinities; and large updates exactly where the sample looks, so that fewer than k (or just the rest)
    are kept and every digit is counted from T and W."""
    rows, cols = shape
    n = rows * cols
    gen = torch.Generator(device=DEV)
    gen.manual_seed(96)
    W = torch.randn(rows, cols, generator=gen, device=DEV) * 0.02
    G = torch.randn(rows, cols, generator=gen, device=DEV) * 1e-4
    if kind == "equal":
        W.zero_()
        G.fill_(1e-4)
    elif kind in ("rows", "columns"):
        size = (rows, 1) if kind == "rows" else (1, cols)
        G *= torch.exp(2 * torch.randn(*size, generator=gen, device=DEV))
    elif kind == "zeros":
        G *= torch.rand(rows, cols, generator=gen, device=DEV) < 0.003
    elif kind == "half_alike":          # the lower rows alike, more than half of all; few in a region of the upper ones
        W[rows // 3:], G[rows // 3:] = 0.0, 1e-4
        G[:rows // 3] *= torch.rand(rows // 3, cols, generator=gen, device=DEV) < 0.02
    elif kind == "not_finite":
        G[3, 5], G[7, 9], G[rows - 1, cols - 1] = float("nan"), float("inf"), -float("nan")
    elif kind != "normal":
        at = torch.from_numpy(sampled_vectors(n)).to(DEV)
        G.mul_(1e-2).view(-1)[:n // 4 * 4].view(-1, 4)[at] = 1 + torch.rand(len(at), 4, generator=gen, device=DEV)
        if kind == "sampled_few":
            G.view(-1)[-1000:] = 3.0
    lay, ctx, T = Layout(rows, cols, 1, 1, 2), PVContext(0), torch.empty_like(W)
    for k in (n // 100, 7, n // 16, n // 8):
        for call in range(2):           # the second finds what the first left in the scratch
            idx = torch.full((k,), -7, dtype=torch.int32, device=DEV)
            T.fill_(5.0)
            ctx.pv_encode_targets_select(lay, W, G, 0.3, T, k, idx)
        torch.cuda.synchronize()
        want_T = torch.empty_like(W)
        ctx.pv_encode_targets(lay, W, G, 0.3, want_T)
        assert torch.equal(T.view(torch.int32), want_T.view(torch.int32))
        key = ((T - W) ** 2).view(-1).view(torch.int32).cpu().numpy()
        key = np.where(key < 0, 0x7FFFFFFF, key)
        least = np.partition(key, n - k)[n - k]
        ties = np.nonzero(key == least)[0][:k - int((key > least).sum())]
        want = np.sort(np.concatenate([np.nonzero(key > least)[0], ties]))
        assert np.array_equal(idx.cpu().numpy(), want)
    ctx.close()


def test_selection_among_many_single_weights_first_called_into_a_graph():
    """A context whose scratch is large enough from a larger shape: the first call among many single weights may be
    captured (the sample's memory is not there, and cannot be allocated), and calls after it sample."""
    rows, cols = 3072, 4096
    n, k = rows * cols, rows * cols // 100
    gen = torch.Generator(device=DEV)
    gen.manual_seed(98)
    W, G = (torch.randn(rows, 2 * cols, generator=gen, device=DEV) for _ in range(2))
    side = torch.cuda.Stream(device=DEV)
    ctx, T = PVContext(0, stream=side), torch.empty_like(W)
    idx = torch.empty(k, dtype=torch.int32, device=DEV)
    torch.cuda.synchronize()
    ctx.pv_encode_targets_select(Layout(rows, 2 * cols, 2, 1, 2), W, G, 0.3, T, k, idx)
    side.synchronize()
    W1, G1 = W[:, :cols].contiguous(), G[:, :cols].contiguous()
    T1, lay = torch.empty_like(W1), Layout(rows, cols, 1, 1, 2)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        ctx.pv_encode_targets_select(lay, W1, G1, 0.3, T1, k, idx)
    for call in ("replay", "eager", "replay", "replay"):
        idx.fill_(-7)
        T1.fill_(5.0)
        torch.cuda.synchronize()
        if call == "replay":
            graph.replay()
        else:
            ctx.pv_encode_targets_select(lay, W1, G1, 0.3, T1, k, idx)
        torch.cuda.synchronize()
        score = ((T1 - W1) ** 2).view(-1)
        least = torch.topk(score, k).values[-1]
        above = torch.nonzero(score > least).view(-1)
        ties = torch.nonzero(score == least).view(-1)[:k - len(above)]
        assert torch.equal(idx.long(), torch.sort(torch.cat([above, ties])).values)
    ctx.close()
