"""GPU parity: the HIP path (through the C ABI) against the CPU oracle, element
by element on the same seeded inputs.

Bars: targets, group scores, selected ids, dequantised weights: bit-exact.
Codes: bit-exact, except on groups the oracle flags as near-ties (best two
objectives closer than 1e-6 relative), where the GPU's choice must be within
1e-6 relative of the oracle's objective when evaluated in oracle arithmetic.
"""
import numpy as np
import pytest
import torch

import oracle
import workloads
from paper_2405_14852_amd import PVContext
from gpu_util import DEV, GpuRun, check_codes_on, dev_f32, dev_i32, dev_u16, host_u16

pytestmark = pytest.mark.gpu

RECON_REL = 1e-5      # tolerance for reconstructed weights (relative L2)


def check_codes(wl, T_np, idx, got, want, info):
    M = wl.layout.num_codebooks
    g2 = got.reshape(-1, M)
    mask = np.ones(len(g2), bool)
    mask[idx] = False
    assert np.array_equal(g2[mask], wl.codes.reshape(-1, M)[mask]), "unselected codes changed"
    return check_codes_on(wl, T_np, idx, got, want, info)


# ------------------------------------------------------------------ targets

@pytest.mark.parametrize("shape,g", [((3, 6), 2), ((256, 256), 8), ((37, 1048), 8), ((1, 4), 1),
                                     ((129, 4100), 4)])
@pytest.mark.parametrize("alpha", [1.0, 0.37, 0.0])
def test_encode_targets_bit_exact(shape, g, alpha):
    wl = workloads.make(shape[0], shape[1], g, 1, 4, seed=1)
    run = GpuRun(wl)
    T = run.targets(alpha).cpu().numpy()
    ref = oracle.encode_targets(wl.W, wl.G, alpha)
    assert np.array_equal(T.view(np.uint32), ref.view(np.uint32))


def test_encode_targets_in_place():
    wl = workloads.make(64, 512, 8, 1, 4, seed=2)
    run = GpuRun(wl)
    ref = oracle.encode_targets(wl.W, wl.G, 0.5)
    W = run.W.clone()
    run.ctx.pv_encode_targets(run.lay, W, run.G, 0.5, W)
    assert np.array_equal(W.cpu().numpy(), ref)


# ------------------------------------------ targets from an Adam update (Sec. 3.4)

@pytest.mark.parametrize("shape,g", [((3, 6), 2), ((256, 256), 8), ((37, 1048), 8), ((1, 4), 1),
                                     ((129, 4100), 4), ((5, 7), 7)])
@pytest.mark.parametrize("step,lr,eps", [(1, 3e-3, 1e-8), (2, 1e-2, 1e-8), (1000, 3e-4, 1e-6)])
def test_encode_targets_adam_bit_exact(shape, g, step, lr, eps):
    wl = workloads.make(shape[0], shape[1], g, 1, 4, seed=21, sigma_g=1e-3)
    rng = np.random.default_rng(21)
    m = (rng.standard_normal(shape) * 1e-3).astype(np.float32) if step > 1 else np.zeros(shape, np.float32)
    v = (rng.random(shape) * 1e-6).astype(np.float32) if step > 1 else np.zeros(shape, np.float32)
    G = wl.G.copy()
    G.ravel()[::7] = 0.0                          # zero gradients among the rest
    if step > 1:
        v.ravel()[::11] = 1e-42                   # subnormal second moments
    run = GpuRun(wl)
    md, vd, Gd = dev_f32(m), dev_f32(v), dev_f32(G)
    T = torch.empty_like(run.W)
    run.ctx.pv_encode_targets_adam(run.lay, run.W, Gd, md, vd, step, lr, 0.9, 0.95, eps, T)
    torch.cuda.synchronize()
    T_ref, m_ref, v_ref = oracle.encode_targets_adam(wl.W, G, m, v, step, lr, 0.9, 0.95, eps)
    assert np.array_equal(T.cpu().numpy().view(np.uint32), T_ref.view(np.uint32))
    assert np.array_equal(md.cpu().numpy().view(np.uint32), m_ref.view(np.uint32))
    assert np.array_equal(vd.cpu().numpy().view(np.uint32), v_ref.view(np.uint32))


def test_encode_targets_adam_sequence_in_place_and_errors():
    """Five updates in a row, T written over the gradient buffer, then selection on the result."""
    from paper_2405_14852_amd import PVError
    wl = workloads.make(64, 512, 8, 1, 4, seed=22, sigma_g=1e-3)
    run = GpuRun(wl)
    rng = np.random.default_rng(22)
    m = np.zeros_like(wl.W)
    v = np.zeros_like(wl.W)
    md, vd = dev_f32(m), dev_f32(v)
    for step in range(1, 6):
        G = (rng.standard_normal(wl.W.shape) * 1e-3).astype(np.float32)
        Gd = dev_f32(G)
        run.ctx.pv_encode_targets_adam(run.lay, run.W, Gd, md, vd, step, 3e-3, 0.9, 0.95, 1e-8, Gd)
        T_ref, m, v = oracle.encode_targets_adam(wl.W, G, m, v, step, 3e-3)
        assert np.array_equal(Gd.cpu().numpy(), T_ref), step
    assert np.array_equal(md.cpu().numpy(), m) and np.array_equal(vd.cpu().numpy(), v)
    idx = run.select(Gd, 50)
    assert np.array_equal(idx, oracle.select_topk_groups(T_ref, wl.W, 8, 50))
    T = torch.empty_like(run.W)
    for bad in (dict(step=0), dict(beta1=1.0), dict(beta2=-0.1)):
        kw = dict(step=1, lr=1e-3, beta1=0.9, beta2=0.95, eps=1e-8)
        kw.update(bad)
        with pytest.raises(PVError):
            run.ctx.pv_encode_targets_adam(run.lay, run.W, Gd, md, vd, kw["step"], kw["lr"],
                                           kw["beta1"], kw["beta2"], kw["eps"], T)
    with pytest.raises(PVError):
        run.ctx.pv_encode_targets_adam(run.lay, run.W, Gd, md, md, 1, 1e-3, 0.9, 0.95, 1e-8, T)


@pytest.mark.parametrize("shape,g", [((256, 256), 8), ((61, 1000), 8), ((33, 4096), 16),
                                     ((129, 4100), 4), ((5, 12), 1), ((100, 36), 6), ((9, 1280), 64)])
@pytest.mark.parametrize("step,frac", [(1, 0.3), (3, 0.01), (50, 1.0), (2, 0.0)])
def test_fused_adam_targets_select_matches_oracle(shape, g, step, frac):
    wl = workloads.make(shape[0], shape[1], g, 1, 4, seed=23, sigma_g=1e-3)
    rng = np.random.default_rng(23)
    m = (rng.standard_normal(shape) * 1e-3).astype(np.float32) if step > 1 else np.zeros(shape, np.float32)
    v = (rng.random(shape) * 1e-6).astype(np.float32) if step > 1 else np.zeros(shape, np.float32)
    run = GpuRun(wl)
    N = wl.layout.num_groups
    k = int(frac * N)
    md, vd = dev_f32(m), dev_f32(v)
    T = torch.empty_like(run.W)
    idx = torch.empty(max(k, 1), dtype=torch.int32, device=DEV)
    sc = torch.empty(N, dtype=torch.float32, device=DEV)
    run.ctx.pv_encode_targets_adam_select(run.lay, run.W, run.G, md, vd, step, 3e-3, 0.9, 0.95, 1e-8,
                                          T, k, idx, sc)
    torch.cuda.synchronize()
    T_ref, m_ref, v_ref = oracle.encode_targets_adam(wl.W, wl.G, m, v, step, 3e-3, 0.9, 0.95, 1e-8)
    idx_ref, sc_ref = oracle.select_topk_groups(T_ref, wl.W, g, k, return_scores=True)
    assert np.array_equal(T.cpu().numpy().view(np.uint32), T_ref.view(np.uint32))
    assert np.array_equal(md.cpu().numpy().view(np.uint32), m_ref.view(np.uint32))
    assert np.array_equal(vd.cpu().numpy().view(np.uint32), v_ref.view(np.uint32))
    assert np.array_equal(sc.cpu().numpy().view(np.uint32), sc_ref.view(np.uint32))
    assert np.array_equal(idx.cpu().numpy()[:k], idx_ref)


# --------------------------------------------------------------- dequantize

@pytest.mark.parametrize("g,M,B", [(8, 1, 8), (8, 2, 8), (16, 1, 12), (8, 1, 16), (2, 1, 3),
                                   (6, 3, 4), (1, 1, 2), (4, 2, 5)])
def test_dequantize_bit_exact(g, M, B):
    wl = workloads.make(67, 24 * g, g, M, B, seed=3)
    run = GpuRun(wl)
    W = run.dequantize(wl.codes)
    ref = oracle.dequantize(wl.codes, wl.codebooks, wl.scales)
    assert np.array_equal(W.view(np.uint32), ref.view(np.uint32))


@pytest.mark.parametrize("shape,B", [((128, 512), 16), ((256, 11008), 16), ((64, 1024), 7)])
def test_dequantize_whole_chunks_of_one_codebook_g8(shape, B):
    """One codebook, g = 8 and a group count that is a multiple of 1024: the kernel that loads
    four codes a lane.  Rows of 1376 groups put row boundaries inside a wave's chunk."""
    wl = workloads.make(shape[0], shape[1], 8, 1, B, seed=29)
    assert wl.layout.num_groups % 1024 == 0
    run = GpuRun(wl)
    W = run.dequantize(wl.codes)
    ref = oracle.dequantize(wl.codes, wl.codebooks, wl.scales)
    assert np.array_equal(W.view(np.uint32), ref.view(np.uint32))
    # the same codes from an array that is not 8-byte aligned: the general kernel, same weights
    flat = wl.codes.reshape(-1)
    big = torch.zeros(flat.size + 8, dtype=torch.int16, device=DEV)
    big[1:1 + flat.size] = torch.from_numpy(flat.view(np.int16)).to(DEV)
    Wd = torch.empty(shape, dtype=torch.float32, device=DEV)
    run.ctx.pv_dequantize(run.lay, big[1:1 + flat.size].view(torch.uint16), run.cb, run.sc, Wd)
    torch.cuda.synchronize()
    assert np.array_equal(Wd.cpu().numpy().view(np.uint32), ref.view(np.uint32))


def test_dequantize_two_codebooks_with_codes_on_an_odd_halfword():
    """The codes of a two-codebook group are read with one 4-byte load when the array allows
    it; an array that starts on an odd 2-byte boundary takes the general kernel: same weights."""
    wl = workloads.make(67, 192, 8, 2, 8, seed=23)
    run = GpuRun(wl)
    flat = wl.codes.reshape(-1)
    big = torch.zeros(flat.size + 8, dtype=torch.int16, device=DEV)
    big[1:1 + flat.size] = torch.from_numpy(flat.view(np.int16)).to(DEV)
    shifted = big[1:1 + flat.size].view(torch.uint16)
    assert shifted.data_ptr() % 4 == 2
    W = torch.empty((67, 192), dtype=torch.float32, device=DEV)
    run.ctx.pv_dequantize(run.lay, shifted, run.cb, run.sc, W)
    torch.cuda.synchronize()
    ref = oracle.dequantize(wl.codes, wl.codebooks, wl.scales)
    assert np.array_equal(W.cpu().numpy().view(np.uint32), ref.view(np.uint32))


@pytest.mark.parametrize("g,M,B", [(8, 1, 8), (8, 2, 8), (16, 1, 12), (6, 3, 4), (1, 1, 2)])
def test_dequantize_groups_updates_only_the_listed_groups(g, M, B):
    wl = workloads.make(67, 24 * g, g, M, B, seed=13)
    run = GpuRun(wl)
    rng = np.random.default_rng(13)
    N = wl.layout.num_groups
    idx = np.sort(rng.choice(N, size=N // 5, replace=False)).astype(np.int32)
    new_codes = wl.codes.copy().reshape(N, M)
    new_codes[idx] = rng.integers(0, 1 << B, size=(len(idx), M), dtype=np.uint16)
    new_codes = new_codes.reshape(wl.codes.shape)
    Wd = dev_f32(oracle.dequantize(wl.codes, wl.codebooks, wl.scales))
    # codes of OTHER groups are scrambled too: they must not be read
    scrambled = new_codes.copy().reshape(N, M)
    other = np.setdiff1d(np.arange(N), idx)
    want = oracle.dequantize(new_codes, wl.codebooks, wl.scales)
    want.reshape(N, g)[other] = oracle.dequantize(wl.codes, wl.codebooks, wl.scales).reshape(N, g)[other]
    scrambled[other] = (scrambled[other] + 1) % (1 << B)
    from gpu_util import dev_i32
    run.ctx.pv_dequantize_groups(run.lay, dev_u16(scrambled.reshape(wl.codes.shape)), run.cb, run.sc,
                                 dev_i32(idx), len(idx), Wd)
    torch.cuda.synchronize()
    assert np.array_equal(Wd.cpu().numpy().view(np.uint32), want.view(np.uint32))


# ---------------------------------------------------------------- selection

@pytest.mark.parametrize("shape,g", [((256, 256), 8), ((61, 1000), 8), ((33, 4096), 16),
                                     ((5, 12), 1), ((100, 36), 6)])
@pytest.mark.parametrize("frac", [0.0, 0.01, 0.3, 1.0])
def test_select_matches_oracle(shape, g, frac):
    wl = workloads.make(shape[0], shape[1], g, 1, 4, seed=4, sigma_g=1e-3)
    run = GpuRun(wl)
    T = run.targets()
    N = wl.layout.num_groups
    k = int(frac * N)
    idx, scores = run.select(T, k, want_scores=True)
    T_ref = oracle.encode_targets(wl.W, wl.G, wl.alpha)
    idx_ref, sc_ref = oracle.select_topk_groups(T_ref, wl.W, g, k, return_scores=True)
    assert np.array_equal(scores.view(np.uint32), sc_ref.view(np.uint32))
    assert np.array_equal(idx, idx_ref)
    # a second call on the same context (histograms must have been left clean)
    idx2 = run.select(T, max(1, k // 2))
    assert np.array_equal(idx2, oracle.select_topk_groups(T_ref, wl.W, g, max(1, k // 2)))


def test_select_ties_lowest_id_first():
    wl = workloads.make(64, 512, 8, 1, 4, seed=5)
    N = wl.layout.num_groups
    W = np.zeros_like(wl.W)
    T = np.zeros_like(wl.W)
    Tg = T.reshape(N, 8)
    Tg[:, 0] = 1.0                       # all scores equal ...
    Tg[np.arange(0, N, 7), 1] = 2.0      # ... except a higher tier
    run = GpuRun(wl)
    Td, Wd = dev_f32(T), dev_f32(W)
    for k in (1, 5, N // 7 + 1, N // 7 + 2, N // 2, N - 1, N):
        idx = run.select(Td, k, W=Wd)
        assert np.array_equal(idx, oracle.select_topk_groups(T, W, 8, k)), k


def test_select_all_zero_scores():
    wl = workloads.make(16, 256, 8, 1, 4, seed=6)
    run = GpuRun(wl)
    idx = run.select(run.W, 10)          # T == W: every score is +0
    assert np.array_equal(idx, np.arange(10, dtype=np.int32))


def test_select_scratch_does_not_depend_on_k():
    """A smaller k on a shape that was seen before allocates nothing (a caller may be capturing)."""
    run = GpuRun(workloads.make(4, 64, 8, 1, 4, seed=4))
    lay = type(run.lay)(2048, 16384, 8, 1, 4)
    W = torch.zeros(2048, 16384, device=DEV)
    T = torch.rand(2048, 16384, device=DEV)
    idx = torch.empty(lay.num_groups, dtype=torch.int32, device=DEV)
    free = []
    for k in (lay.num_groups // 2, lay.num_groups // 100, lay.num_groups, 1):
        run.ctx.pv_select_topk_groups(lay, T, W, k, idx)
        torch.cuda.synchronize()
        free.append(torch.cuda.mem_get_info()[0])
    assert min(free) == max(free), free


def test_select_without_memory_for_its_lists():
    """The lists of candidates take 2 bytes a group: where the device has no room for them the
    selection does without, also in later calls."""
    run = GpuRun(workloads.make(4, 64, 8, 1, 4, seed=4))
    rows = columns = 1 << 14
    lay, small = type(run.lay)(rows, columns, 1, 1, 4), type(run.lay)(256, 256, 1, 1, 4)
    W = torch.zeros(rows, columns, device=DEV)
    T = torch.zeros(rows, columns, device=DEV)
    scores = torch.empty(rows * columns, device=DEV)
    rng = np.random.default_rng(5)
    at = np.unique(rng.integers(0, rows * columns, 4000)).astype(np.int32)
    T.view(-1)[dev_i32(at).long()] = dev_f32(rng.uniform(1.0, 2.0, at.size))
    idx = torch.empty(at.size, dtype=torch.int32, device=DEV)
    run.ctx.pv_select_topk_groups(small, T, W, 256, idx, scores)       # loads the kernels
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    fill = []
    while torch.cuda.mem_get_info()[0] > 400 << 20:       # the lists of 2^28 groups take 512 MiB
        fill.append(torch.empty(torch.cuda.mem_get_info()[0] - (300 << 20), dtype=torch.uint8, device=DEV))
    try:
        for _ in range(2):
            idx.fill_(-1)
            run.ctx.pv_select_topk_groups(lay, T, W, at.size, idx, scores)
            torch.cuda.synchronize()
            assert np.array_equal(idx.cpu().numpy(), at)
    finally:
        del fill
        torch.cuda.empty_cache()


# ------------------------------------------- targets + selection in one sweep

@pytest.mark.parametrize("N", [255, 4097, 24575, 24576, 24577, 32767, 32768, 32769, 40001, 262145, 1050001, 9000001])
@pytest.mark.parametrize("values", ["spread", "narrow", "equal", "clustered"])
def test_select_on_both_sides_of_its_dispatch(N, values):
    """One block up to 24 576 groups, three kernels beyond; a wave's list of candidates fits,
    overflows (many keys in one digit, large scores next to each other) or is not kept (large k)."""
    rng = np.random.default_rng(N)
    W = np.zeros((1, N), np.float32)
    if values == "spread":
        T = rng.standard_normal((1, N)).astype(np.float32)
    elif values == "narrow":
        T = (1.0 + 1e-5 * rng.random((1, N))).astype(np.float32)
    elif values == "equal":
        T = np.full((1, N), 0.5, np.float32)
    else:
        T = (1e-3 * rng.standard_normal((1, N))).astype(np.float32)
        T[0, N // 3:N // 3 + N // 20] += 1.0
    wl = workloads.make(1, N, 1, 1, 4, seed=4)
    run = GpuRun(wl)
    run.W = dev_f32(W)
    for k in sorted({1, N // 100 + 1, N // 8, N // 8 + 1, N - 1, N}):
        idx = run.select(dev_f32(T), k)
        assert np.array_equal(idx, oracle.select_topk_groups(T, W, 1, k)), (N, values, k)


@pytest.mark.parametrize("shape,g", [((256, 256), 8), ((61, 1000), 8), ((33, 4096), 16),
                                     ((129, 4100), 4), ((5, 12), 1), ((100, 36), 6),
                                     ((17, 640), 32), ((9, 1280), 64),
                                     ((301, 4099), 1), ((257, 2050), 2), ((3, 7), 1), ((1, 2), 2)])
@pytest.mark.parametrize("frac,alpha", [(0.0, 1.0), (0.01, 1.0), (0.3, 0.37), (1.0, 1.0)])
def test_fused_targets_select_matches_oracle(shape, g, frac, alpha):
    wl = workloads.make(shape[0], shape[1], g, 1, 4, seed=14, sigma_g=1e-3)
    run = GpuRun(wl)
    N = wl.layout.num_groups
    k = int(frac * N)
    T, idx, scores = run.targets_select(k, alpha=alpha, want_scores=True)
    T_ref = oracle.encode_targets(wl.W, wl.G, alpha)
    idx_ref, sc_ref = oracle.select_topk_groups(T_ref, wl.W, g, k, return_scores=True)
    assert np.array_equal(T.cpu().numpy().view(np.uint32), T_ref.view(np.uint32))
    assert np.array_equal(scores.view(np.uint32), sc_ref.view(np.uint32))
    assert np.array_equal(idx, idx_ref)
    # the two separate calls on the same context give the same ids afterwards
    idx2 = run.select(run.targets(alpha), k)
    assert np.array_equal(idx2, idx_ref)


def test_fused_targets_select_in_place_over_gradient_and_errors():
    wl = workloads.make(64, 512, 8, 1, 4, seed=15, sigma_g=1e-3)
    run = GpuRun(wl)
    k = 40
    T_ref = oracle.encode_targets(wl.W, wl.G, 0.5)
    idx_ref = oracle.select_topk_groups(T_ref, wl.W, 8, k)
    Gd = run.G.clone()
    idx = torch.empty(k, dtype=torch.int32, device=DEV)
    run.ctx.pv_encode_targets_select(run.lay, run.W, Gd, 0.5, Gd, k, idx)   # T written over G
    torch.cuda.synchronize()
    assert np.array_equal(Gd.cpu().numpy(), T_ref)
    assert np.array_equal(idx.cpu().numpy(), idx_ref)
    from paper_2405_14852_amd import PVError
    with pytest.raises(PVError):
        run.ctx.pv_encode_targets_select(run.lay, run.W, run.G, 0.5, run.W, k, idx)   # T aliases W
    with pytest.raises(PVError):
        run.ctx.pv_encode_targets_select(run.lay, run.W, run.G, 0.5, Gd, -1, idx)
    with pytest.raises(PVError):
        run.ctx.pv_encode_targets_select(run.lay, run.W, run.G, 0.5, Gd,
                                         wl.layout.num_groups + 1, idx)


# ---------------------------------------------------------- re-encode, M = 1

def reencode_case(wl, mode, idx=None, T_np=None):
    run = GpuRun(wl)
    run.ctx.pv_set_search_mode(mode)
    if T_np is None:
        T_np = oracle.encode_targets(wl.W, wl.G, wl.alpha)
    if idx is None:
        idx = oracle.select_topk_groups(T_np, wl.W, wl.layout.group_size, wl.k)
    got, nch = run.reencode(dev_f32(T_np), idx)
    want, info = oracle.reencode_groups(T_np, wl.codebooks, wl.scales, idx, wl.codes,
                                        beam_width=wl.beam_width)
    ndiff = check_codes(wl, T_np, idx, got, want, info)
    if ndiff == 0:
        assert nch == info["num_changed"]
    return run, got, want, info


def check_route(run, k, filtered):
    """The last search (mode 0, one codebook, k listed groups): a matrix-core filter took it (as several launches or as one,
    see check_launches), or the one launch that evaluates everything did."""
    st = run.ctx.pv_reencode_stats()
    assert (st["filtered"] + st["fallback"], st["exact"]) == ((k, 0) if filtered else (0, k))


def check_launches(run, T_np, idx, several):
    """The search of this list in mode 0, once more and timed: the filter that prepares, contracts and re-ranks in launches of
    their own, or one launch that does it all for a codebook that fits the LDS (the counters tell the same of both)."""
    run.ctx.pv_set_search_mode(0)
    run.ctx.pv_timing_enable(True)
    run.ctx.pv_timing_reset()
    run.reencode(dev_f32(T_np), idx)
    n = {name: run.ctx.pv_timing_read(name)[1] for name in ("prep", "score_mfma", "rerank", "exact_scan")}
    run.ctx.pv_timing_enable(False)
    assert n == {"prep": int(several), "score_mfma": 1, "rerank": int(several), "exact_scan": 0}


@pytest.mark.parametrize("mode", [1, 0])
@pytest.mark.parametrize("g,B,shape,tau", [
    (8, 8, (256, 256), 1.0),        # config 1 as stated
    (8, 16, (64, 1024), 0.3),       # 1x16, several tiles + ragged tail of selected groups
    (16, 16, (48, 1024), 0.4),      # 1-bit config shape
    (16, 14, (48, 1024), 0.4),      # 14-bit codebook over groups of 16 (0.875 bit, App. K / Sec. 4.4)
    (8, 14, (40, 512), 0.5),        # 14 bits over groups of 8
    (8, 12, (32, 264), 1.0),
    (16, 5, (16, 256), 1.0),
    (4, 3, (8, 64), 1.0),
    (1, 2, (4, 16), 1.0),
    (8, 1, (4, 64), 1.0),
    (32, 6, (8, 512), 1.0),         # group sizes beyond the matrix-core filter: exact scan
    (64, 4, (8, 1024), 1.0),        # the largest group size
    (12, 5, (8, 240), 1.0),         # a group size that is no multiple of four
])
def test_reencode_m1_matches_oracle(mode, g, B, shape, tau):
    wl = workloads.make(shape[0], shape[1], g, 1, B, seed=7, sigma_g=2e-3, tau=tau)
    reencode_case(wl, mode)


@pytest.mark.parametrize("g", [8, 16])
@pytest.mark.parametrize("k", [1, 31, 32, 33, 511, 512, 513, 4095, 4096, 4097, 4609, 8200])
def test_reencode_m1_list_lengths_around_the_launch_plan(g, k):
    """2048 codewords fit the LDS: one launch, whose batches and blocks change with the list length."""
    wl = workloads.make(96, 96 * g, g, 1, 11, seed=50, sigma_g=2e-3, tau=1.0)
    T_np = oracle.encode_targets(wl.W, wl.G, wl.alpha)
    idx = np.sort(np.random.default_rng(k).choice(wl.layout.num_groups, size=k, replace=False)).astype(np.int32)
    run, got, want, info = reencode_case(wl, 0, idx=idx, T_np=T_np)
    st = run.ctx.pv_reencode_stats()
    assert st["filtered"] + st["fallback"] == k
    check_launches(run, T_np, idx, several=False)


@pytest.mark.parametrize("g,B", [(8, 13), (16, 12)])
@pytest.mark.parametrize("k", [1, 31, 32, 33, 511, 512, 513, 4095, 4096, 4097, 4609, 8200, 32768, 43521, 65536, 65537, 131073])
def test_reencode_m1_list_lengths_around_the_filters_launch_plan(g, B, k):
    """The plan of the filter in several launches changes with the list length (group tiles per wave, codeword
    splits, merged partitions, padded tail): lengths on both sides of every switch.  Codes and count equal the exact scan's,
    a sample the oracle's."""
    wl = workloads.make(96 if k < 9000 else 1366, 96 * g, g, 1, B, seed=50, sigma_g=2e-3, tau=1.0)
    T_np = oracle.encode_targets(wl.W, wl.G, wl.alpha)
    rng = np.random.default_rng(k)
    idx = np.sort(rng.choice(wl.layout.num_groups, size=k, replace=False)).astype(np.int32)
    run, T = GpuRun(wl), dev_f32(T_np)
    run.ctx.pv_set_search_mode(1)
    want, n_want = run.reencode(T, idx)
    run.ctx.pv_set_search_mode(0)
    got, n_got = run.reencode(T, idx)
    assert np.array_equal(got, want) and n_got == n_want
    check_route(run, k, filtered=True)
    check_launches(run, T_np, idx, several=True)
    sub = np.sort(rng.choice(idx, size=min(k, 256), replace=False))
    ref, info = oracle.reencode_groups(T_np, wl.codebooks, wl.scales, sub, wl.codes)
    check_codes_on(wl, T_np, sub, got, ref, info)


@pytest.mark.parametrize("g,B,k", [(8, 6, 1), (8, 6, 16384), (8, 7, 13), (8, 8, 8191), (8, 8, 16385), (8, 9, 4095),
                                   (8, 9, 4096), (8, 9, 16384), (8, 10, 3), (8, 10, 8192), (8, 10, 8193), (16, 6, 5),
                                   (16, 8, 4097), (16, 9, 16384), (16, 9, 4094), (16, 10, 8192), (16, 10, 8193)])
@pytest.mark.parametrize("case", ["plain", "ties", "odd"])
def test_reencode_m1_in_one_launch(g, B, k, case):
    """Little work is one launch: lists that end inside a wave's and a block's groups, both sides of the
    line and of the split of the codebook over a block's waves; exact ties (equal codewords, targets on them);
    codewords and targets that are not finite, scales of zero and below, ids outside the matrix, stored codes
    above 2^B.  Codes and count equal the exact scan's, twice in a row (the counters are left zero)."""
    wl = workloads.make(160, 128 * g, g, 1, B, seed=97, sigma_g=2e-3, tau=1.0)
    rng = np.random.default_rng(k)
    if case == "ties":
        wl.codebooks[0, 1::2] = wl.codebooks[0, ::2]
        wl.codebooks[0, -3:] = 0.0
    T_np = oracle.encode_targets(wl.W, wl.G, wl.alpha)
    if case == "ties":
        T_np[::3] = 0.0
    idx = np.sort(rng.choice(wl.layout.num_groups, size=k, replace=False)).astype(np.int32)
    if case == "odd":
        wl.scales[::5] = 0.0
        wl.scales[1::5] *= np.float32(-1.0)
        wl.codebooks[0, 3, 1], wl.codebooks[0, 5, 0] = np.nan, np.inf
        T_np[2, 7], T_np[9] = np.inf, np.nan
        wl.codes[::7] |= np.uint16(1 << B)
        idx = np.sort(np.where(rng.random(k) < 0.1, idx + wl.layout.num_groups, idx)).astype(np.int32)
    run, T = GpuRun(wl), dev_f32(T_np)
    run.ctx.pv_set_search_mode(1)
    want, n_want = run.reencode(T, idx)
    run.ctx.pv_set_search_mode(0)
    for _ in range(2):
        got, n_got = run.reencode(T, idx)
        assert np.array_equal(got, want) and n_got == n_want
    st = run.ctx.pv_reencode_stats()
    valid = int((idx < wl.layout.num_groups).sum())
    if k <= 16384 and k * g << B <= (1 << 26 if g == 8 else 1 << 27):
        assert st["exact"] == valid and st["filtered"] == st["fallback"] == 0
    if case != "odd":
        ref, info = oracle.reencode_groups(T_np, wl.codebooks, wl.scales, idx, wl.codes)
        check_codes_on(wl, T_np, idx, got, ref, info)


@pytest.mark.parametrize("g,B,k", [(8, 8, 16385), (8, 8, 131077), (8, 9, 16385), (8, 10, 8193), (8, 11, 1), (8, 11, 33),
                                   (8, 11, 32769), (8, 12, 31), (8, 12, 16449), (16, 8, 16385), (16, 9, 16385),
                                   (16, 10, 8193), (16, 11, 65), (16, 11, 16449),
                                   # a batch more than there are blocks, in every form
                                   (8, 9, 65569), (8, 10, 32801), (16, 8, 98337), (16, 9, 65569), (16, 10, 32801)])
@pytest.mark.parametrize("case", ["plain", "ties", "odd"])
def test_reencode_m1_small_codebook(g, B, k, case):
    """Codebooks that fit the LDS: the filter in one launch.  Lists that end inside a tile of groups, a block's groups
    and a second round of the blocks; exact ties, several equal codewords behind one key and in one partition; codewords
    and targets that are not finite, scales of zero and below, targets far outside, ids outside the matrix, stored codes above
    2^B.  Codes and count equal the exact scan's, twice in a row (the counters are left zero)."""
    wl = workloads.make(160 if k < 20000 else 1040, 128 * g, g, 1, B, seed=101, sigma_g=2e-3, tau=1.0)
    rng = np.random.default_rng(k)
    if case == "ties":
        wl.codebooks[0, 1::2] = wl.codebooks[0, ::2]
        wl.codebooks[0, -40:] = 0.0
    T_np = oracle.encode_targets(wl.W, wl.G, wl.alpha)
    if case == "ties":
        T_np[::3] = 0.0
    idx = np.sort(rng.choice(wl.layout.num_groups, size=k, replace=False)).astype(np.int32)
    if case == "odd":
        wl.scales[::5] = 0.0
        wl.scales[1::5] *= np.float32(-1.0)
        wl.scales[2::5] *= np.float32(1e-3)
        if k % 2:
            wl.codebooks[0, 3, 1], wl.codebooks[0, 5, 0] = np.nan, np.inf
        T_np[2, 7], T_np[9] = np.inf, np.nan
        wl.codes[::7] |= np.uint16(1 << B)
        idx = np.sort(np.where(rng.random(k) < 0.1, idx + wl.layout.num_groups, idx)).astype(np.int32)
    run, T = GpuRun(wl), dev_f32(T_np)
    run.ctx.pv_set_search_mode(1)
    want, n_want = run.reencode(T, idx)
    run.ctx.pv_set_search_mode(0)
    for _ in range(2):
        got, n_got = run.reencode(T, idx)
        assert np.array_equal(got, want) and n_got == n_want
    st = run.ctx.pv_reencode_stats()
    valid = int((idx < wl.layout.num_groups).sum())
    assert st["filtered"] + st["fallback"] == valid and st["exact"] == 0
    assert case != "plain" or st["fallback"] < 0.02 * k + 2      # the certificate holds for nearly every group
    if case != "odd" and k < 20000:
        ref, info = oracle.reencode_groups(T_np, wl.codebooks, wl.scales, idx, wl.codes)
        check_codes_on(wl, T_np, idx, got, ref, info)


@pytest.mark.parametrize("g,B", [(8, 8), (8, 9), (8, 10), (8, 11), (8, 12), (16, 8), (16, 9), (16, 10), (16, 11)])
@pytest.mark.parametrize("case", ["one_large", "decades", "clusters", "far"])
def test_reencode_m1_small_codebook_much_within_reach(g, B, case):
    """Codebooks whose largest codeword leaves the others little of the fp16 range, tight clusters, targets far outside: many
    keys and partitions can hold the nearest.  Codes and count equal the exact scan's, and what is evaluated in double stays the
    32 codewords behind the best key and little else (beyond the fp16 range: everything)."""
    k = 16449
    wl = workloads.make(160, 128 * g, g, 1, B, seed=105, sigma_g=0.016 * 2.0 ** (-B / g), tau=1.0)
    rng = np.random.default_rng(B)
    cb = wl.codebooks[0]
    if case == "one_large":
        cb[7] *= np.float32(100.0)
    elif case == "decades":
        cb /= (rng.random((len(cb), 1)) ** 0.7 + 1e-3).astype(np.float32)
    elif case == "clusters":
        cb[:] = cb[np.arange(len(cb)) % 64] + (2e-5 * rng.standard_normal(cb.shape)).astype(np.float32)
    else:
        wl.scales[::3] *= np.float32(1e-4)
    wl.W[:] = oracle.dequantize(wl.codes, wl.codebooks, wl.scales)
    if case == "far":
        wl.W[::6] += np.float32(0.02)
    T_np = oracle.encode_targets(wl.W, wl.G, wl.alpha)
    idx = np.sort(rng.choice(wl.layout.num_groups, size=k, replace=False)).astype(np.int32)
    run, T = GpuRun(wl), dev_f32(T_np)
    run.ctx.pv_set_search_mode(1)
    want, n_want = run.reencode(T, idx)
    run.ctx.pv_set_search_mode(0)
    got, n_got = run.reencode(T, idx)
    assert np.array_equal(got, want) and n_got == n_want
    st = run.ctx.pv_reencode_stats()
    assert st["filtered"] + st["fallback"] == k and st["exact"] == 0
    assert case == "far" or st["reranked_candidates"] <= 48 * k


@pytest.mark.parametrize("B,k", [(12, 2051), (14, 32767), (12, 32768), (13, 32785), (16, 33001)])
@pytest.mark.parametrize("case", ["plain", "ties", "odd"])
def test_reencode_m1_g16_row_of_lanes_a_codeword(B, k, case):
    """Groups of 16 behind the filter, up to 32767 a lane a codeword, above a row of lanes.  Several codewords of a lane and of a
    row within reach (ties), partitions left open, values that are not finite, scales of zero and below, ids outside the
    matrix.  Codes and count equal the exact scan's."""
    wl = workloads.make(320, 2048, 16, 1, B, seed=103, sigma_g=2e-3, tau=1.0)
    rng = np.random.default_rng(k)
    if case == "ties":
        wl.codebooks[0, 1::2] = wl.codebooks[0, ::2]
        wl.codebooks[0, -40:] = 0.0
    T_np = oracle.encode_targets(wl.W, wl.G, wl.alpha)
    if case == "ties":
        T_np[::3] = 0.0
    idx = np.sort(rng.choice(wl.layout.num_groups, size=k, replace=False)).astype(np.int32)
    if case == "odd":
        wl.scales[::5] = 0.0
        wl.scales[1::5] *= np.float32(-1.0)
        wl.scales[2::5] *= np.float32(1e-3)
        if k % 2:
            wl.codebooks[0, 3, 1], wl.codebooks[0, 5, 0] = np.nan, np.inf
        T_np[2, 7], T_np[9] = np.inf, np.nan
        idx = np.sort(np.where(rng.random(k) < 0.1, idx + wl.layout.num_groups, idx)).astype(np.int32)
    run, T = GpuRun(wl), dev_f32(T_np)
    run.ctx.pv_set_search_mode(1)
    want, n_want = run.reencode(T, idx)
    run.ctx.pv_set_search_mode(0)
    got, n_got = run.reencode(T, idx)
    assert np.array_equal(got, want) and n_got == n_want
    st = run.ctx.pv_reencode_stats()
    valid = int((idx < wl.layout.num_groups).sum())
    assert st["filtered"] + st["fallback"] == valid and st["exact"] == 0
    assert st["reranked_candidates"] <= 64 * valid       # what the team looks at beside the open partitions


@pytest.mark.parametrize("case", ["zeros", "clusters"])
def test_reencode_m1_g16_many_codewords_within_reach(case):
    """Many codewords of a row of lanes need their exact objective (a third of the codebook unused and zero; codewords in
    tight clusters): the row takes them a lane each.  Codes equal the exact scan's, and a list of the length from which on rows
    of lanes share a codeword costs what one group less does (one after the other by the row: 3 to 4 times as much)."""
    wl = workloads.make(320, 2048, 16, 1, 12, seed=104, sigma_g=1e-2, tau=1.0)
    rng = np.random.default_rng(104)
    cb = wl.codebooks[0]
    if case == "zeros":
        cb[rng.permutation(4096)[:1229]] = 0.0
    else:
        cb[:] = cb[rng.integers(0, 64, size=4096)] + (2e-5 * rng.standard_normal(cb.shape)).astype(np.float32)
    wl.W[:] = oracle.dequantize(wl.codes, wl.codebooks, wl.scales)
    T_np = oracle.encode_targets(wl.W, wl.G, wl.alpha)
    idx = np.sort(rng.choice(wl.layout.num_groups, size=32768, replace=False)).astype(np.int32)
    run, T = GpuRun(wl), dev_f32(T_np)
    run.ctx.pv_set_search_mode(1)
    want, n_want = run.reencode(T, idx)
    run.ctx.pv_set_search_mode(0)
    got, n_got = run.reencode(T, idx)
    assert np.array_equal(got, want) and n_got == n_want
    ids, codes, took = dev_i32(idx), run.codes.clone(), {32767: [], 32768: []}
    for k in (32767, 32768) * 8:
        codes.copy_(run.codes)
        start, stop = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        start.record()
        run.ctx.pv_reencode_groups(run.lay, T, run.cb, run.sc, ids, k, 1, codes)
        stop.record()
        torch.cuda.synchronize()
        took[k].append(start.elapsed_time(stop))
    assert np.median(took[32768]) < 1.5 * np.median(took[32767])


def test_reencode_m1_of_a_smaller_k_can_be_captured():
    """The shape was seen with a list that the filter takes; a short list goes another way, and a captured
    call cannot allocate.  The replay also after the context counted something else."""
    wl = workloads.make(160, 1024, 8, 1, 8, seed=98, tau=1.0, sigma_g=2e-3)
    N, k = wl.layout.num_groups, 8192
    side = torch.cuda.Stream(device=DEV)
    run = GpuRun(wl, PVContext(0, stream=side))
    T_np = oracle.encode_targets(wl.W, wl.G, wl.alpha)
    T, idx = dev_f32(T_np), dev_i32(np.arange(N, dtype=np.int32))
    count = torch.zeros(1, dtype=torch.int64, device=DEV)
    first, codes = run.codes.clone(), run.codes.clone()
    torch.cuda.synchronize()
    run.ctx.pv_reencode_groups(run.lay, T, run.cb, run.sc, idx, N, 1, first, count)
    side.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        run.ctx.pv_reencode_groups(run.lay, T, run.cb, run.sc, idx, k, 1, codes, count)
    ids = np.arange(k, dtype=np.int32)
    want, info = oracle.reencode_groups(T_np, wl.codebooks, wl.scales, ids, wl.codes)
    for rep in range(3):
        codes.view(torch.int16).copy_(run.codes.view(torch.int16))
        count.fill_(-5)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        check_codes(wl, T_np, ids, host_u16(codes), want, info)
        assert int(count.item()) == int((host_u16(codes) != wl.codes).sum()) > 0
        run.ctx.pv_reencode_groups(run.lay, T, run.cb, run.sc, idx, 77 + rep, 1, first, count)
        side.synchronize()


@pytest.mark.parametrize("g,k", [(8, 1), (8, 127), (8, 128), (8, 129), (8, 98304), (8, 98305), (8, 131072),
                                 (16, 1), (16, 15), (16, 17), (16, 8192), (16, 8193), (16, 65536)])
@pytest.mark.parametrize("left", ["all", "some", "none"])
def test_reencode_m2_lists_for_the_exact_kernel(g, k, left):
    """What the filter of the two-codebook search leaves goes into a list a block: nothing, every group of
    every block (a codeword that is not finite), some; list lengths around a block's groups, a launch's blocks and a
    second round of them.  Codes and count equal the exact kernel's, whatever call came before."""
    wl = workloads.make(1024, 1024, g, 2, 8, seed=99, sigma_g=2e-3, tau=1.0)
    rng = np.random.default_rng(k)
    T_np = oracle.encode_targets(wl.W, wl.G, wl.alpha)
    if left == "all":
        wl.codebooks[1, 9, 2] = np.inf
    elif left == "some":
        T_np[::3, 5::g] = np.nan
    idx = np.sort(rng.choice(wl.layout.num_groups, size=k, replace=False)).astype(np.int32)
    run, T = GpuRun(wl), dev_f32(T_np)
    run.ctx.pv_set_search_mode(1)
    want, n_want = run.reencode(T, idx, beam_width=8)
    run.ctx.pv_set_search_mode(0)
    for _ in range(2):
        got, n_got = run.reencode(T, idx, beam_width=8)
        assert np.array_equal(got, want) and n_got == n_want
        st = run.ctx.pv_reencode_stats()
        assert st["filtered"] + st["fallback"] == k and st["exact"] == 0
        assert left != "all" or st["filtered"] == 0
        run.reencode(T, idx[: (k + 1) // 2], beam_width=4)


@pytest.mark.parametrize("B,k", [(16, 32768), (16, 34001), (15, 65536), (14, 131072)])
@pytest.mark.parametrize("regime", ["near", "far", "lumps", "degenerate"])
def test_reencode_m1_cells_of_the_codebook(B, k, regime):
    """Lists long enough for the search that leaves out whole cells: current codes near the targets,
    current codes drawn at random (the dense contraction takes over), a codebook of two lumps and
    constant coordinates (few, crowded cells), groups that the filter does not take."""
    wl = workloads.make(256, 8 * ((k + 255) // 256 + 3), 8, 1, B, seed=70, sigma_g=4e-3, tau=1.0)
    if regime == "lumps":
        wl.codebooks[0, : 1 << (B - 1)] *= np.float32(0.05)
        wl.codebooks[0, : 1 << (B - 1)] += np.float32(0.06)
        wl.codebooks[0, :, 2] = np.float32(0.01)
        wl.codebooks[0, 1:200] = wl.codebooks[0, 0]
    if regime == "degenerate":
        wl.scales[::5] = 0.0
        wl.scales[1::5] *= np.float32(-1e-3)
    if regime != "far":
        wl.W = oracle.dequantize(wl.codes, wl.codebooks, wl.scales)
    T_np = oracle.encode_targets(wl.W, wl.G, wl.alpha)
    if regime == "degenerate":
        T_np[3, ::7] = np.float32(1e30)
    N = wl.layout.num_groups
    idx = np.sort(np.random.default_rng(k).choice(N, size=k, replace=False)).astype(np.int32)
    reencode_case(wl, 0, idx=idx, T_np=T_np)


def _cells_case(k, B, regime, seed, g=8):
    wl = workloads.make(512, g * ((k + 511) // 512 + 3), g, 1, B, seed=seed, sigma_g=4e-3, tau=1.0)
    if regime == "near":
        wl.W = oracle.dequantize(wl.codes, wl.codebooks, wl.scales)
    T_np = oracle.encode_targets(wl.W, wl.G, wl.alpha)
    idx = np.sort(np.random.default_rng(k).choice(wl.layout.num_groups, size=k, replace=False)).astype(np.int32)
    return wl, T_np, idx


@pytest.mark.parametrize("B,k", [(16, 112721), (15, 150001), (14, 262145)])
@pytest.mark.parametrize("regime", ["near", "far"])
def test_reencode_m1_cells_with_more_items_than_blocks(B, k, regime):
    """Lists so long that a scoring block takes several work items, of cells (more than 256: near) and of
    the dense contraction (more than 512: far).  A sample of the groups is checked."""
    wl, T_np, idx = _cells_case(k, B, regime, 72)
    run = GpuRun(wl)
    got, nch = run.reencode(dev_f32(T_np), idx)
    sub = idx[::k // 4000]
    want, info = oracle.reencode_groups(T_np, wl.codebooks, wl.scales, sub, wl.codes)
    check_codes_on(wl, T_np, sub, got, want, info)
    mask = np.ones(wl.layout.num_groups, bool)
    mask[idx] = False
    assert np.array_equal(got.ravel()[mask], wl.codes.ravel()[mask])
    assert nch == (got != wl.codes).sum()


@pytest.mark.parametrize("codewords", ["finite", "some_not"])
def test_reencode_m1_cells_non_finite_inputs(codewords):
    """Targets, scales and codewords that are not finite, in lists that the cells take: such groups are
    searched in full, as the oracle does, and the others as ever."""
    wl, T_np, idx = _cells_case(33000, 16, "near", 74)
    T_np[3, ::11] = np.nan
    T_np[5, ::9] = np.inf
    T_np[7, ::9] = -3e38
    wl.scales[[9, 11, 13, 15]] = [np.inf, np.nan, 0.0, 1e-38]
    if codewords == "some_not":
        wl.codebooks[0, 7, 2] = np.nan
        wl.codebooks[0, 300, 5] = np.inf
        wl.codebooks[0, 65535, 0] = -np.inf
        wl.codes[20:24, :8] = np.uint16(300)
        wl.codes[24:28, :8] = np.uint16(7)
    got, _ = GpuRun(wl).reencode(dev_f32(T_np), idx)
    gpr = wl.layout.groups_per_row
    odd = [n for n in idx if n // gpr < 30]
    sub = np.sort(np.unique(np.concatenate([np.array(odd, np.int32), idx[::16]])))
    want, info = oracle.reencode_groups(T_np, wl.codebooks, wl.scales, sub, wl.codes)
    check_codes_on(wl, T_np, sub, got, want, info)


def test_reencode_m1_on_one_context_equals_fresh_contexts():
    """What a context keeps between calls (counters of cells and of norm buckets that are left at zero,
    scratch that grows) makes no difference, whichever of the ways through the search comes next."""
    from paper_2405_14852_amd import PVContext
    cases = [(8, 16, 40000, "near"), (8, 16, 40000, "far"), (8, 16, 33000, "near"), (8, 14, 140000, "near"),
             (16, 12, 6000, "far"), (8, 15, 70000, "near"), (8, 8, 3000, "near"), (16, 16, 5000, "near"),
             (8, 14, 140000, "far"), (16, 10, 700, "far"), (8, 12, 5000, "near"), (16, 12, 6000, "far"),
             (8, 16, 40000, "near")]
    shared = PVContext(0)
    known = {}
    for case in cases:
        g, B, k, regime = case
        wl, T_np, idx = _cells_case(k, B, regime, 73, g)
        if case not in known:
            known[case] = GpuRun(wl).reencode(dev_f32(T_np), idx)
        got, nch = GpuRun(wl, shared).reencode(dev_f32(T_np), idx)
        assert np.array_equal(got, known[case][0]) and nch == known[case][1], case
    shared.close()


@pytest.mark.parametrize("g", [8, 16])
@pytest.mark.parametrize("B", [5, 7, 10, 11, 13, 14])
@pytest.mark.parametrize("norms", ["one", "spread", "tiny"])
def test_reencode_m1_codebook_preparation(g, B, norms):
    """Every way of taking the codebook's statistics (in the preparing launch, in one before it, or all in one launch: 10 and
    11 bits), and norms on which the norm ordering is put to the test: all alike, far beyond a sample's, at the bottom of float32."""
    # (128 and 1024 codewords: more groups than the launch that evaluates everything takes)
    wl = workloads.make({7: 512, 10: 256}.get(B, 64), 64 * g, g, 1, B, seed=71, sigma_g=4e-3, tau=0.55)
    if norms == "one":
        wl.codebooks[:] = np.float32(0.02) * np.sign(wl.codebooks)
    if norms == "spread":
        wl.codebooks[0, 3::41] *= np.float32(30.0)
        wl.codebooks[0, 5::43] *= np.float32(1e-3)
        wl.codebooks[0, 7] = np.float32(0.0)
    if norms == "tiny":
        wl.codebooks *= np.float32(1e-14)
        wl.scales *= np.float32(1e14)
    run, *_ = reencode_case(wl, 0)
    check_route(run, wl.k, filtered=True)
    T_np = oracle.encode_targets(wl.W, wl.G, wl.alpha)
    check_launches(run, T_np, oracle.select_topk_groups(T_np, wl.W, g, wl.k), several=B not in (10, 11))


@pytest.mark.parametrize("B,rows", [(5, 64), (6, 64), (9, 64), (13, 64), (16, 64), (6, 256), (9, 256)])
def test_reencode_m1_codebook_sizes_with_long_lists(B, rows):
    """More than 4096 listed groups (two group tiles per wave) at every codebook size class; up to 16384 of
    small ones are one launch."""
    wl = workloads.make(rows, 1024, 8, 1, B, seed=51, sigma_g=2e-3, tau=0.6)
    assert wl.k > 4096
    run, *_ = reencode_case(wl, 0)
    check_route(run, wl.k, filtered=rows == 256 or B not in (6, 9))


@pytest.mark.parametrize("seed", range(14))
def test_reencode_m1_filter_agrees_with_the_exact_scan_on_large_lists(seed):
    """Tens of thousands of groups per case, varied gradient sizes, scale and codebook spreads:
    the matrix-core filter with its certificate (mode 0; one launch below 13 bits, g = 16: 12, several from there) and the
    exact scan (mode 1) must write identical codes; a sample is checked against the oracle as well."""
    rng = np.random.default_rng(2000 + seed)
    g = 8 if seed % 2 == 0 else 16
    B = int(rng.integers(9, 14)) if seed < 8 else int(rng.integers(13, 15)) if g == 8 else int(rng.integers(12, 15))
    wl = workloads.make(256, 128 * g, g, 1, B, seed=90 + seed, sigma_g=float(10.0 ** rng.uniform(-4, -2)),
                        sigma_c=float(10.0 ** rng.uniform(-2.5, -1.0)), tau=0.7)
    wl.scales *= np.float32(10.0 ** rng.uniform(-1, 1))
    if seed % 3 == 0:
        wl.scales[rng.integers(0, 256, size=20)] *= np.float32(-1.0)
    T_np = oracle.encode_targets(wl.W, wl.G, wl.alpha)
    idx = oracle.select_topk_groups(T_np, wl.W, g, wl.k)
    run = GpuRun(wl)
    T = dev_f32(T_np)
    run.ctx.pv_set_search_mode(1)
    exact, n_exact = run.reencode(T, idx)
    run.ctx.pv_set_search_mode(0)
    fast, n_fast = run.reencode(T, idx)
    st = run.ctx.pv_reencode_stats()
    assert np.array_equal(fast, exact) and n_fast == n_exact
    assert st["filtered"] + st["fallback"] == wl.k
    check_launches(run, T_np, idx, several=B >= (13 if g == 8 else 12))
    sub = np.sort(rng.choice(idx, size=512, replace=False))
    want, info = oracle.reencode_groups(T_np, wl.codebooks, wl.scales, sub, wl.codes)
    check_codes_on(wl, T_np, sub, fast, want, info)


@pytest.mark.parametrize("mode", [1, 0])
# everything evaluated in one launch, the filter in one (twice), the filter in several (twice)
@pytest.mark.parametrize("g,B", [(8, 10), (8, 11), (16, 11), (8, 13), (16, 12)])
def test_reencode_m1_scale_edge_cases(mode, g, B):
    wl = workloads.make(32, 64 * g, g, 1, B, seed=8, sigma_g=2e-3, tau=1.0)
    wl.scales[3] = 0.0          # every code ties: previous code kept
    wl.scales[5] = -0.9         # negative scale
    wl.scales[7] = 1e-6         # targets far outside the codebook's range after normalisation
    wl.scales[9] = 300.0
    run, got, want, _ = reencode_case(wl, mode)
    if mode == 0:
        check_route(run, wl.k, filtered=B >= 11)
    if B >= 11:
        T_np = oracle.encode_targets(wl.W, wl.G, wl.alpha)
        check_launches(run, T_np, oracle.select_topk_groups(T_np, wl.W, g, wl.k), several=B >= 12)
    gpr = wl.layout.groups_per_row
    assert np.array_equal(got.reshape(-1)[3 * gpr:4 * gpr], wl.codes.reshape(-1)[3 * gpr:4 * gpr])


@pytest.mark.parametrize("mode", [1, 0])
@pytest.mark.parametrize("g,B", [(8, 8), (8, 11), (16, 11), (8, 13), (16, 12)])      # as above
def test_reencode_m1_duplicate_codewords_tie_rule(mode, g, B):
    wl = workloads.make(16, 32 * g, g, 1, B, seed=9, sigma_g=2e-3, tau=1.0)
    half = 1 << (B - 1)
    wl.codebooks[0, half:] = wl.codebooks[0, :half]     # every codeword exists twice
    run, got, want, info = reencode_case(wl, mode)
    if mode == 0:
        check_route(run, wl.k, filtered=B >= 11)
    if B >= 11:
        T_np = oracle.encode_targets(wl.W, wl.G, wl.alpha)
        check_launches(run, T_np, oracle.select_topk_groups(T_np, wl.W, g, wl.k), several=B >= 12)
    assert np.array_equal(got, want)                     # exact ties resolve identically


@pytest.mark.parametrize("g,B", [(8, 10), (16, 9), (8, 11), (16, 11), (16, 13), (8, 13)])   # as above
@pytest.mark.parametrize("case", ["targets_on_codewords", "mixed_magnitudes", "tiny_values", "huge_values",
                                  "clustered_codebook", "one_dimension_dominates"])
def test_reencode_m1_inputs_that_stress_the_filter(g, B, case):
    """Inputs chosen against the fp16 filter and its bounds, in one launch (11 bits) and in several; the decision must stay the
    oracle's (and, below 2048 codewords, that of the one launch that takes so little work)."""
    wl = workloads.make(24, 64 * g, g, 1, B, seed=12, sigma_g=2e-3, tau=1.0)
    rng = np.random.default_rng(12)
    T_np = None
    if case == "targets_on_codewords":       # distance exactly zero for the right codeword
        pick = rng.integers(0, 1 << B, size=wl.layout.num_groups)
        T_np = (wl.codebooks[0, pick].reshape(24, 64, g) * wl.scales[:, None, None]).reshape(24, 64 * g)
        T_np = T_np.astype(np.float32)
    elif case == "mixed_magnitudes":         # half of the codewords a hundred times larger
        wl.codebooks[0, ::2] *= np.float32(100.0)
    elif case == "tiny_values":
        wl.codebooks *= np.float32(1e-20)
        wl.W *= np.float32(1e-20)
        wl.G *= np.float32(1e-20)
    elif case == "huge_values":
        wl.codebooks *= np.float32(1e15)
        wl.W *= np.float32(1e15)
        wl.G *= np.float32(1e15)
    elif case == "clustered_codebook":       # all codewords within a tiny ball: nothing can be excluded
        base = wl.codebooks[0, 0].copy()
        wl.codebooks[0] = base + (rng.standard_normal(wl.codebooks[0].shape) * 1e-7).astype(np.float32)
    elif case == "one_dimension_dominates":
        wl.codebooks[0, :, 0] *= np.float32(1000.0)
        wl.W[:, ::g] *= np.float32(1000.0)
    run, got, want, info = reencode_case(wl, 0, T_np=T_np)
    check_route(run, wl.k, filtered=B >= 11)
    if B >= 11:
        T_np = oracle.encode_targets(wl.W, wl.G, wl.alpha) if T_np is None else T_np
        check_launches(run, T_np, oracle.select_topk_groups(T_np, wl.W, g, wl.k), several=B >= 13)
    if case == "targets_on_codewords":
        assert (info["obj_new"] <= 1e-12).all()


@pytest.mark.parametrize("mode", [1, 0])
def test_reencode_fixed_point_when_update_is_zero(mode):
    wl = workloads.make(32, 512, 8, 1, 12, seed=10, tau=1.0)
    W = oracle.dequantize(wl.codes, wl.codebooks, wl.scales)
    wl.W[:] = W
    run = GpuRun(wl)
    run.ctx.pv_set_search_mode(mode)
    T = run.targets(0.0)
    got, nch = run.reencode(T, np.arange(wl.layout.num_groups, dtype=np.int32))
    assert nch == 0 and np.array_equal(got, wl.codes)


def test_reencode_empty_selection_and_errors():
    from paper_2405_14852_amd import PVError
    wl = workloads.make(8, 64, 8, 1, 4, seed=11)
    run = GpuRun(wl)
    T = run.targets()
    got, nch = run.reencode(T, np.zeros(0, np.int32))
    assert nch == 0 and np.array_equal(got, wl.codes)
    with pytest.raises(PVError):
        run.ctx.pv_reencode_groups(run.lay, T, run.cb, run.sc,
                                   torch.zeros(4, dtype=torch.int32, device=DEV),
                                   wl.layout.num_groups + 1, 1, run.codes)
    with pytest.raises(PVError):
        run.ctx.pv_reencode_groups(run.lay, T, run.cb, run.sc, None, 0, 0, run.codes)
    bad = type(run.lay)(8, 60, 8, 1, 4)
    with pytest.raises(PVError):
        run.ctx.pv_encode_targets(bad, run.W, run.G, 1.0, T)
    with pytest.raises(PVError):
        run.ctx.pv_select_topk_groups(run.lay, T, run.W, -1,
                                      torch.zeros(4, dtype=torch.int32, device=DEV))
    bad = type(run.lay)(8, 64, 8, 1, 17)
    with pytest.raises(PVError):
        run.ctx.pv_dequantize(bad, run.codes, run.cb, run.sc, T)


@pytest.mark.parametrize("mode", [1, 0])
@pytest.mark.parametrize("g,M,B,beam", [(8, 1, 10, 1), (16, 1, 9, 1), (8, 1, 11, 1), (16, 1, 11, 1), (8, 2, 8, 8), (8, 3, 4, 4),
                                        (4, 1, 3, 1)])
def test_reencode_reads_stored_codes_modulo_the_codebook_size(mode, g, M, B, beam):
    """Stray bits above B in the stored codes: the library reads the low B bits (the oracle
    refuses such input, so it is given the clean codes); a group that keeps its code keeps its
    stray bits, a group that changes is written clean, num_changed counts tuples modulo 2^B."""
    wl = workloads.make(16, 32 * g, g, M, B, seed=77, sigma_g=2e-3, tau=1.0, beam_width=beam)
    rng = np.random.default_rng(77)
    stray = (rng.integers(0, 1 << (16 - B), size=wl.codes.shape) << B).astype(np.uint16)
    stray[rng.random(wl.codes.shape) < 0.5] = 0
    dirty = wl.codes | stray
    T_np = oracle.encode_targets(wl.W, wl.G, wl.alpha)
    # half of the groups get their own reconstruction as target, so that they keep their code
    keep = rng.random(wl.layout.num_groups) < 0.5
    W_own = oracle.dequantize(wl.codes, wl.codebooks, wl.scales).reshape(-1, g)
    T_np = T_np.reshape(-1, g).copy()
    T_np[keep] = W_own[keep]
    T_np = T_np.reshape(wl.W.shape)
    idx = np.arange(wl.layout.num_groups, dtype=np.int32)
    run = GpuRun(wl)
    run.ctx.pv_set_search_mode(mode)
    got, nch = run.reencode(dev_f32(T_np), idx, codes=dev_u16(dirty))
    if mode == 0 and M == 1 and g >= 8:
        check_route(run, len(idx), filtered=B == 11)
    want, info = oracle.reencode_groups(T_np, wl.codebooks, wl.scales, idx, wl.codes, beam_width=beam)
    mask = np.uint16((1 << B) - 1)
    ndiff = check_codes_on(wl, T_np, idx, got & mask, want, info)
    assert abs(nch - info["num_changed"]) <= ndiff
    g2, w2, d2, c2 = got.reshape(-1, M), want.reshape(-1, M), dirty.reshape(-1, M), wl.codes.reshape(-1, M)
    same = (w2 == c2).all(1) & ((g2 & mask) == w2).all(1)
    assert same.sum() > 0 and (~same).sum() > 0
    assert np.array_equal(g2[same], d2[same])                    # kept groups: untouched, stray bits stay
    moved = (w2 != c2).any(1) & ((g2 & mask) == w2).all(1)
    assert np.array_equal(g2[moved], w2[moved])                  # changed groups: written clean


# ------------------------------------------------------- ceiling probes

def test_probe_kernels_copy_exactly_and_report_plausible_rates():
    from paper_2405_14852_amd import PVContext, PVError
    ctx = PVContext(0)
    src = torch.randn(1 << 20, dtype=torch.float32, device=DEV)
    dst = torch.zeros_like(src)
    ctx.pv_probe_copy(dst, src)
    torch.cuda.synchronize()
    assert torch.equal(dst, src)
    sink = torch.zeros(256 * 16 * 64, dtype=torch.float32, device=DEV)
    ctx.pv_probe_mfma_f16(1024, sink)          # the first launch loads the code
    ctx.pv_timing_enable(True)
    waves = ctx.pv_probe_mfma_f16(1024, sink)
    ms, n = ctx.pv_timing_read("probe_mfma")
    assert waves == 256 * 4 * 4 and n == 1
    rate = waves * 1024 * 2.0 * 32 * 32 * 16 / (ms * 1e-3) / 1e12
    assert 200.0 < rate < 2600.0           # TFLOP/s: below the published peak, far above vector rates
    assert torch.isfinite(sink).all() and float(sink.abs().max()) > 0
    with pytest.raises(PVError):
        ctx.pv_probe_mfma_f16(3, sink)
    with pytest.raises(PVError):
        ctx.pv_probe_copy(dst[1:], src[1:])     # 4-byte offset: not 16-byte aligned


# ------------------------------------------------------- re-encode, beam search

@pytest.mark.parametrize("M,B,g,beam,shape", [
    (2, 8, 8, 8, (64, 256)),     # the 2x8 configuration, beam 8
    (2, 8, 8, 1, (16, 256)),
    (2, 8, 8, 3, (16, 256)),
    (3, 4, 8, 8, (16, 128)),
    (2, 5, 16, 16, (8, 256)),
    (4, 3, 4, 4, (8, 64)),
    (2, 2, 2, 64, (4, 32)),
    (2, 8, 16, 8, (32, 512)),    # two 8-bit codebooks over groups of 16 (wave-per-group kernel)
    (8, 2, 8, 16, (8, 128)),     # the largest number of codebooks
    (2, 4, 64, 8, (8, 512)),     # the largest group size
    (2, 12, 8, 1, (8, 128)),     # the largest candidate pool (beam 1 x 4096 codewords)
])
def test_reencode_beam_matches_oracle(M, B, g, beam, shape):
    wl = workloads.make(shape[0], shape[1], g, M, B, seed=12, sigma_g=2e-3, tau=0.5,
                        beam_width=beam)
    reencode_case(wl, 0)


def test_reencode_beam_duplicate_codewords():
    wl = workloads.make(8, 256, 8, 2, 6, seed=13, sigma_g=2e-3, tau=1.0, beam_width=4)
    wl.codebooks[:, 32:] = wl.codebooks[:, :32]
    _, got, want, _ = reencode_case(wl, 0)
    assert np.array_equal(got, want)


# Two 8-bit codebooks (the additive configuration of App. K): mode 0 runs the matrix-core
# filter with its double-precision certificates and hands the undecided groups to the exact
# kernel, mode 1 runs the exact kernel alone.  Both must give the oracle's codes.

@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("g", [8, 16])
@pytest.mark.parametrize("beam", [1, 2, 5, 8])
def test_reencode_2x8_both_paths(mode, g, beam):
    wl = workloads.make(24, 40 * g, g, 2, 8, seed=21 + beam, sigma_g=2e-3, tau=0.47, beam_width=beam)
    run, got, want, info = reencode_case(wl, mode)
    st = run.ctx.pv_reencode_stats()
    if mode == 0:
        assert st["filtered"] + st["fallback"] == wl.k and st["exact"] == 0
        assert st["filtered"] > 0.9 * wl.k          # the filter decides nearly every group
    else:
        assert st["exact"] == wl.k and st["filtered"] == 0


@pytest.mark.parametrize("g", [8, 16])
@pytest.mark.parametrize("k", [1, 2, 3, 7])
def test_reencode_2x8_short_lists(g, k):
    """Fewer groups than one wave's pair, odd list lengths."""
    wl = workloads.make(4, 16 * g, g, 2, 8, seed=30 + k, sigma_g=2e-3, tau=1.0, beam_width=8)
    T_np = oracle.encode_targets(wl.W, wl.G, wl.alpha)
    idx = np.sort(np.random.default_rng(k).choice(wl.layout.num_groups, size=k, replace=False)).astype(np.int32)
    _, got, want, _ = reencode_case(wl, 0, idx=idx, T_np=T_np)
    assert np.array_equal(got, want)


@pytest.mark.parametrize("g", [8, 16])
@pytest.mark.parametrize("case", ["duplicates", "scales", "targets_on_sums", "integers", "tiny_values",
                                  "huge_values", "one_dimension_dominates", "identical_codebooks"])
def test_reencode_2x8_inputs_that_stress_the_filter(g, case):
    wl = workloads.make(16, 24 * g, g, 2, 8, seed=40, sigma_g=2e-3, tau=1.0, beam_width=8)
    rng = np.random.default_rng(41)
    exact = True          # exact ties must resolve as in the oracle (lexicographic order)
    if case == "duplicates":
        wl.codebooks[:, 128:] = wl.codebooks[:, :128]
    elif case == "scales":
        wl.scales[2] = 0.0
        wl.scales[3] = -0.8
        wl.scales[4] = 1e-6
        wl.scales[5] = 400.0
    elif case == "targets_on_sums":      # objective 0 for one pair: the expanded form may go negative
        c = rng.integers(0, 256, size=(wl.layout.num_groups, 2))
        rec = wl.codebooks[0][c[:, 0]] + wl.codebooks[1][c[:, 1]]
        rows = np.repeat(np.arange(16), wl.layout.groups_per_row)
        wl.W = (rec * wl.scales[rows, None]).reshape(wl.W.shape).astype(np.float32)
        wl.G[:] = 0
    elif case == "integers":             # many exact ties between different pairs
        wl.codebooks = rng.integers(-3, 4, size=wl.codebooks.shape).astype(np.float32)
        wl.W = rng.integers(-6, 7, size=wl.W.shape).astype(np.float32)
        wl.G[:] = 0
        wl.scales[:] = 1.0
    elif case == "tiny_values":
        wl.codebooks *= np.float32(1e-18)
        wl.W *= np.float32(1e-18)
        wl.G *= np.float32(1e-18)
    elif case == "huge_values":
        wl.codebooks *= np.float32(1e15)
        wl.W *= np.float32(1e15)
        wl.G *= np.float32(1e15)
    elif case == "one_dimension_dominates":
        wl.codebooks[:, :, 0] *= np.float32(1e4)
        wl.W[:, ::g] *= np.float32(1e4)
    elif case == "identical_codebooks":
        wl.codebooks[1] = wl.codebooks[0]
    run, got, want, info = reencode_case(wl, 0)
    if exact:
        assert np.array_equal(got, want)
    st = run.ctx.pv_reencode_stats()
    assert st["filtered"] + st["fallback"] == wl.k
    if case == "scales":
        gpr = wl.layout.groups_per_row
        assert np.array_equal(got.reshape(-1, 2)[2 * gpr:3 * gpr], wl.codes.reshape(-1, 2)[2 * gpr:3 * gpr])


@pytest.mark.parametrize("copies,step", [(10, 3e-6), (12, 3e-6), (40, 1e-5), (12, 1e-7), (256, 2e-7)])
def test_reencode_2x8_near_copies_around_the_beam_boundary(copies, step):
    """First codebook made of clusters of near-copies: the 8th and 9th best first codes differ
    by less than the filter's 24-bit keys resolve (or, for the smallest steps, not at all).
    The kernel then pulls in up to three more candidates and ranks them exactly, or leaves
    the group to the exact kernel.  The codes are the oracle's either way."""
    wl = workloads.make(16, 256, 8, 2, 8, seed=46, sigma_g=2e-3, tau=1.0, beam_width=8)
    base = wl.codebooks[0].copy()
    for c in range(256):
        wl.codebooks[0, c] = base[c // copies] * np.float32(1.0 + step * (c % copies))
    run, got, want, info = reencode_case(wl, 0)
    assert np.array_equal(got, want)
    st = run.ctx.pv_reencode_stats()
    assert st["filtered"] + st["fallback"] == wl.k


@pytest.mark.parametrize("M,B,g,beam", [(2, 8, 8, 8), (2, 8, 8, 2), (3, 4, 8, 4)])
def test_reencode_beam_repeated_sweeps(M, B, g, beam):
    """A second call on the same list is a second sweep over the codebooks, seeded with the
    first sweep's winner (App. D's local search repeated): same codes as the oracle applied
    twice, objective non-increasing, and a fixed point once nothing moves."""
    wl = workloads.make(16, 32 * g, g, M, B, seed=60, sigma_g=4e-3, tau=1.0, beam_width=beam)
    run = GpuRun(wl)
    T_np = oracle.encode_targets(wl.W, wl.G, wl.alpha)
    idx = np.arange(wl.layout.num_groups, dtype=np.int32)
    T = dev_f32(T_np)
    got = wl.codes
    want = wl.codes
    prev_obj = None
    for sweep in range(4):
        got, nch = run.reencode(T, idx, codes=dev_u16(got))
        want, info = oracle.reencode_groups(T_np, wl.codebooks, wl.scales, idx, want, beam_width=beam)
        ndiff = check_codes_on(wl, T_np, idx, got, want, info)
        # a group resolved differently on a near-tie may count as changed on one side only
        assert abs(nch - info["num_changed"]) <= ndiff
        got = want       # continue from the oracle's codes when a near-tie was resolved differently
        if prev_obj is not None:
            assert (info["obj_prev"] <= prev_obj * (1 + 1e-12)).all()
        prev_obj = info["obj_new"]
        if info["num_changed"] == 0:
            break
    assert sweep >= 1        # the second sweep still finds better tuples for some groups


@pytest.mark.parametrize("seed", range(8))
def test_reencode_2x8_filter_agrees_with_the_exact_kernel_on_large_lists(seed):
    """Tens of thousands of groups per case, varied gradient sizes, scale spreads, codebook
    spreads and beam widths: the filtered path (mode 0) and the exact kernel (mode 1) must
    write identical codes; a sample is checked against the oracle as well."""
    rng = np.random.default_rng(1000 + seed)
    g = 8 if seed % 2 == 0 else 16
    beam = int(rng.integers(1, 9))
    wl = workloads.make(512, 128 * g, g, 2, 8, seed=70 + seed, sigma_g=float(10.0 ** rng.uniform(-4, -2)),
                        sigma_c=float(10.0 ** rng.uniform(-2.5, -1.0)), tau=0.6, beam_width=beam)
    wl.scales *= np.float32(10.0 ** rng.uniform(-1, 1))
    if seed % 3 == 0:
        wl.scales[rng.integers(0, 512, size=40)] *= np.float32(-1.0)
    T_np = oracle.encode_targets(wl.W, wl.G, wl.alpha)
    idx = oracle.select_topk_groups(T_np, wl.W, g, wl.k)
    run = GpuRun(wl)
    T = dev_f32(T_np)
    run.ctx.pv_set_search_mode(1)
    exact, n_exact = run.reencode(T, idx)
    run.ctx.pv_set_search_mode(0)
    fast, n_fast = run.reencode(T, idx)
    st = run.ctx.pv_reencode_stats()
    assert np.array_equal(fast, exact) and n_fast == n_exact
    assert st["filtered"] + st["fallback"] == wl.k and st["filtered"] > 0.9 * wl.k
    sub = np.sort(rng.choice(idx, size=512, replace=False))
    want, info = oracle.reencode_groups(T_np, wl.codebooks, wl.scales, sub, wl.codes, beam_width=beam)
    check_codes_on(wl, T_np, sub, fast, want, info)


def test_reencode_2x8_non_finite_inputs_end_normally():
    wl = workloads.make(8, 128, 8, 2, 8, seed=44, sigma_g=2e-3, tau=1.0, beam_width=8)
    T_np = oracle.encode_targets(wl.W, wl.G, wl.alpha)
    T_np[1, :8] = np.nan
    T_np[2, 8:16] = np.inf
    wl.scales[5] = np.inf
    run = GpuRun(wl)
    idx = np.arange(wl.layout.num_groups, dtype=np.int32)
    got, _ = run.reencode(dev_f32(T_np), idx)
    assert got.max() < 256
    clean = np.ones(wl.layout.num_groups, bool)
    gpr = wl.layout.groups_per_row
    clean[gpr * 1] = clean[gpr * 2 + 1] = False
    clean[5 * gpr:6 * gpr] = False
    sub = idx[clean]
    want, info = oracle.reencode_groups(T_np, wl.codebooks, wl.scales, sub, wl.codes, beam_width=8)
    check_codes_on(wl, T_np, sub, got, want, info)


# ------------------------------------------------------------- whole path

@pytest.mark.parametrize("name,shape", [("c1_256x256_1x8", None),
                                        ("c2_4096x4096_1x16", (128, 1024)),
                                        ("c3_11008x4096_2x8", (96, 512)),
                                        ("c5a_14336x4096_1x16g16", (64, 2048))])
def test_whole_path_small(name, shape):
    kw = {} if shape is None else dict(out_features=shape[0], in_features=shape[1], tau=0.2)
    wl = workloads.make_config(name, seed=0, **kw)
    run = GpuRun(wl)
    g = wl.layout.group_size
    T = run.targets()
    T_ref = oracle.encode_targets(wl.W, wl.G, wl.alpha)
    assert np.array_equal(T.cpu().numpy(), T_ref)
    idx = run.select(T, wl.k)
    idx_ref = oracle.select_topk_groups(T_ref, wl.W, g, wl.k)
    assert np.array_equal(idx, idx_ref)
    got, _ = run.reencode(T, idx)
    want, info = oracle.reencode_groups(T_ref, wl.codebooks, wl.scales, idx_ref, wl.codes,
                                        beam_width=wl.beam_width)
    check_codes(wl, T_ref, idx_ref, got, want, info)
    assert (info["obj_new"] <= info["obj_prev"]).all()
    W2 = run.dequantize(want)
    W2_ref = oracle.dequantize(want, wl.codebooks, wl.scales)
    rel = np.linalg.norm((W2 - W2_ref).astype(np.float64)) / np.linalg.norm(W2_ref.astype(np.float64))
    assert rel <= RECON_REL and np.array_equal(W2, W2_ref)
