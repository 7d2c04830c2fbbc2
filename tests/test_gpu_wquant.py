"""GPU parity of the offline weight quantiser (fq_cas_scales, fq_pts_exponent, fq_quantize_weights)
against the CPU oracle: channel scales to the last FP32 bit, the per-tensor exponent exactly, INT4 codes
and FP8 group scales bit for bit."""
import numpy as np
import pytest

import oracle
from paper_2505_20839_amd import workloads
from parity_util import bf16_bits_from_gpu, check_gemm, to_gpu_bf16

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

T = 7 * 2.0 ** -9


@pytest.fixture(scope="module")
def fq():
    from paper_2505_20839_amd import binding
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    binding.lib()
    return binding


def _bits(x):
    return workloads.f32_to_bf16_bits(np.asarray(x, np.float32))


# (K >= 8192 with whole 16-byte steps: the kernel of 64-channel blocks; 8200 leaves its last block 8 channels)
@pytest.mark.parametrize("N,K,seed", [(40, 128, 0), (300, 1000, 1), (7, 64, 2), (1024, 512, 3), (70, 8192, 4), (300, 8200, 5)])
def test_cas_scales_match_oracle(fq, N, K, seed):
    Wb = workloads.draw_weights(N, K, seed=seed, channel_spread=1.0)
    Wb[:, K // 3] = 0                                          # an all-zero channel keeps lambda = 1
    target = float(np.float32(0.03))                            # the entry point takes the target as FP32
    lam = fq.fq_cas_scales(to_gpu_bf16(Wb), target).cpu().numpy()
    want = oracle.cas_scales(Wb, target)
    assert lam.dtype == np.float32 and lam[K // 3] == 1.0
    w32 = want.astype(np.float32)
    ulp = np.abs(np.nextafter(w32, np.float32(np.inf)) - w32)
    assert np.all(np.abs(lam.astype(np.float64) - want) <= ulp), "more than one FP32 ulp from the FP64 value"
    assert np.mean(lam == w32) > 0.999


PTS_CASES = {
    "typical": dict(std=0.02, zero_frac=0.0),                  # the overflow band stops the search
    "tiny": dict(std=2e-5, zero_frac=0.0),
    "with_zeros": dict(std=0.02, zero_frac=0.3),
    "wide": dict(std=0.5, channel_spread=2.0),
}


@pytest.mark.parametrize("case", sorted(PTS_CASES))
@pytest.mark.parametrize("with_lambda", [False, True])
def test_pts_exponent_matches_oracle(fq, case, with_lambda):
    Wb = workloads.draw_weights(48, 512, seed=len(case), **PTS_CASES[case])
    W = to_gpu_bf16(Wb)
    lam = fq.fq_cas_scales(W, 0.05) if with_lambda else None
    n = int(fq.fq_pts_exponent(W, lam)[0])
    assert n == oracle.pts_exponent(Wb, None if lam is None else lam.cpu().numpy())


def test_pts_exponent_hand_matrices(fq):
    """The cases that pin the two conditions of the definition and their edges, through the GPU."""
    def n_of(values):
        v = np.zeros((1, 128), np.float32)
        v[0, :len(values)] = values
        n = int(fq.fq_pts_exponent(to_gpu_bf16(_bits(v)))[0])
        assert n == oracle.pts_exponent(_bits(v))
        return n
    assert n_of([1.0, -0.5, T]) == 0                           # zeros of the padding never matter
    assert n_of([]) == 0
    assert n_of([1.0, T / 8]) == 3
    assert n_of([0.5, 2.0 ** -40]) == 9
    assert n_of([224.0, 2.0 ** -40]) == 0
    assert n_of([223.0, 2.0 ** -40]) == 1
    assert n_of([448.0, T / 4]) == 2
    assert n_of([2.0 ** -100]) == 94
    assert n_of([2.0 ** -130]) == 124


@pytest.mark.parametrize("N,K,n_pts,with_lambda,rne", [(33, 256, 0, False, False), (64, 512, 9, True, False),
                                                       (64, 512, 9, True, True), (5, 128, 3, False, True),
                                                       (257, 1408, 11, True, False)])
def test_quantize_weights_matches_oracle_bit_for_bit(fq, N, K, n_pts, with_lambda, rne):
    Wb = workloads.draw_weights(N, K, seed=N + K, std=0.02 * 2.0 ** (9 - n_pts), zero_frac=0.05)
    Wb[0, :128] = 0                                            # an all-zero group
    Wb[N - 1, K - 128:] = _bits(np.full(128, T / 2 ** n_pts * 0.9))   # a group under Lemma B.1's threshold
    W = to_gpu_bf16(Wb)
    lam = fq.fq_cas_scales(W, 0.02 * 2.0 ** (9 - n_pts)) if with_lambda else None
    lam_np = None if lam is None else lam.cpu().numpy()
    q, gs = fq.fq_quantize_weights(W, lam, n_pts, sigma_nearest=rne)
    torch.cuda.synchronize()
    q_ref, gs_ref = oracle.quantize_weights(Wb, lam_np, n_pts, sigma_rne=rne)
    assert np.array_equal(gs.cpu().numpy(), gs_ref)
    assert np.array_equal(q.cpu().numpy(), q_ref)
    assert gs_ref[0, 0] == 0 and (with_lambda or rne or gs_ref[N - 1, -1] == 0)
    assert q_ref.min() == -8 or q_ref.max() == 7               # the range is used


def test_chain_from_bf16_weights_to_the_gemm(fq):
    """Channel scales, per-tensor exponent, quantiser, packing and the GEMM with w_tscale = 2^-n: the
    result equals the oracle's GEMM on the oracle's own codes, and stays close to X W^T in FP64."""
    M, N, K = 96, 160, 1024
    Wb = workloads.draw_weights(N, K, seed=77)
    W = to_gpu_bf16(Wb)
    n = int(fq.fq_pts_exponent(W)[0])
    q, gs = fq.fq_quantize_weights(W, None, n)
    d = workloads.draw(M, N, K, seed=78)
    A, s = fq.fq_quantize_act(to_gpu_bf16(d["X_bf16"]))
    Y = fq.fq_w4a8_gemm(A, s, fq.fq_pack_weights(q), gs, 2.0 ** -n, N)
    torch.cuda.synchronize()
    assert n == oracle.pts_exponent(Wb)
    q_ref, gs_ref = oracle.quantize_weights(Wb, None, n)
    Yr, B = oracle.w4a8_gemm(A.cpu().numpy(), s.cpu().numpy(), q_ref, gs_ref, 2.0 ** -n, want_bound=True)
    check_gemm(bf16_bits_from_gpu(Y), Yr, B, "chain")
    exact = oracle.bf16_bits_to_f64(d["X_bf16"]) @ oracle.bf16_bits_to_f64(Wb).T
    rel = np.linalg.norm(oracle.bf16_bits_to_f64(bf16_bits_from_gpu(Y)) - exact) / np.linalg.norm(exact)
    assert rel < 0.25, rel              # INT4 steps of max/7 on uneven channels: 10-20 % is the format's own error


def test_full_size_gate_up_matrix(fq):
    """Llama2-7B gate/up shape (11008 x 4096): sampled channels against the oracle; the exponent against the
    two conditions of the definition evaluated with numpy on the whole matrix."""
    N, K = 11008, 4096
    Wb = workloads.draw_weights(N, K, seed=5)
    W = to_gpu_bf16(Wb)
    lam = fq.fq_cas_scales(W, 0.02)
    n = int(fq.fq_pts_exponent(W, lam)[0])
    q, gs = fq.fq_quantize_weights(W, lam, n)
    torch.cuda.synchronize()
    lam_np = lam.cpu().numpy()
    rows = [0, 1, 31, 32, 5000, 11007]
    q_ref, gs_ref = oracle.quantize_weights(Wb[rows], lam_np, n)
    assert np.array_equal(q.cpu().numpy()[rows], q_ref) and np.array_equal(gs.cpu().numpy()[rows], gs_ref)
    cols = [0, 1, 63, 64, 2047, 4095]
    want = oracle.cas_scales(Wb, float(np.float32(0.02)))[cols].astype(np.float32)
    assert np.allclose(lam_np[cols], want, rtol=2e-7, atol=0)
    v = np.abs(oracle.scaled_weights(Wb, lam_np).astype(np.float64))

    def stops(m):                                              # does the search stop at m?
        nz = v[v > 0]
        return bool(np.all(nz * 2.0 ** m >= T)) or bool(np.any((v * 2.0 ** m >= 224) & (v * 2.0 ** m < 448)))
    assert stops(n) and not any(stops(m) for m in range(n))

# (channels per workgroup: 64 from K = 16384 on, 32 from 8192, else 16, on a 256-unit device; a last line of 8 channels)
@pytest.mark.parametrize("N,K", [(1, 8), (513, 72), (1025, 4104), (130, 8200), (40, 16392), (2048, 72), (2049, 72), (6100, 136), (1100, 8200)])
def test_cas_scales_of_whole_lines_and_remainders(fq, N, K):
    """Row counts around a pass of the workgroup and channel counts around a 128-byte line, with subnormal, huge and zero
    weights: the FP64 mean of every channel."""
    Wb = workloads.draw_weights(N, K, seed=N + K, channel_spread=2.0)
    Wb[:, 0] = 1                                               # the smallest bf16 subnormal throughout
    Wb[:, 1] = 0x7F7F                                          # the largest bf16
    Wb[:, 2] = 0x8000                                          # -0
    Wb[0, 3::5] |= 0x8000
    lam = fq.fq_cas_scales(to_gpu_bf16(Wb), 0.02).cpu().numpy()
    mean = np.abs(oracle.bf16_bits_to_f64(Wb)).mean(axis=0)
    with np.errstate(divide="ignore", over="ignore"):
        want = np.where(mean == 0, 1.0, 0.02 / mean).astype(np.float32)
    assert np.array_equal(lam, want) or np.max(np.abs(lam.view(np.int32).astype(np.int64) - want.view(np.int32))) <= 1


# (workgroups of 256 threads up to 32768 threads, of 1024 beyond; one pass over the rows and several, a last one that is shorter)
@pytest.mark.parametrize("N,K", [(1, 128), (63, 128), (65, 384), (4097, 128), (2060, 4096), (64, 4096), (65, 4096), (191, 11008), (400, 11008)])
def test_pts_exponent_counts_every_workgroup(fq, N, K):
    """Every workgroup's rows count: the smallest non-zero and the largest element placed in every corner, twice in a row into
    fresh scratch (whatever the memory held before)."""
    Wb = np.full((N, K), 0x3F80, np.uint16)                    # 1.0 throughout
    base = int(fq.fq_pts_exponent(to_gpu_bf16(Wb))[0])
    assert base == oracle.pts_exponent(Wb)
    for pos in [(0, 0), (0, K - 1), (N - 1, 0), (N - 1, K - 1), (N // 2, K // 2)]:
        Wc = Wb.copy(); Wc[pos] = 0x43DF                       # 446: the largest bf16 below 7 * 2^6
        for _ in range(2):
            assert int(fq.fq_pts_exponent(to_gpu_bf16(Wc))[0]) == oracle.pts_exponent(Wc)
        # where that one element decides: 2^-12 among ones (condition 1: n = 6), 446 among 2^-20 (condition 2: n = 0, not 14)
        for rest, one, n in ((0x3F80, 0x3980, 6), (0x3580, 0x43DF, 0)):
            Wc = np.full((N, K), rest, np.uint16); Wc[pos] = one
            assert int(fq.fq_pts_exponent(to_gpu_bf16(Wc))[0]) == n and (N * K > 1 << 15 or oracle.pts_exponent(Wc) == n)


@pytest.mark.parametrize("N,K,n_pts", [(1, 128, 0), (15, 128, 1), (16, 128, 2), (17, 128, 0), (15, 640, 3), (67, 128, 126), (129, 384, 7),
                                       (128, 16384, 5), (1489, 1408, 4), (512, 4224, 0), (16417, 128, 2)])
def test_quantize_weights_at_the_edges_of_a_workgroup(fq, N, K, n_pts):
    """Group counts around the 16 a workgroup takes of a small matrix (up to 16384 groups) and the 32 of a larger one, quotients on
    and beside the rounding boundaries, huge v * 2^n, zero
    groups and groups whose scale casts to zero: codes and scales bit for bit."""
    rng = np.random.default_rng(N * K)
    Wb = workloads.draw_weights(N, K, seed=N, channel_spread=1.0)
    g = Wb.reshape(-1, 128)
    g[0] = 0
    for i in range(g.shape[0]):
        if i % 3 == 1:                                         # half-integer multiples of an E4M3 scale, one bf16 step around
            step = np.float32(2.0) ** int(rng.integers(-6, 3)) * np.float32(rng.integers(8, 16)) / 8
            x = workloads.f32_to_bf16_bits((rng.integers(-14, 15, 128) * step / 2).astype(np.float32))
            x[0] = workloads.f32_to_bf16_bits(np.array([7 * step], np.float32))[0]
            g[i] = np.where((x & 0x7FFF) > 0, x + rng.integers(-1, 2, 128).astype(np.uint16), x)
        elif i % 7 == 2:
            g[i] = 1                                           # scale casts to zero
    for rne in (False, True):
        q, gs = fq.fq_quantize_weights(to_gpu_bf16(Wb), None, n_pts, rne)
        qr, gr = oracle.quantize_weights(Wb, None, n_pts, sigma_rne=rne)
        assert np.array_equal(gs.cpu().numpy(), gr) and np.array_equal(q.cpu().numpy(), qr)


@pytest.mark.parametrize("n_pts", [0, 63, 64, 65, 100, 126])
@pytest.mark.parametrize("N,K", [(3, 128), (257, 8320)])
def test_quantize_weights_from_the_smallest_to_the_largest_weights(fq, N, K, n_pts):
    """Magnitudes from bf16's smallest to its largest, so that v * 2^n lies below, in and above the scale's range on both sides of
    the exponent from which 2^n multiplies the weights instead of the scale; an odd number of rows, so that the last pair is half a
    pair: codes and scales bit for bit."""
    rng = np.random.default_rng(N + n_pts)
    e = np.repeat(rng.integers(0, 255, (N, K // 128)), 128, axis=1)        # one exponent per group, three binades wide
    e = np.clip(e - rng.integers(0, 3, (N, K)), 0, 254)
    e[0, :128] = 135 - n_pts                                               # a group in the middle of the scale's range
    Wb = ((rng.integers(0, 2, (N, K)) << 15) | (e << 7) | rng.integers(0, 128, (N, K))).astype(np.uint16)
    for rne in (False, True):
        q, gs = fq.fq_quantize_weights(to_gpu_bf16(Wb), None, n_pts, rne)
        qr, gr = oracle.quantize_weights(Wb, None, n_pts, sigma_rne=rne)
        assert np.array_equal(gs.cpu().numpy(), gr) and np.array_equal(q.cpu().numpy(), qr)


@pytest.mark.parametrize("N,K", [(5, 72), (700, 72), (129, 8208), (70, 16392), (3, 75)])
def test_cas_scales_of_channels_that_are_not_finite(fq, N, K):
    """A NaN anywhere in a channel gives a NaN scale, an infinity a scale of 0, in every form of the kernel (K odd: the one
    without whole 16-byte steps); the other channels, sums beyond 2^128 of finite weights among them, keep their means."""
    Wb = workloads.draw_weights(N, K, seed=N + K)
    nan, inf = [0, 9, K - 1], [1, 17, K - 3]
    Wb[N - 1, nan] = [0x7F81, 0xFFC0, 0x7FFF]
    Wb[N // 2, inf] = [0x7F80, 0xFF80, 0x7F80]
    Wb[0, 9] = 0x7F80                                          # NaN and infinity in one channel
    Wb[:, 5] = 0x7F7F
    lam = fq.fq_cas_scales(to_gpu_bf16(Wb), 0.02).cpu().numpy()
    assert np.isnan(lam[nan]).all() and (lam[inf] == 0).all()
    rest = np.setdiff1d(np.arange(K), nan + inf)
    mean = np.abs(oracle.bf16_bits_to_f64(Wb[:, rest])).mean(axis=0)
    want = (0.02 / mean).astype(np.float32)
    assert np.max(np.abs(lam[rest].view(np.int32).astype(np.int64) - want.view(np.int32))) <= 1


@pytest.mark.parametrize("N,K", [(1, 1 << 25), (2, (17 << 20) + 8)])
def test_cas_scales_of_rows_beyond_32_bit_band_offsets(fq, N, K):
    """Rows so long that the 128 rows a workgroup reads side by side span 4 GiB and more: every row counts once (K past 2^24: offsets
    that wrapped would read the first rows again in the place of rows past N)."""
    W = torch.full((N, K), 0.5, dtype=torch.bfloat16, device="cuda")
    W[:, -1] = 2.0
    lam = fq.fq_cas_scales(W, 0.25)
    torch.cuda.synchronize()
    assert bool((lam[:-1] == 0.5).all()) and float(lam[-1]) == 0.125


# (rows shared out over the chip: an even slab of channels, uneven ones, a last share with fewer rows, more rows than one share's
# ring of bands; K = 1640: 205 columns in slabs of 52)
@pytest.mark.parametrize("N,K", [(5120, 1640), (5121, 4096), (9001, 1032), (16400, 512), (5200, 8192), (40000, 216)])
def test_cas_scales_with_scratch(fq, N, K):
    """The means of every channel, non-finite channels among them, against FP64 and against the call without scratch, which sums
    the same FP64 values in another order: one FP32 step apart at most."""
    assert fq.lib().fq_cas_scales_workspace_bytes(N, K) > 0
    g = torch.Generator(device="cuda").manual_seed(N + K)
    W = (torch.randn((N, K), generator=g, device="cuda") * 0.02).to(torch.bfloat16)
    W[:, 2] = 0
    W[:, 3] = 3.3895313892515355e38                            # the largest bf16: sums beyond 2^128
    W[N - 1, K - 1] = float("nan")
    W[0, 8] = float("inf")
    lam = fq.fq_cas_scales(W, 0.02)
    plain = torch.empty_like(lam)
    assert fq.lib().fq_cas_scales(W.data_ptr(), 0.02, plain.data_ptr(), N, K, torch.cuda.current_stream().cuda_stream) == 0
    assert bool(torch.isnan(lam[K - 1])) and float(lam[8]) == 0.0 and float(lam[2]) == 1.0
    mean = W.double().abs().mean(dim=0)
    want = torch.where(mean == 0, torch.ones_like(mean), 0.02 / mean).float()
    ok = torch.ones(K, dtype=torch.bool, device="cuda")
    ok[[8, K - 1]] = False
    for got in (plain, want):
        assert int((lam.view(torch.int32) - got.view(torch.int32))[ok].abs().max()) <= 1


@pytest.mark.parametrize("N,K", [(5120, 1640), (9001, 1032), (40000, 216)])
def test_cas_scales_same_bits_where_the_sums_are_exact(fq, N, K):
    """Magnitudes 2^-31 .. 1 in steps of 2^-38 and more, sums below 2^15: FP64 holds every partial sum, so that the calls with and
    without scratch and the one on a misaligned W agree in every bit, and with the FP64 mean."""
    g = torch.Generator(device="cuda").manual_seed(N)
    e = torch.randint(-30, 1, (N, K), generator=g, device="cuda", dtype=torch.int32)
    store = torch.empty((N * K + 1,), dtype=torch.bfloat16, device="cuda")
    W, off = torch.ldexp(torch.rand((N, K), generator=g, device="cuda") * 0.5 + 0.5, e).to(torch.bfloat16), store[1:].view(N, K)
    off.copy_(W)
    lam = fq.fq_cas_scales(W, 0.02)
    others = [torch.empty_like(lam) for _ in range(2)]
    for M, out in zip((W, off), others):
        assert fq.lib().fq_cas_scales(M.data_ptr(), 0.02, out.data_ptr(), N, K, torch.cuda.current_stream().cuda_stream) == 0
    assert all(torch.equal(lam, out) for out in others + [fq.fq_cas_scales(off, 0.02)])
    assert torch.equal(lam, (float(np.float32(0.02)) / (W.double().abs().sum(dim=0) / N)).float())


@pytest.mark.parametrize("N,K", [(3, 128), (64, 4096), (65, 4096), (2060, 4096), (400, 11008)])
def test_pts_exponent_without_scratch(fq, N, K):
    """The statistics met in the caller's 64 bytes: the same exponent, wherever the element that decides is."""
    for pos in [(0, 0), (N - 1, K - 1), (N // 2, K // 2)]:
        for rest, one, n in ((0x3F80, 0x3980, 6), (0x3580, 0x43DF, 0)):
            Wb = np.full((N, K), rest, np.uint16); Wb[pos] = one
            W, out = to_gpu_bf16(Wb), torch.empty((16,), dtype=torch.int32, device="cuda")
            assert fq.lib().fq_pts_exponent(W.data_ptr(), 0, out.data_ptr(), N, K, torch.cuda.current_stream().cuda_stream) == 0
            assert int(out[0]) == n == int(fq.fq_pts_exponent(W)[0])
