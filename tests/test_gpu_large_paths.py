"""GPU parity of every path of the large-M kernel: whole tiles (256 rows x 128 channels) and half tiles,
with whole-row stores and with element-wise stores at ragged edges, each as the plain GEMM, with the
residual added (out of place and in place) and with the fused gate/up epilogue -- every output element
against the CPU oracle.  Which path a shape takes depends on the device's compute-unit count, so each
test first asks the library (fq_w4a8_gemm_plan) and asserts that the shape reaches the path it is meant for."""
import numpy as np
import pytest

import oracle
from paper_2505_20839_amd import workloads
from parity_util import bf16_bits_from_gpu, check_gemm, to_gpu_bf16

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def fq():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU: torch.cuda.is_available() is False")
    from paper_2505_20839_amd import binding
    binding.lib()
    binding.fq_test_force_kernel(None)
    return binding


def _gpu(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


# shape -> the kinds of work item it must contain on this device
WHOLE_EVEN = (2048, 8192, 256)       # 512 whole tiles, nothing ragged
WHOLE_RAGGED = (2100, 4112, 384)     # whole tiles; last row tile has 52 rows, last channel tile 16 channels
MIXED = (2048, 8200, 256)            # whole tiles, half tiles, and a ragged last channel tile of 8 channels


def _plan(fq, shape):
    return fq.fq_w4a8_gemm_plan(*shape)


def test_shapes_reach_the_paths_they_are_meant_for(fq):
    p = _plan(fq, WHOLE_EVEN)
    assert p["kernel"] == "large" and p["whole"] > 0 and p["whole_ragged"] == p["half"] == p["half_ragged"] == 0
    p = _plan(fq, WHOLE_RAGGED)
    assert p["whole"] > 0 and p["whole_ragged"] > 0
    p = _plan(fq, MIXED)
    assert p["whole"] > 0 and p["half"] > 0 and p["whole_ragged"] + p["half_ragged"] > 0
    # the benchmark workloads: c2 mixes whole and half tiles, c4a / c4b are whole tiles throughout
    assert _plan(fq, (2048, 11008, 4096))["whole"] > 0
    assert _plan(fq, (8192, 14336, 4096))["whole"] == 32 * 112
    assert _plan(fq, (8192, 4096, 4096))["whole"] > 0          # attention output projection at prefill, with residual


def _problem(shape, seed, **kw):
    M, N, K = shape
    return workloads.draw(M, N, K, seed=seed, outlier_frac=0.01, **kw)


@pytest.mark.parametrize("shape", [WHOLE_EVEN, WHOLE_RAGGED, MIXED])
def test_plain_gemm_every_element(fq, shape):
    M, N, K = shape
    d = _problem(shape, seed=M + N)
    A, s = fq.fq_quantize_act(to_gpu_bf16(d["X_bf16"]))
    Yg = fq.fq_w4a8_gemm(A, s, fq.fq_pack_weights(_gpu(d["q"])), _gpu(d["gscale"]), d["w_tscale"], N)
    torch.cuda.synchronize()
    Y, B = oracle.w4a8_gemm(A.cpu().numpy(), s.cpu().numpy(), d["q"], d["gscale"], d["w_tscale"], want_bound=True)
    check_gemm(bf16_bits_from_gpu(Yg), Y, B, "plain %s" % (shape,))


@pytest.mark.parametrize("shape", [WHOLE_EVEN, WHOLE_RAGGED, MIXED])
def test_residual_every_element_and_in_place(fq, shape):
    M, N, K = shape
    d = _problem(shape, seed=2 * M + N)
    A, s = fq.fq_quantize_act(to_gpu_bf16(d["X_bf16"]))
    packed, gs = fq.fq_pack_weights(_gpu(d["q"])), _gpu(d["gscale"])
    An, sn = A.cpu().numpy(), s.cpu().numpy()
    Rb = workloads.draw_residual(M, N, scale=4.0, seed=M + N)
    R = to_gpu_bf16(Rb)
    Yg = fq.fq_w4a8_gemm_add(A, s, packed, gs, d["w_tscale"], N, R)
    torch.cuda.synchronize()
    assert np.array_equal(bf16_bits_from_gpu(R), Rb)           # the residual itself is not written
    Y, B = oracle.w4a8_gemm_add(An, sn, d["q"], d["gscale"], d["w_tscale"], Rb, want_bound=True)
    check_gemm(bf16_bits_from_gpu(Yg), Y, B, "add %s" % (shape,))
    Yi = fq.fq_w4a8_gemm_add(A, s, packed, gs, d["w_tscale"], N, R, out=R)
    torch.cuda.synchronize()
    assert np.array_equal(bf16_bits_from_gpu(Yi), bf16_bits_from_gpu(Yg)), "in place differs"


@pytest.mark.parametrize("shape", [WHOLE_EVEN, WHOLE_RAGGED, MIXED])
def test_swiglu_every_element(fq, shape):
    M, N, K = shape
    d = _problem(shape, seed=3 * M + N, gs_lo=0.01, gs_hi=0.1, w_tscale=0.25)
    A, s = fq.fq_quantize_act(to_gpu_bf16(d["X_bf16"]))
    Hg = fq.fq_w4a8_gemm_swiglu(A, s, fq.fq_pack_weights(_gpu(d["q"])), _gpu(d["gscale"]), d["w_tscale"], N)
    torch.cuda.synchronize()
    H, B = oracle.w4a8_gemm_swiglu(A.cpu().numpy(), s.cpu().numpy(), d["q"], d["gscale"], d["w_tscale"], want_bound=True)
    check_gemm(bf16_bits_from_gpu(Hg), H, B, "swiglu %s" % (shape,))


@pytest.mark.parametrize("shape", [WHOLE_EVEN, WHOLE_RAGGED, MIXED])
def test_zero_activations_return_the_residual_bit_for_bit(fq, shape):
    """All-zero activations: every output is bf16(0 + R[m,n]) = R[m,n], so each element of the residual has to
    arrive at its own place in every kind of tile."""
    M, N, K = shape
    q = np.random.default_rng(M).integers(-8, 8, (N, K), dtype=np.int8)
    gs = np.full((N, K // 128), 0x38, np.uint8)
    Rb = np.random.default_rng(N).integers(0, 0x7F80, (M, N)).astype(np.uint16)
    Rb |= np.random.default_rng(N + 1).integers(0, 2, (M, N)).astype(np.uint16) << 15
    Rb[Rb == 0x8000] = 0                                       # 0 + (-0) is +0
    Yg = fq.fq_w4a8_gemm_add(_gpu(np.zeros((M, K), np.uint8)), _gpu(np.ones(M, np.float32)),
                             fq.fq_pack_weights(_gpu(q)), _gpu(gs), 1.0, N, to_gpu_bf16(Rb))
    torch.cuda.synchronize()
    bad = np.argwhere(bf16_bits_from_gpu(Yg) != Rb)
    assert bad.size == 0, "%s: first wrong element %s" % (shape, bad[:1])


def test_exactly_sized_workspace_with_ragged_rows(fq):
    """A workspace of exactly fq_w4a8_gemm_workspace_bytes, placed at the very end of an allocation whose next
    bytes hold a pattern: the result is the oracle's, and the bytes behind the workspace are never written."""
    M, N, K = 300, 256, 1024
    d = workloads.draw(M, N, K, seed=17, outlier_frac=0.01)
    need = fq.fq_w4a8_gemm_workspace_bytes(M, N, K)
    arena = torch.full((need + 4096,), 0xA5, dtype=torch.uint8, device="cuda")
    ws = arena[:need]
    A, s = fq.fq_quantize_act(to_gpu_bf16(d["X_bf16"]), workspace=ws)
    Yg = fq.fq_w4a8_gemm(A, s, fq.fq_pack_weights(_gpu(d["q"])), _gpu(d["gscale"]), d["w_tscale"], N, workspace=ws,
                         workspace_prepared=True)
    torch.cuda.synchronize()
    assert bool((arena[need:] == 0xA5).all())
    Y, B = oracle.w4a8_gemm(A.cpu().numpy(), s.cpu().numpy(), d["q"], d["gscale"], d["w_tscale"], want_bound=True)
    check_gemm(bf16_bits_from_gpu(Yg), Y, B, "exact workspace")


def test_attention_output_projection_with_residual_at_prefill_size(fq):
    """M = 8192, N = K = 4096 (Llama3-8B attention output projection at prefill) with the residual stream updated
    in place: whole tiles + residual at a real size, one row of every eight against the oracle."""
    M, N, K = 8192, 4096, 4096
    d = workloads.draw(M, N, K, seed=41, act="laplace", outlier_frac=0.01)
    need = fq.fq_w4a8_gemm_workspace_bytes(M, N, K)
    ws = torch.empty((need,), dtype=torch.uint8, device="cuda")
    A, s = fq.fq_quantize_act(to_gpu_bf16(d["X_bf16"]), workspace=ws)
    rows = np.array([8 * i + (5 * i) % 8 for i in range(M // 8)])
    Rb = workloads.draw_residual(M, N, scale=workloads.RESIDUAL_SCALE, seed=42)
    R = to_gpu_bf16(Rb)
    fq.fq_w4a8_gemm_add(A, s, fq.fq_pack_weights(_gpu(d["q"])), _gpu(d["gscale"]), d["w_tscale"], N, R, out=R,
                        workspace=ws, workspace_prepared=True)
    torch.cuda.synchronize()
    Y, B = oracle.w4a8_gemm_add(A.cpu().numpy()[rows], s.cpu().numpy()[rows], d["q"], d["gscale"], d["w_tscale"],
                                Rb[rows], want_bound=True)
    check_gemm(bf16_bits_from_gpu(R)[rows], Y, B, "o_proj + residual")


@pytest.mark.parametrize("shape", [(300, 200, 1024), (129, 72, 1024), (1000, 1160, 256), (257, 136, 128), (513, 4104, 256)])
def test_masked_stores_at_ragged_edges(fq, shape):
    """Rows past M and channels past N inside an edge tile (N a multiple of 8: whole-row stores with a mask): every element
    against the oracle, plain and with the residual read from an array that ends where the output ends, and no byte
    behind the output written (a store that ignored the mask would land in the next row or behind the array)."""
    M, N, K = shape
    d = _problem(shape, seed=M + N)
    A, s = fq.fq_quantize_act(to_gpu_bf16(d["X_bf16"]))
    packed, gs = fq.fq_pack_weights(_gpu(d["q"])), _gpu(d["gscale"])
    Rb = workloads.draw_residual(M, N, scale=workloads.RESIDUAL_SCALE, seed=M)
    arena = torch.full((M * N + 4096,), -1, dtype=torch.int16, device="cuda")
    out = arena[:M * N].view(torch.bfloat16).view(M, N)
    A_ref, s_ref = A.cpu().numpy(), s.cpu().numpy()
    fq.fq_w4a8_gemm(A, s, packed, gs, d["w_tscale"], N, out=out)
    torch.cuda.synchronize()
    assert bool((arena[M * N:] == -1).all())
    Y, B = oracle.w4a8_gemm(A_ref, s_ref, d["q"], d["gscale"], d["w_tscale"], want_bound=True)
    check_gemm(bf16_bits_from_gpu(out), Y, B, "masked %s" % (shape,))
    out.copy_(to_gpu_bf16(Rb))
    fq.fq_w4a8_gemm_add(A, s, packed, gs, d["w_tscale"], N, out, out=out)
    torch.cuda.synchronize()
    assert bool((arena[M * N:] == -1).all())
    Y, B = oracle.w4a8_gemm_add(A_ref, s_ref, d["q"], d["gscale"], d["w_tscale"], Rb, want_bound=True)
    check_gemm(bf16_bits_from_gpu(out), Y, B, "masked residual %s" % (shape,))


@pytest.mark.parametrize("M,N", [(1000, 1296), (300, 528), (129, 2064)])
def test_masked_gate_up_tiles(fq, M, N):
    """The fused gate/up layer with quantised output at ragged edges: the masked rows and channels of an edge tile
    reach neither the output nor its scales and codes (the oracle's on the GPU's H)."""
    K = 512
    d = _problem((M, N, K), seed=M + N)
    A, s = fq.fq_quantize_act(to_gpu_bf16(d["X_bf16"]))
    packed, gs = fq.fq_pack_weights(_gpu(d["q"])), _gpu(d["gscale"])
    H, codes, scales = fq.fq_w4a8_gemm_swiglu_quant(A, s, packed, gs, d["w_tscale"], N)
    torch.cuda.synchronize()
    C_or, s_or = oracle.quantize_act(bf16_bits_from_gpu(H))
    codes = codes.cpu().numpy()
    assert np.array_equal(scales.cpu().numpy(), s_or)
    assert np.array_equal(codes & 0x7F, C_or & 0x7F) and np.array_equal((codes & 0x80)[(C_or & 0x7F) != 0], (C_or & 0x80)[(C_or & 0x7F) != 0])
    Hr, B = oracle.w4a8_gemm_swiglu(A.cpu().numpy(), s.cpu().numpy(), d["q"], d["gscale"], d["w_tscale"], want_bound=True)
    check_gemm(bf16_bits_from_gpu(H), Hr, B, "masked gate/up %d x %d" % (M, N))


# Group counts around the eight that share a fetch of scales (groups 1 .. 8, 9 .. 16, ... and group 0 by itself), rows of scales
# at every alignment, a ragged last channel block, whole and half tiles.
@pytest.mark.parametrize("G", [1, 2, 3, 7, 8, 9, 10, 11, 15, 16, 17, 18, 19, 33])
@pytest.mark.parametrize("lut", [False, True])
def test_scales_of_every_group_count(fq, G, lut):
    rng = np.random.default_rng(G)
    M, N, K = 330, 203, 128 * G
    A = (rng.integers(0, 0x58, (M, K)) | rng.integers(0, 2, (M, K)) << 7).astype(np.uint8)
    q = rng.integers(-8, 8, (N, K), dtype=np.int8)
    gsn = rng.integers(0x08, 0x40, (N, G)).astype(np.uint8)
    a = rng.uniform(0.5, 2.0, M).astype(np.float32)
    packed = fq.fq_pack_weights(_gpu(q))
    fq.fq_test_force_kernel("large")
    try:
        Y = (fq.fq_w4a8_gemm_lut if lut else fq.fq_w4a8_gemm)(_gpu(A), _gpu(a), packed, _gpu(gsn), 0.5, N)
        torch.cuda.synchronize()
    finally:
        fq.fq_test_force_kernel(None)
    Yr, B = (oracle.w4a8_gemm_lut if lut else oracle.w4a8_gemm)(A, a, q, gsn, 0.5, want_bound=True)
    check_gemm(bf16_bits_from_gpu(Y), Yr, B, "G = %d" % G)


# ---- the K-split kernel (8-wave workgroups that split K inside the workgroup) --------------------------

KSPLIT_SHAPES = [(65, 64, 1024), (128, 128, 1024), (300, 256, 1024), (129, 200, 1408), (512, 520, 2048),
                 (100, 96, 11008), (130, 64, 16384), (257, 513, 1024),
                 # 256 x 128 tiles with K halved
                 (700, 1100, 2048), (1024, 512, 4096), (600, 264, 11008), (513, 130, 1408)]


def test_few_tile_shapes_take_the_k_split_kernel(fq):
    assert _plan(fq, (128, 14336, 4096))["kernel"] == "ksplit128x64"
    assert _plan(fq, (512, 4096, 4096))["kernel"] == "ksplit128x64"
    assert _plan(fq, (512, 14336, 4096))["kernel"] == "large"              # more than one round of 128 x 64 tiles
    assert _plan(fq, (2048, 11008, 4096))["kernel"] == "large"
    # workgroups that share a tile along K: as many as fill the compute units, two groups or more per K split each
    assert _plan(fq, (128, 4096, 4096))["ksplit_slices"] == 4
    assert _plan(fq, (128, 4096, 11008))["ksplit_slices"] == 4
    assert _plan(fq, (256, 4096, 4096))["ksplit_slices"] == 2
    assert _plan(fq, (512, 4096, 4096))["ksplit_slices"] == 1
    assert _plan(fq, (100, 96, 11008))["ksplit_slices"] == 8
    assert _plan(fq, (129, 200, 1408))["ksplit_slices"] == 1
    fq.fq_test_force_kernel("ksplit")
    try:
        for shape in KSPLIT_SHAPES:
            assert _plan(fq, shape)["kernel"] == ("ksplit128x64" if shape[0] <= 512 else "ksplit256x128"), shape
    finally:
        fq.fq_test_force_kernel(None)


@pytest.mark.parametrize("shape", KSPLIT_SHAPES)
def test_k_split_kernel_every_element(fq, shape):
    """Plain GEMM, residual out of place and in place, on the K-split kernel: even and ragged tiles, K splits of
    unequal length (K/128 = 11, 43 + 43), several rounds of zero-point units (K = 16384), against the oracle; and the
    large-M kernel's result on the same operands within the FP32 summation-order margin."""
    M, N, K = shape
    d = _problem(shape, seed=7 * M + N + K)
    A, s = fq.fq_quantize_act(to_gpu_bf16(d["X_bf16"]))
    packed, gs = fq.fq_pack_weights(_gpu(d["q"])), _gpu(d["gscale"])
    An, sn = A.cpu().numpy(), s.cpu().numpy()
    Rb = workloads.draw_residual(M, N, scale=4.0, seed=M + N)
    R = to_gpu_bf16(Rb)
    try:
        fq.fq_test_force_kernel("ksplit")
        Yk = fq.fq_w4a8_gemm(A, s, packed, gs, d["w_tscale"], N)
        Ya = fq.fq_w4a8_gemm_add(A, s, packed, gs, d["w_tscale"], N, R)
        torch.cuda.synchronize()
        assert np.array_equal(bf16_bits_from_gpu(R), Rb)
        Yi = fq.fq_w4a8_gemm_add(A, s, packed, gs, d["w_tscale"], N, R, out=R)
        Yk2 = fq.fq_w4a8_gemm(A, s, packed, gs, d["w_tscale"], N)
        fq.fq_test_force_kernel("large")
        Yl = fq.fq_w4a8_gemm(A, s, packed, gs, d["w_tscale"], N)
        torch.cuda.synchronize()
    finally:
        fq.fq_test_force_kernel(None)
    Y, B = oracle.w4a8_gemm(An, sn, d["q"], d["gscale"], d["w_tscale"], want_bound=True)
    check_gemm(bf16_bits_from_gpu(Yk), Y, B, "k-split %s" % (shape,))
    assert np.array_equal(bf16_bits_from_gpu(Yk), bf16_bits_from_gpu(Yk2)), "not deterministic"
    diff = np.abs(oracle.bf16_bits_to_f64(bf16_bits_from_gpu(Yk)) - oracle.bf16_bits_to_f64(bf16_bits_from_gpu(Yl)))
    assert np.all(diff <= oracle.bf16_ulp_array(Y) + 1e-4 * B)
    Yr, Br = oracle.w4a8_gemm_add(An, sn, d["q"], d["gscale"], d["w_tscale"], Rb, want_bound=True)
    check_gemm(bf16_bits_from_gpu(Ya), Yr, Br, "k-split + residual %s" % (shape,))
    assert np.array_equal(bf16_bits_from_gpu(Yi), bf16_bits_from_gpu(Ya)), "in place differs"


# 56 < M <= 64 with at least half a round of 64 x 64 tiles: the K-split kernel without a workspace (zero point through
# the matrix cores); ragged last channel tile (8200), K splits of unequal length (K / 128 = 11), every K split a ghost
# step short of the others (K / 128 = 9)
KSPLIT64_SHAPES = [(64, 8192, 1024), (57, 16384, 1024), (60, 8200, 1408), (64, 8256, 1152)]


@pytest.mark.parametrize("shape", KSPLIT64_SHAPES)
def test_k_split_kernel_without_workspace_every_element(fq, shape):
    """Plain GEMM and residual (out of place, in place) on 64 x 64 tiles against the oracle, and against the M <= 64
    kernel, whose arithmetic it shares (same zero-point instruction, same order inside a group): equal within the FP32
    summation-order margin."""
    M, N, K = shape
    assert _plan(fq, shape)["kernel"] == "ksplit64x64" and fq.fq_w4a8_gemm_workspace_bytes(M, N, K) == 0
    d = _problem(shape, seed=5 * M + N + K)
    A, s = fq.fq_quantize_act(to_gpu_bf16(d["X_bf16"]))
    packed, gs = fq.fq_pack_weights(_gpu(d["q"])), _gpu(d["gscale"])
    An, sn = A.cpu().numpy(), s.cpu().numpy()
    Rb = workloads.draw_residual(M, N, scale=4.0, seed=M + N)
    R = to_gpu_bf16(Rb)
    try:
        Yk = fq.fq_w4a8_gemm(A, s, packed, gs, d["w_tscale"], N)
        Ya = fq.fq_w4a8_gemm_add(A, s, packed, gs, d["w_tscale"], N, R)
        torch.cuda.synchronize()
        assert np.array_equal(bf16_bits_from_gpu(R), Rb)
        Yi = fq.fq_w4a8_gemm_add(A, s, packed, gs, d["w_tscale"], N, R, out=R)
        Yk2 = fq.fq_w4a8_gemm(A, s, packed, gs, d["w_tscale"], N)
        fq.fq_test_force_kernel("small")
        assert _plan(fq, shape)["kernel"] == "smallm"
        Ys = fq.fq_w4a8_gemm(A, s, packed, gs, d["w_tscale"], N)
        torch.cuda.synchronize()
    finally:
        fq.fq_test_force_kernel(None)
    Y, B = oracle.w4a8_gemm(An, sn, d["q"], d["gscale"], d["w_tscale"], want_bound=True)
    check_gemm(bf16_bits_from_gpu(Yk), Y, B, "k-split 64 x 64 %s" % (shape,))
    assert np.array_equal(bf16_bits_from_gpu(Yk), bf16_bits_from_gpu(Yk2)), "not deterministic"
    diff = np.abs(oracle.bf16_bits_to_f64(bf16_bits_from_gpu(Yk)) - oracle.bf16_bits_to_f64(bf16_bits_from_gpu(Ys)))
    assert np.all(diff <= oracle.bf16_ulp_array(Y) + 1e-4 * B)
    Yr, Br = oracle.w4a8_gemm_add(An, sn, d["q"], d["gscale"], d["w_tscale"], Rb, want_bound=True)
    check_gemm(bf16_bits_from_gpu(Ya), Yr, Br, "k-split 64 x 64 + residual %s" % (shape,))
    assert np.array_equal(bf16_bits_from_gpu(Yi), bf16_bits_from_gpu(Ya)), "in place differs"


def test_k_split_kernel_without_workspace_keeps_to_its_shapes(fq):
    assert _plan(fq, (64, 14336, 4096))["kernel"] == "ksplit64x64"          # the decode sweep's largest batch
    assert _plan(fq, (56, 14336, 4096))["kernel"] == "smallm"               # below the top of the range
    assert _plan(fq, (64, 4096, 4096))["kernel"] == "smallm"                # a quarter of a round of tiles
    assert _plan(fq, (64, 14336, 11008))["kernel"] == "smallm"              # long K
    assert _plan(fq, (64, 16448, 4096))["kernel"] == "smallm"               # more than one round
    assert _plan(fq, (64, 8192, 512))["kernel"] == "smallm"                 # fewer than two groups per K split
    assert _plan(fq, (65, 14336, 4096))["kernel"] == "ksplit128x64"


def test_k_split_kernel_zero_activations_return_the_residual(fq):
    for shape in [(300, 264, 1024), (1024, 640, 2048), (700, 1032, 2048)]:
        M, N, K = shape
        q = np.random.default_rng(M).integers(-8, 8, (N, K), dtype=np.int8)
        gs = np.full((N, K // 128), 0x38, np.uint8)
        Rb = np.random.default_rng(N).integers(0, 0x7F80, (M, N)).astype(np.uint16)
        Rb |= np.random.default_rng(N + 1).integers(0, 2, (M, N)).astype(np.uint16) << 15
        Rb[Rb == 0x8000] = 0
        try:
            fq.fq_test_force_kernel("ksplit")
            Yg = fq.fq_w4a8_gemm_add(_gpu(np.zeros((M, K), np.uint8)), _gpu(np.ones(M, np.float32)),
                                     fq.fq_pack_weights(_gpu(q)), _gpu(gs), 1.0, N, to_gpu_bf16(Rb))
            torch.cuda.synchronize()
        finally:
            fq.fq_test_force_kernel(None)
        bad = np.argwhere(bf16_bits_from_gpu(Yg) != Rb)
        assert bad.size == 0, "%s: first wrong element %s" % (shape, bad[:1])


def test_a_prepared_workspace_serves_several_sliced_gemms(fq):
    """Projections that share one activation matrix run one after the other on the workspace the quantiser
    prepared: the tiles' arrival counters are back at zero after every call, so each result equals the one a
    freshly prepared workspace gives, bit for bit, and matches the oracle."""
    M, K = 128, 4096
    shapes_n = [1024, 320, 1024]
    ds = [_problem((M, N, K), seed=90 + i) for i, N in enumerate(shapes_n)]
    X = to_gpu_bf16(ds[0]["X_bf16"])
    need = max(fq.fq_w4a8_gemm_workspace_bytes(M, N, K) for N in shapes_n)
    for N in shapes_n:
        assert _plan(fq, (M, N, K))["ksplit_slices"] == 4
    ws = torch.empty((need,), dtype=torch.uint8, device="cuda")
    A, s = fq.fq_quantize_act(X, workspace=ws)
    outs = []
    for d, N in zip(ds, shapes_n):
        packed, gs = fq.fq_pack_weights(_gpu(d["q"])), _gpu(d["gscale"])
        outs.append(fq.fq_w4a8_gemm(A, s, packed, gs, d["w_tscale"], N, workspace=ws, workspace_prepared=True))
    torch.cuda.synchronize()
    An, sn = A.cpu().numpy(), s.cpu().numpy()
    for d, N, Yg in zip(ds, shapes_n, outs):
        packed, gs = fq.fq_pack_weights(_gpu(d["q"])), _gpu(d["gscale"])
        fresh = fq.fq_w4a8_gemm(A, s, packed, gs, d["w_tscale"], N)
        torch.cuda.synchronize()
        assert np.array_equal(bf16_bits_from_gpu(Yg), bf16_bits_from_gpu(fresh)), N
        Y, B = oracle.w4a8_gemm(An, sn, d["q"], d["gscale"], d["w_tscale"], want_bound=True)
        check_gemm(bf16_bits_from_gpu(Yg), Y, B, "shared workspace, N = %d" % N)


# (M, N, K) -> the tiles of the K-split kernel that serve it on a 256-unit device: 1 128 x 64, 2 128 x 128; even and ragged
# edges, K splits of equal and unequal length (9, 10, 11, 17 and 19 groups), steps that are no multiple of 4
SPLIT_TILE_SHAPES = [((600, 1024, 1024), 1), ((513, 200, 1408), 1), ((1000, 2040, 1280), 1), ((300, 8200, 1024), 2), ((257, 10000, 1152), 2),
                     ((700, 4104, 2048), 2), ((1025, 3001, 2176), 2), ((1024, 4096, 2432), 2), ((2000, 2048, 2048), 2), ((130, 16384, 2048), 2),
                     ((128, 22016, 1024), 2), ((513, 6144, 1280), 2)]


@pytest.mark.parametrize("shape,tiles", SPLIT_TILE_SHAPES)
def test_large_m_range_on_k_split_tiles(fq, shape, tiles):
    """Problems of the large-M range whose 128-row tiles fit on the device at once: plain, with the residual and in place against
    the oracle (all rows, sampled channels with both edges), and close to the large-M kernel's own tiles."""
    M, N, K = shape
    plan = fq.fq_w4a8_gemm_plan(M, N, K, 256)
    assert plan["kernel"] == ("ksplit128x64" if tiles == 1 else "ksplit128x128") and plan["ksplit_slices"] == 1
    assert plan["ksplit_tiles"] == -(-M // 128) * -(-N // (64 * tiles))
    assert fq.fq_w4a8_gemm_workspace_bytes(M, N, K) == 2 * (2 * -(-(K // 128) // 16)) * M * 16 + (4096 if M <= 512 else 0)
    d = _problem(shape, seed=M + N + K)
    A, s = fq.fq_quantize_act(to_gpu_bf16(d["X_bf16"]))
    packed, gs = fq.fq_pack_weights(_gpu(d["q"])), _gpu(d["gscale"])
    Rb = workloads.draw_residual(M, N, scale=workloads.RESIDUAL_SCALE, seed=N)
    R = to_gpu_bf16(Rb)
    Y = fq.fq_w4a8_gemm(A, s, packed, gs, d["w_tscale"], N)
    YR = fq.fq_w4a8_gemm_add(A, s, packed, gs, d["w_tscale"], N, R)
    fq.fq_w4a8_gemm_add(A, s, packed, gs, d["w_tscale"], N, R, out=R)
    fq.fq_test_force_kernel("large")
    try:
        YL = fq.fq_w4a8_gemm(A, s, packed, gs, d["w_tscale"], N)
        torch.cuda.synchronize()
    finally:
        fq.fq_test_force_kernel(None)
    assert torch.equal(YR, R)
    pick = np.unique(np.concatenate([np.arange(min(N, 130)), np.arange(max(0, N - 130), N), np.arange(0, N, 61)]))
    A_ref, s_ref = A.cpu().numpy(), s.cpu().numpy()
    Yr, B = oracle.w4a8_gemm(A_ref, s_ref, d["q"][pick], d["gscale"][pick], d["w_tscale"], want_bound=True)
    check_gemm(bf16_bits_from_gpu(Y)[:, pick], Yr, B, "split tiles %s" % (shape,))
    # the same sums in another FP32 order: at most one bf16 step + 1e-4 of the terms' magnitudes apart
    y, yl = oracle.bf16_bits_to_f64(bf16_bits_from_gpu(Y))[:, pick], oracle.bf16_bits_to_f64(bf16_bits_from_gpu(YL))[:, pick]
    assert np.all(np.abs(y - yl) <= oracle.bf16_ulp_array(yl) + 1e-4 * B)
    Yr, B = oracle.w4a8_gemm_add(A_ref, s_ref, d["q"][pick], d["gscale"][pick], d["w_tscale"], Rb[:, pick], want_bound=True)
    check_gemm(bf16_bits_from_gpu(YR)[:, pick], Yr, B, "split tiles + residual %s" % (shape,))


# Zero-point units past the two rounds that travel from the start: a third round (71 groups), a second batch of later rounds (260
# groups), on both shapes; the odd number of units of 65 groups; splits that run 4 n + 1, 2 and 3 steps.
@pytest.mark.parametrize("shape,tiles", [((600, 1024, 9088), 1), ((520, 72, 33280), 1), ((1000, 2560, 9088), 2), ((513, 130, 8320), 1),
                                         ((513, 130, 2560), 1), ((513, 130, 3072), 1), ((513, 130, 3584), 1)])
def test_k_split_zero_point_rounds(fq, shape, tiles):
    test_large_m_range_on_k_split_tiles(fq, shape, tiles)


# K slices whose borders fall inside a zero-point unit (11, 14 and 22 groups a slice), with an empty place beside the last unit
@pytest.mark.parametrize("shape", [(100, 96, 11008), (200, 4096, 3584), (129, 1000, 11008)])
def test_k_split_slices_share_zero_point_units(fq, shape):
    assert _plan(fq, shape)["ksplit_slices"] > 1
    test_k_split_kernel_every_element(fq, shape)


# the last round in halves (11 tiles on an XCD's 64 slots) and in quarters: 1 or 2 tiles behind a full round, with a ragged last row
# tile (52 rows: the second to fourth quarter are empty) and a ragged channel edge; quarters alone, odd group counts, two
# rounds of zero-point units
TAIL_SHAPES = [(2048, 9600, 256), (2100, 7304, 384), (300, 2000, 4224), (459, 136, 128)]


@pytest.mark.parametrize("shape", TAIL_SHAPES)
def test_last_round_in_halves_and_quarters(fq, shape):
    fq.fq_test_force_kernel("large")
    try:
        test_plain_gemm_every_element(fq, shape)
        test_residual_every_element_and_in_place(fq, shape)
        test_swiglu_every_element(fq, shape)
        test_zero_activations_return_the_residual_bit_for_bit(fq, shape)
    finally:
        fq.fq_test_force_kernel(None)
