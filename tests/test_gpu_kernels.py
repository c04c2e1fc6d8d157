"""GPU parity of the single kernels against the CPU oracle, through the C ABI.
Sizes span several tiles and ragged tails; the oracle is double precision."""
import numpy as np
import pytest

import oracle as orc
import sb_inputs as si

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def T():
    import torch
    assert torch.cuda.is_available(), "these tests need the GPU"
    return torch


def _dev(T, a):
    a = np.ascontiguousarray(a)
    if a.dtype == np.uint16:
        a = a.view(np.int16)
    return T.from_numpy(a).cuda()


def _rand_w(g, N, K, bf16, std=0.02):
    w = (g.standard_normal((N, K)) * std).astype(np.float32)
    return si.round_to_bf16(w) if bf16 else w


def _oracle_rows(W, x):
    return np.stack([orc.matvec(W, x[m].astype(np.float64)) for m in range(x.shape[0])])


@pytest.mark.parametrize("M,d", [(1, 256), (3, 4096), (8, 5120), (2, 688)])
def test_rmsnorm(T, M, d):
    import paper_2604_12247_amd as sb
    g = np.random.default_rng(M * 1000 + d)
    x = g.standard_normal((M, d)).astype(np.float32) * 0.3
    gain = (1 + 0.1 * g.standard_normal(d)).astype(np.float32)
    out = sb.op_rmsnorm(_dev(T, x), _dev(T, gain), 1e-6).cpu().numpy()
    ref = np.stack([orc.rmsnorm(x[m], gain, 1e-6) for m in range(M)])
    assert np.max(np.abs(out - ref)) <= 2e-6 * np.max(np.abs(ref))


VALU_CASES = [  # (N, K, bf16): N ragged against the 16-row block, K ragged against the 512 stride
    (50, 688, False), (768, 256, False), (1024, 256, True), (100, 4096, True), (4096, 11008, True),
    (37, 2056, False),
]


@pytest.mark.parametrize("N,K,bf16", VALU_CASES)
@pytest.mark.parametrize("M", [1, 3, 8])
def test_gemv_valu(T, N, K, bf16, M):
    import paper_2604_12247_amd as sb
    g = np.random.default_rng(N + K + M)
    W = _rand_w(g, N, K, bf16)
    x = g.standard_normal((M, K)).astype(np.float32)
    y = sb.op_gemv(_dev(T, W), _dev(T, x), sb.PROJ_VALU).cpu().numpy()
    ref = _oracle_rows(W, x)
    assert np.max(np.abs(y - ref)) <= 1e-5 * np.max(np.abs(ref)) + 1e-7


# either side of the lines between one and four weight rows per wave (256 blocks of four; for as few rows as a weight has bytes 512, and 1024
# with K >= 1024 or for gate / up)
@pytest.mark.parametrize("N,K,bf16", [(4080, 264, False), (4096, 264, False), (4097, 1032, True), (8191, 136, False), (8208, 136, True),
                                      (16383, 1032, False), (16400, 1032, True)])
@pytest.mark.parametrize("M", [1, 2, 3, 4, 5])
def test_gemv_valu_rows_per_wave(T, N, K, bf16, M):
    """The rows per wave change who adds a row's products, not how: the bits of a row equal those of eight rows together."""
    import paper_2604_12247_amd as sb
    g = np.random.default_rng(N + K)
    W = _rand_w(g, N, K, bf16)
    x = g.standard_normal((8, K)).astype(np.float32)
    Wd = _dev(T, W)
    y = sb.op_gemv(Wd, _dev(T, x[:M]), sb.PROJ_VALU).cpu().numpy()
    ref = _oracle_rows(W, x[:M])
    assert np.max(np.abs(y - ref)) <= 1e-5 * np.max(np.abs(ref)) + 1e-7
    assert np.array_equal(y, sb.op_gemv(Wd, _dev(T, x), sb.PROJ_VALU).cpu().numpy()[:M])
    if N % 2 == 0:   # the same lines for gate / up, which takes the rows in pairs
        u = sb.op_gate_up(Wd, _dev(T, x[:M]), sb.PROJ_VALU).cpu().numpy()
        assert np.max(np.abs(u - np.stack([orc.swiglu(r) for r in ref]))) <= 1e-4 * np.max(np.abs(ref))
        assert np.array_equal(u, sb.op_gate_up(Wd, _dev(T, x), sb.PROJ_VALU).cpu().numpy()[:M])


MFMA_CASES = [(16, 128), (64, 256), (4096, 4096), (12288, 4096), (4096, 11008), (32000, 4096), (48, 384),
              (15024, 256),      # two row tiles per block, an odd number of tiles: the last block owns one
              (4096, 14336),
              (6144, 4096), (5120, 5120), (5120, 13824)]   # between 4096 and 8192 output rows: one or two tiles per block, by the rows, of four waves


@pytest.mark.parametrize("N,K", MFMA_CASES)
@pytest.mark.parametrize("M", [1, 5, 8])
def test_gemv_mfma(T, N, K, M):
    import paper_2604_12247_amd as sb
    g = np.random.default_rng(N + K + M + 1)
    W = _rand_w(g, N, K, True)
    x = g.standard_normal((M, K)).astype(np.float32)
    Wd = _dev(T, W)
    y = sb.op_gemv(Wd, _dev(T, x), sb.PROJ_MFMA).cpu().numpy()
    ref = _oracle_rows(W, x)
    # activations carry 16 mantissa bits (two bf16 parts): error ~ 2^-17 per term
    assert np.max(np.abs(y - ref)) <= 3e-5 * np.max(np.abs(ref)) + 1e-7
    # the tile-packed copy of the weights gives the same bits
    yp = sb.op_gemv(sb.op_repack(Wd), _dev(T, x), sb.PROJ_MFMA_PACKED).cpu().numpy()
    assert np.array_equal(yp, y)


GEMM_CASES = [(16, 128, 1), (48, 384, 5), (4096, 4096, 128), (12288, 4096, 37), (4096, 11008, 64), (22016, 4096, 128),
              (4112, 256, 17), (8192 + 80, 512, 97), (32000, 4096, 128)]


@pytest.mark.parametrize("N,K,M", GEMM_CASES)
def test_prompt_pass_gemm(T, N, K, M):
    """The projection of the prompt passes (up to 128 rows, k splits added in order) against the
    double-precision product of the same bf16 weights; unwritten rows of the scratch hold NaN."""
    import paper_2604_12247_amd as sb
    g = np.random.default_rng(N + K + M + 2)
    W = _rand_w(g, N, K, True)
    x = g.standard_normal((M, K)).astype(np.float32)
    Wp = sb.op_repack(_dev(T, W))
    scratch = T.empty(sb.lib().sb_op_gemm_scratch_bytes(N, K), dtype=T.uint8, device="cuda")
    scratch.fill_(0xFF)
    y = sb.op_gemm(Wp, _dev(T, x), scratch).cpu().numpy()
    ref = _oracle_rows(W, x)
    assert np.all(np.isfinite(y))
    assert np.max(np.abs(y - ref)) <= 3e-5 * np.max(np.abs(ref)) + 1e-7
    # a row's result does not depend on the rows beside it
    if M > 3:
        y3 = sb.op_gemm(Wp, _dev(T, x[:3]), scratch).cpu().numpy()
        assert np.array_equal(y3, y[:3])


# every height of a pass (1 to 8 column tiles, odd ones straddle the two planes in the staging), one and two weight
# tiles per wave ([4096 x 1024] and [20480 x 2560]), a last row block that is not full ([20496 x ...])
@pytest.mark.parametrize("N,K", [(4096, 1024), (20496, 2560)])
@pytest.mark.parametrize("M", [1, 16, 17, 40, 64, 70, 96, 97, 113, 128])
def test_prompt_pass_gemm_heights(T, N, K, M):
    import paper_2604_12247_amd as sb
    g = np.random.default_rng(N + M)
    W = T.from_numpy(_rand_w(g, N, K, True).view(np.int16)).cuda()
    x = T.from_numpy(g.standard_normal((M, K)).astype(np.float32)).cuda()
    y = sb.op_gemm(sb.op_repack(W), x).double()
    ref = x.double() @ W.view(T.bfloat16).double().t()
    # 16 mantissa bits per activation: 2^-17 a term, fp32 sums over K <= 2560
    assert float((y - ref).abs().max()) <= 3e-5 * float(ref.abs().max())


# the epilogue's two forms (512 blocks of 256 columns and 16 rows: N = 20480 at seven and six column tiles) with one to four weight
# tiles in the last wave, rows that end inside a column tile, one and several partial sums
@pytest.mark.parametrize("N", [20480, 20496, 20512, 20528, 48])
@pytest.mark.parametrize("K", [128, 1280])
@pytest.mark.parametrize("M", [90, 100, 33])
def test_prompt_pass_gemm_last_columns(T, N, K, M):
    import paper_2604_12247_amd as sb
    g = T.Generator(device="cuda")
    g.manual_seed(N + K + M)
    W = (T.randn(N, K, generator=g, device="cuda") * 0.02).to(T.bfloat16)
    x = T.randn(M, K, generator=g, device="cuda")
    y = sb.op_gemm(sb.op_repack(W), x).double()
    ref = x.double() @ W.double().t().contiguous()
    assert float((y - ref).abs().max()) <= 3e-5 * float(ref.abs().max())   # 16-bit activation parts, as in test_prompt_pass_gemm


# rows on a 16-byte boundary are split into their two parts inside the GEMM, any others by a launch of their own: the same bits, at every
# number of column tiles (a last unit of 16 or 32 rows), one and two weight tiles per wave, steps requested singly and whole; no row past
# the last is read into a result
@pytest.mark.parametrize("N,K", [(4096, 1024), (20480, 2560), (20480, 6528)])
@pytest.mark.parametrize("M", [9, 16, 17, 47, 64, 65, 95, 112, 127, 128])
def test_prompt_pass_gemm_unaligned_rows(T, N, K, M):
    import paper_2604_12247_amd as sb
    g = T.Generator(device="cuda")
    g.manual_seed(N + K + M)
    Wp = sb.op_repack((T.randn(N, K, generator=g, device="cuda") * 0.02).to(T.bfloat16))
    buf = T.full((4 + M * K + 1,), float("nan"), device="cuda")
    buf[4:-1] = T.randn(M * K, generator=g, device="cuda")
    x = buf[4:-1].view(M, K)
    off = T.full((M * K + 1,), float("nan"), device="cuda")
    off[1:] = x.reshape(-1)
    z = off[1:].view(M, K)
    assert x.data_ptr() % 16 == 0 and z.data_ptr() % 16 == 4
    assert T.equal(sb.op_gemm(Wp, x), sb.op_gemm(Wp, z))


# rows that the caller left where the partial sums come: they are read whole before the first is written (65536: thread blocks of two row
# blocks, of which the first's sums are stored while all blocks have half the rows' products before them)
@pytest.mark.parametrize("N,K,M", [(4096, 4096, 100), (65536, 512, 128)])
def test_prompt_pass_gemm_rows_in_the_scratch_area(T, N, K, M):
    import paper_2604_12247_amd as sb
    g = T.Generator(device="cuda")
    g.manual_seed(N + K + M)
    Wp = sb.op_repack((T.randn(N, K, generator=g, device="cuda") * 0.02).to(T.bfloat16))
    x = T.randn(M, K, generator=g, device="cuda")
    y = sb.op_gemm(Wp, x)
    planes = 2 * 128 * K * 2                                    # the rows' two parts come first, then the partial sums
    scratch = T.empty(sb.lib().sb_op_gemm_scratch_bytes(N, K), dtype=T.uint8, device="cuda")
    inside = scratch[planes:planes + 4 * M * K].view(T.float32).view(M, K)
    inside.copy_(x)
    assert T.equal(sb.op_gemm(Wp, inside, scratch), y)


# a single pass whose thread blocks own 9, 10, 15, 16 and 17 k blocks: odd numbers of weight blocks are requested whole
@pytest.mark.parametrize("N,K", [(17088, 4096), (7184, 10368), (20480, 6144), (20480, 6528), (20480, 6784)])
@pytest.mark.parametrize("M", [9, 40, 128])
def test_prompt_pass_gemm_long_ranges(T, N, K, M):
    import paper_2604_12247_amd as sb
    g = T.Generator(device="cuda")
    g.manual_seed(N + K + M)
    W = (T.randn(N, K, generator=g, device="cuda") * 0.02).to(T.bfloat16)
    x = T.randn(M, K, generator=g, device="cuda")
    scratch = T.empty(sb.lib().sb_op_gemm_scratch_bytes(N, K), dtype=T.uint8, device="cuda")
    y = sb.op_gemm(sb.op_repack(W), x, scratch).double()
    ref = x.double() @ W.double().t().contiguous()
    assert float((y - ref).abs().max()) <= 3e-5 * float(ref.abs().max())   # 16-bit activation parts, as in test_prompt_pass_gemm


# every number of k blocks that a wave is left with at the end (and waves without any): eight waves and a ring of two, four and a ring of three
# with one and two tiles, and the gate / up form with two pairs of tiles
@pytest.mark.parametrize("kb", [1, 2, 3, 4, 5, 7, 8, 9, 11, 13, 16, 17, 20, 23, 24, 25, 29, 33, 41, 47])
def test_gemv_mfma_last_blocks(T, kb):
    import paper_2604_12247_amd as sb
    K = 128 * kb
    g = T.Generator(device="cuda")
    g.manual_seed(kb)
    for N, M in ((528, 1), (528, 8), (4128, 2), (8208, 1), (12320, 6)):
        W = (T.randn(N, K, generator=g, device="cuda") * 0.02).to(T.bfloat16)
        x = T.randn(M, K, generator=g, device="cuda")
        ref = x.double() @ W.double().t().contiguous()
        y, yp = sb.op_gemv(W, x, sb.PROJ_MFMA), sb.op_gemv(sb.op_repack(W), x, sb.PROJ_MFMA_PACKED)
        assert T.equal(y, yp)
        assert float((y.double() - ref).abs().max()) <= 3e-5 * float(ref.abs().max())   # 16-bit activation parts, as in test_prompt_pass_gemm
    if kb >= 33:   # (K > 4096)
        N, M = 12320, 3
        W = (T.randn(2 * N, K, generator=g, device="cuda") * 0.02).to(T.bfloat16)
        x = T.randn(M, K, generator=g, device="cuda")
        z = x.double() @ W.double().t().contiguous()
        ref = T.nn.functional.silu(z[:, :N]) * z[:, N:]
        y = sb.op_gate_up(sb.op_repack(W), x, sb.PROJ_MFMA_PACKED).double()
        # the two factors are off by at most 3e-5 of their largest value each; silu's slope is at most 1.1
        assert float((y - ref).abs().max()) <= 2.1 * 3e-5 * float(z.abs().max()) ** 2


# either side of the lines between the block shapes (4096, 6144, 8192 and 12288 output rows, K = 2048, 4096 and 8192, three and five rows)
@pytest.mark.parametrize("N,K", [(4112, 4096), (4112, 1920), (4112, 8320), (6144, 2048), (6160, 2048), (8176, 256), (8192, 2048), (8208, 4224),
                                 (12288, 384), (12304, 384), (12304, 4224)])
@pytest.mark.parametrize("kernel", ["mfma", "mfma_packed"])
def test_gemv_mfma_block_shapes(T, kernel, N, K):
    import paper_2604_12247_amd as sb
    k = {"mfma": sb.PROJ_MFMA, "mfma_packed": sb.PROJ_MFMA_PACKED}[kernel]
    g = np.random.default_rng(N + K)
    W = _rand_w(g, N, K, True)
    x = g.standard_normal((8, K)).astype(np.float32)
    Wd = _dev(T, W)
    if kernel == "mfma_packed":
        Wd = sb.op_repack(Wd)
    y8 = sb.op_gemv(Wd, _dev(T, x), k).cpu().numpy()
    ref = _oracle_rows(W, x)
    assert np.max(np.abs(y8 - ref)) <= 3e-5 * np.max(np.abs(ref))     # 16-bit activation parts, as in test_gemv_mfma
    for M in (1, 2, 3, 4, 5, 7):
        assert np.array_equal(sb.op_gemv(Wd, _dev(T, x[:M]), k).cpu().numpy(), y8[:M]), M


# k blocks 0, 4 and 12 hold 2^24, 1 and 1: a wave that owns all three loses both ones to its 2^24, one that does not own the first adds them up
@pytest.mark.parametrize("kernel", ["mfma", "mfma_packed"])
@pytest.mark.parametrize("N", [4096, 4112, 6144, 6160, 8192, 8208, 12288, 12304, 16384])
@pytest.mark.parametrize("K", [2048, 4096, 4224])
def test_gemv_mfma_order_of_additions(T, kernel, N, K):
    """k blocks are dealt to eight waves up to 4096 output rows and to four above, whatever K, the rows and the form of the weights."""
    import paper_2604_12247_amd as sb
    W = T.zeros(N, K, dtype=T.bfloat16, device="cuda")
    for kb, v in ((0, 2.0 ** 24), (4, 1), (12, 1)):
        W[:, kb * 128] = v
    if kernel == "mfma_packed":
        W = sb.op_repack(W)
    for M in (1, 3, 8):
        y = sb.op_gemv(W, T.ones(M, K, device="cuda"), sb.PROJ_MFMA_PACKED if kernel == "mfma_packed" else sb.PROJ_MFMA)
        assert bool((y == 2.0 ** 24 + (2 if N <= 4096 else 0)).all()), M


GATE_UP_SHAPES = [(64, 256, 3), (11008, 4096, 1), (11008, 4096, 6), (14336, 4096, 8)]
GATE_UP_CASES = [(k, *c) for k in ("valu", "mfma", "mfma_packed") for c in GATE_UP_SHAPES] + [("valu", 1000, 512, 5)]


@pytest.mark.parametrize("kernel,N,K,M", GATE_UP_CASES)   # (the MFMA kernels take whole 16-row tiles: no ragged N there)
def test_gate_up_swiglu(T, kernel, N, K, M):
    """The gate/up sweep with its SwiGLU epilogue as the decode path runs it, against the oracle's
    mat-vec and SwiGLU, at the 7B and 8B FFN shapes and a ragged one."""
    import paper_2604_12247_amd as sb
    g = np.random.default_rng(N + K + M)
    W = _rand_w(g, 2 * N, K, True, std=0.03)
    x = g.standard_normal((M, K)).astype(np.float32)
    kid = {"valu": sb.PROJ_VALU, "mfma": sb.PROJ_MFMA, "mfma_packed": sb.PROJ_MFMA_PACKED}[kernel]
    Wd = _dev(T, W)
    if kernel == "mfma_packed":
        Wd = sb.op_repack(Wd)
    u = sb.op_gate_up(Wd, _dev(T, x), kid).cpu().numpy()
    for m in range(M):
        ref = orc.swiglu(orc.matvec(W, x[m].astype(np.float64)))
        scale = np.max(np.abs(ref))
        assert np.max(np.abs(u[m] - ref)) <= 1e-4 * scale, (m, np.max(np.abs(u[m] - ref)), scale)


# one and two pairs of tiles per block: 768 pairs, 769 (the last block owns one), 1024 and 1025, K on either side of 4096
@pytest.mark.parametrize("N,K", [(12288, 4224), (12304, 4224), (12304, 4096), (16384, 4224), (16400, 4224)])
def test_gate_up_pairs_per_block(T, N, K):
    import paper_2604_12247_amd as sb
    g = np.random.default_rng(N + K)
    W = _rand_w(g, 2 * N, K, True, std=0.03)
    x = g.standard_normal((8, K)).astype(np.float32)
    Wp = sb.op_repack(_dev(T, W))
    u8 = sb.op_gate_up(Wp, _dev(T, x), sb.PROJ_MFMA_PACKED).cpu().numpy()
    for m in (0, 7):
        ref = orc.swiglu(orc.matvec(W, x[m].astype(np.float64)))
        assert np.max(np.abs(u8[m] - ref)) <= 1e-4 * np.max(np.abs(ref)), m
    for M in (1, 2, 3, 5):
        assert np.array_equal(sb.op_gate_up(Wp, _dev(T, x[:M]), sb.PROJ_MFMA_PACKED).cpu().numpy(), u8[:M]), M


@pytest.mark.parametrize("kernel", ["valu", "mfma", "mfma_packed"])
def test_gemv_row_result_does_not_depend_on_m(T, kernel):
    """A row's output is bit-identical whether it is computed alone or with others."""
    import paper_2604_12247_amd as sb
    k = {"valu": sb.PROJ_VALU, "mfma": sb.PROJ_MFMA, "mfma_packed": sb.PROJ_MFMA_PACKED}[kernel]
    g = np.random.default_rng(5)
    for N, K in ((4096, 4096), (1024, 11008), (32000, 256), (6144, 512), (15360, 256)):
        W = _dev(T, _rand_w(g, N, K, True))
        if kernel == "mfma_packed":
            W = sb.op_repack(W)
        x = g.standard_normal((8, K)).astype(np.float32)
        y8 = sb.op_gemv(W, _dev(T, x), k).cpu().numpy()
        for M in (1, 2, 5):
            yM = sb.op_gemv(W, _dev(T, x[:M]), k).cpu().numpy()
            assert np.array_equal(yM, y8[:M]), (N, K, M)
        # and a row does not care which slot it sits in
        y1 = sb.op_gemv(W, _dev(T, x[3:4]), k).cpu().numpy()
        assert np.array_equal(y1[0], y8[3])


@pytest.mark.parametrize("kernel", ["valu", "mfma", "mfma_packed"])
@pytest.mark.parametrize("N,K,M", [(1024, 256, 1), (32000, 4096, 1), (32000, 4096, 6), (128256, 512, 2), (128256, 4096, 3),
                                   (15024, 256, 3)])   # an odd number of 16-row tiles, two per block
def test_head_argmax_and_confidence(T, kernel, N, K, M):
    import paper_2604_12247_amd as sb
    k = {"valu": sb.PROJ_VALU, "mfma": sb.PROJ_MFMA, "mfma_packed": sb.PROJ_MFMA_PACKED}[kernel]
    g = np.random.default_rng(N + K + M)
    W = _rand_w(g, N, K, True, std=0.05)
    x = g.standard_normal((M, K)).astype(np.float32)
    Wd = sb.op_repack(_dev(T, W)) if kernel == "mfma_packed" else _dev(T, W)
    for Tl in (2.0, 1.0):
        am, cf, z = sb.op_head(Wd, _dev(T, x), Tl, k, want_logits=True)
        am, cf, z = am.cpu().numpy(), cf.cpu().numpy(), z.cpu().numpy()
        ref = _oracle_rows(W, x)
        assert np.max(np.abs(z - ref)) <= 2e-2 * np.max(np.abs(ref))
        assert np.max(np.abs(z - ref)) <= 1e-4 * np.max(np.abs(ref))      # what the kernels actually reach
        for m in range(M):
            o_am, o_cf = orc.act(ref[m], Tl)
            top2 = np.sort(ref[m])[-2:]
            if top2[1] - top2[0] >= 1e-2:
                assert am[m] == o_am
            assert am[m] == int(np.argmax(z[m]))      # consistent with its own logits, lowest index
            assert abs(cf[m] - o_cf) <= 1e-3
            assert abs(cf[m] - o_cf) <= 1e-5 + 1e-4 * o_cf


def test_head_ties_take_lowest_index(T):
    import paper_2604_12247_amd as sb
    # identical weight rows give exactly equal logits in any arithmetic
    g = np.random.default_rng(9)
    row = si.round_to_bf16((g.standard_normal(256) * 0.05).astype(np.float32))
    W = si.round_to_bf16((g.standard_normal((1024, 256)) * 0.001).astype(np.float32))
    x = si.bf16_to_f32(row).astype(np.float32)[None, :] * 4
    for rows in ((700, 33), (5, 1000), (512, 511)):
        W2 = W.copy()
        for r in rows:
            W2[r] = row
        for k in (sb.PROJ_VALU, sb.PROJ_MFMA, sb.PROJ_MFMA_PACKED):
            Wd = sb.op_repack(_dev(T, W2)) if k == sb.PROJ_MFMA_PACKED else _dev(T, W2)
            am, cf, _ = sb.op_head(Wd, _dev(T, x), 1.0, k)
            assert int(am.cpu()[0]) == min(rows)


# block partials of a row (VALU: 16 weight rows each; MFMA from 15000 rows: 32): 128 threads a row up to 1024 of them, 256 up to
# 4096, 512 above, and from 8193 on more than these hold in registers
@pytest.mark.parametrize("kernel,N", [("valu", 16), ("valu", 2064), ("valu", 16384), ("valu", 16400), ("mfma_packed", 32768),
                                      ("mfma_packed", 32784), ("valu", 65536), ("valu", 65552), ("valu", 131072), ("valu", 140000)])
def test_head_merge_edges(T, kernel, N):
    """Confidence of every row against 64 bits from the same logits, the same bits whatever rows are beside it."""
    import paper_2604_12247_amd as sb
    k = {"valu": sb.PROJ_VALU, "mfma_packed": sb.PROJ_MFMA_PACKED}[kernel]
    g = np.random.default_rng(N)
    W = _rand_w(g, N, 128, True, std=0.2)
    x = g.standard_normal((8, 128)).astype(np.float32)
    Wd = sb.op_repack(_dev(T, W)) if kernel == "mfma_packed" else _dev(T, W)
    am, cf, z = (t.cpu().numpy() for t in sb.op_head(Wd, _dev(T, x), 1.3, k, want_logits=True))
    z64 = z.astype(np.float64)
    ref = 1.0 / np.exp((z64 - z64.max(1, keepdims=True)) / 1.3).sum(1)
    assert np.array_equal(am, z.argmax(1))
    # a term: exp of an argument up to 16 rounded once by 2^-24 of it (1e-6) and two products; the sums add less
    assert np.max(np.abs(cf - ref) / ref) <= 4e-6
    for M in (1, 2, 3, 5):
        amM, cfM, _ = (None if t is None else t.cpu().numpy() for t in sb.op_head(Wd, _dev(T, x[:M]), 1.3, k))
        assert np.array_equal(amM, am[:M]) and np.array_equal(cfM, cf[:M]), M


@pytest.mark.parametrize("kernel,N", [("valu", 2064), ("mfma_packed", 32000), ("valu", 16400), ("valu", 70000), ("valu", 140000)])
def test_head_confidence_of_non_finite_logits_is_nan(T, kernel, N):
    """A logit that is not a number, or a row of which no logit is finite, leaves no confidence."""
    import paper_2604_12247_amd as sb
    k = {"valu": sb.PROJ_VALU, "mfma_packed": sb.PROJ_MFMA_PACKED}[kernel]
    g = np.random.default_rng(N + 1)
    W = _rand_w(g, N, 128, True)
    x = np.abs(g.standard_normal((3, 128))).astype(np.float32) + 0.1

    def conf(W, x):
        Wd = sb.op_repack(_dev(T, W)) if kernel == "mfma_packed" else _dev(T, W)
        return sb.op_head(Wd, _dev(T, x), 1.0, k)[1].cpu().numpy()

    good = conf(W, x)
    assert np.all(np.isfinite(good))
    xn = x.copy()
    xn[1] = np.nan   # every logit of row 1
    c = conf(W, xn)
    assert np.isnan(c[1]) and c[0] == good[0] and c[2] == good[2]
    for n in (0, N // 2 + 5, N - 1):   # one logit of every row: the first, the last, one inside a block
        Wn = W.copy()
        Wn[n] = 0x7fc0
        assert np.all(np.isnan(conf(Wn, x))), n
    W[:] = 0xff80    # -inf: no finite logit (the bf16 pairs of the matrix cores make NaN of it, the same here)
    assert np.all(np.isnan(conf(W, x)))


def _bf16_value(a):
    return si.bf16_to_f32(si.round_to_bf16(a))


def _rotated(k, c, s):
    """Keys [M, heads, hd] rotated as a decode pass stores them: x cos - (y sin), x sin + (y cos), the product in brackets rounded by
    itself and the rest once (64 mantissa bits hold the other product; the sum is rounded twice, which 3e4 values do not show)."""
    h = k.shape[-1] // 2
    x, y, c, s = k[..., :h], k[..., h:], c[:, None], s[:, None]
    L = np.longdouble
    return np.concatenate([(L(1) * x * c - (y * s)).astype(np.float32), (L(1) * x * s + (y * c)).astype(np.float32)], -1)


def _attention_case(T, Hq, Hkv, hd, kv_bf16, n_ctx, M, base, shuffle, seed, oracle=True):
    """Append n_ctx + M rows in passes, then compare the last pass's output rows."""
    import paper_2604_12247_amd as sb
    g = np.random.default_rng(seed)
    kvd = sb.BF16 if kv_bf16 else sb.FP32
    n_tot = n_ctx + M
    n_pages = (n_tot + 15) // 16 + 1
    rows = (Hq + 2 * Hkv) * hd
    qkv = g.standard_normal((n_tot, rows)).astype(np.float32)
    es = 2 if kv_bf16 else 4
    pool = T.empty(3 * 2 * n_pages * Hkv * 16 * hd * es, dtype=T.uint8, device="cuda")
    pool.fill_(0xFF)     # NaN patterns: unwritten cache must never leak into a result
    order = g.permutation(n_pages).astype(np.int32) if shuffle else np.arange(n_pages, dtype=np.int32)
    table = _dev(T, order)
    c, s = sb.rope_table(hd, base, n_pages * 16)
    cd, sd = _dev(T, c), _dev(T, s)
    layer = 1
    pos = 0
    out = None
    passes = [8] * (n_ctx // 8) + ([n_ctx % 8] if n_ctx % 8 else []) + [M]
    scratch = T.empty(sb.lib().sb_op_attention_scratch_bytes(Hq, hd, kvd, n_pages), dtype=T.uint8, device="cuda")
    for m in passes:
        q = _dev(T, qkv[pos:pos + m])
        o = sb.op_attention(q, Hq, Hkv, hd, kvd, pool, table, layer, cd, sd, pos, scratch)
        if pos + m == n_tot:
            out = o.cpu().numpy()
        pos += m
    if not oracle:
        return None, out
    # oracle: rotate, round K/V as the cache does, attend
    def rnd(a):
        return si.bf16_to_f32(si.round_to_bf16(a.astype(np.float32))) if kv_bf16 else a.astype(np.float32)
    K = np.zeros((n_tot, Hkv, hd), np.float32); V = np.zeros_like(K)
    for t in range(n_tot):
        for h in range(Hkv):
            K[t, h] = exact = orc.rope_apply(qkv[t, (Hq + h) * hd:(Hq + h + 1) * hd], t, base)
            if kv_bf16:
                # (as the cache holds it: where the float rotation and the double one lie on two sides of a rounding boundary, a unit of one
                # key apart, 2^-8 of it, moves an output by up to 2^-8 of that key's share of its score; test_new_keys_bits pins the bits)
                K[t, h] = _bf16_value(_rotated(qkv[t:t + 1, (Hq + h) * hd:(Hq + h + 1) * hd][:, None], c[t:t + 1], s[t:t + 1])[0, 0])
                assert np.all(np.abs(K[t, h] - exact) <= 2.0 ** -8 * np.abs(exact) + 1e-6)
            V[t, h] = rnd(qkv[t, (Hq + Hkv + h) * hd:(Hq + Hkv + h + 1) * hd])
    G = Hq // Hkv
    worst = 0.0
    for r in range(M):
        p = n_ctx + r
        for h in range(Hq):
            q = orc.rope_apply(qkv[p, h * hd:(h + 1) * hd], p, base)
            ref = orc.attention_head(q, K[:p + 1, h // G], V[:p + 1, h // G])
            got = out[r, h * hd:(h + 1) * hd]
            worst = max(worst, float(np.max(np.abs(got - ref))))
    return worst, out


ATT_CASES = [  # Hq, Hkv, hd, kv_bf16, n_ctx, M, rope base, shuffled pages
    (4, 4, 64, False, 0, 1, 1e4, False),       # a single key
    (4, 4, 64, False, 29, 4, 1e4, True),
    (4, 2, 64, True, 130, 8, 1e4, True),       # crosses a chunk boundary inside the pass
    (8, 8, 128, True, 300, 6, 1e4, True),
    (8, 2, 128, True, 257, 6, 5e5, True),      # GQA, two query groups
    (2, 2, 128, False, 70, 3, 1e4, False),     # fp32 cache with 64-key chunks
    (8, 8, 128, True, 1018, 6, 1e4, True),     # eight whole 128-key chunks at the last row
    (8, 8, 128, True, 1020, 6, 1e4, True),     # the pass's rows straddle a chunk boundary
    (4, 2, 64, True, 1000, 8, 5e5, True),      # two query heads per kv head, sixteen query columns, head_dim 64, long context
    (8, 8, 128, True, 63, 3, 1e4, False),      # shorter than one chunk
    (8, 8, 128, True, 1030, 5, 1e4, True),     # nine chunks, the last one nearly empty
    (2, 1, 128, True, 65532, 4, 1e4, True),    # the longest context the kernels take: 512 chunks, 4096 shuffled pages
    (32, 32, 128, True, 3300, 6, 1e4, True),   # 32 x 26 blocks: more than the chip holds at once
    (16, 16, 64, True, 8300, 3, 1e4, True),    # 16 x 65 blocks, head_dim 64
    (32, 1, 64, True, 200, 3, 1e4, True),      # one kv head for 32 query heads: six 16-query groups per block
    (16, 1, 128, False, 90, 5, 1e4, False),    # the same on the fp32-cache kernel
]


@pytest.mark.parametrize("case", ATT_CASES)
def test_rope_append_attention(T, case):
    """One call per pass: rotary embedding, KV append and attention over the paged cache."""
    worst, _ = _attention_case(T, *case, seed=sum(int(x) for x in case[:6]))
    assert worst <= 2e-5, worst


def _check_rotated_k_cache(Kc, Ko):
    """Cached K (bf16 bits) against the oracle's.  The kernel rotates in float, the oracle in double:
    a value within float error of a rounding boundary may land on the neighbouring bf16 value (one
    unit in the last place, about 1 element in 30 000), and where the two products of the rotation
    cancel almost completely the float error (<= 2^-22 of the operands, here < 3e-6) can be a few units
    of the tiny result.  Nothing else may differ."""
    dk = np.abs(Kc.astype(np.int32) - Ko.astype(np.int32))
    da = np.abs(si.bf16_to_f32(Kc).astype(np.float64) - si.bf16_to_f32(Ko).astype(np.float64))
    assert not np.any((dk > 1) & (da > 3e-6)), (int(dk.max()), float(da.max()))
    assert (dk != 0).mean() <= 1e-3, float((dk != 0).mean())


PROMPT_ATT_CASES = [  # Hq, Hkv, hd, rows already cached, rows of this call, rope base
    (4, 4, 64, 0, 1, 1e4),          # a single key
    (4, 4, 64, 0, 70, 1e4),         # two query blocks, one chunk
    (4, 2, 64, 37, 200, 1e4),       # GQA, a cached prefix, chunk boundary inside a query block
    (6, 2, 128, 0, 150, 5e5),       # group of 3: query blocks straddle rows
    (8, 8, 128, 130, 333, 1e4),     # several chunks, ragged last block and last page
    (16, 1, 128, 40, 100, 1e4),     # one kv head for 16 query heads: a row fills a wave's 16 queries
]


@pytest.mark.parametrize("case", PROMPT_ATT_CASES)
def test_prompt_attention(T, case):
    """All rows of a prompt pass in one call (running soft-max per query): every output row and the
    cache it leaves against the oracle's attention, rows before pos0 cached by the per-pass kernel."""
    import paper_2604_12247_amd as sb
    Hq, Hkv, hd, n_ctx, M, base = case
    g = np.random.default_rng(5 + sum(int(x) for x in case[:5]))
    n_tot = n_ctx + M
    n_pages = (n_tot + 15) // 16 + 1
    rows = (Hq + 2 * Hkv) * hd
    qkv = (g.standard_normal((n_tot, rows)) * 1.2).astype(np.float32)
    pool = T.empty(2 * 2 * n_pages * Hkv * 16 * hd * 2, dtype=T.uint8, device="cuda")
    pool.fill_(0xFF)
    table = _dev(T, g.permutation(n_pages).astype(np.int32))
    c, s = sb.rope_table(hd, base, n_pages * 16)
    cd, sd = _dev(T, c), _dev(T, s)
    for pos in range(0, n_ctx, 8):
        sb.op_attention(_dev(T, qkv[pos:min(pos + 8, n_ctx)]), Hq, Hkv, hd, sb.BF16, pool, table, 1, cd, sd, pos)
    out = sb.op_prompt_attention(_dev(T, qkv[n_ctx:]), Hq, Hkv, hd, pool, table, 1, cd, sd, n_ctx).cpu().numpy()
    # a decode-style pass after it reads the cache the call left
    nxt = (g.standard_normal((1, rows))).astype(np.float32)
    after = sb.op_attention(_dev(T, nxt), Hq, Hkv, hd, sb.BF16, pool, table, 1, cd, sd, n_tot).cpu().numpy()

    # The cache first.  V is a plain rounding of the input: exact.  K is rounded after the rotation:
    # equal to the oracle's but for float rounding (_check_rotated_k_cache).  The attention below is
    # then checked against the oracle's attention over the keys the cache holds.
    raw = pool.view(T.int16).cpu().numpy().view(np.uint16).reshape(2, 2, n_pages, Hkv, 16 * hd)
    tbl = table.cpu().numpy()
    Kc = np.zeros((n_tot + 1, Hkv, hd), np.uint16); Vc = np.zeros_like(Kc)
    for t in range(n_tot + 1):
        pg = tbl[t // 16]
        for h in range(Hkv):
            Kc[t, h] = raw[1, 0, pg, h].reshape(16, hd)[t % 16]
            Vc[t, h] = raw[1, 1, pg, h].reshape(hd, 16)[:, t % 16]
    allq = np.concatenate([qkv, nxt])
    Ko = np.zeros_like(Kc); Vo = np.zeros_like(Kc)
    for t in range(n_tot + 1):
        for h in range(Hkv):
            Ko[t, h] = si.round_to_bf16(orc.rope_apply(allq[t, (Hq + h) * hd:(Hq + h + 1) * hd], t, base).astype(np.float32))
            Vo[t, h] = si.round_to_bf16(allq[t, (Hq + Hkv + h) * hd:(Hq + Hkv + h + 1) * hd])
    assert np.array_equal(Vc, Vo)
    _check_rotated_k_cache(Kc, Ko)
    K, V = si.bf16_to_f32(Kc), si.bf16_to_f32(Vc)
    G = Hq // Hkv
    worst = 0.0
    check_rows = range(M) if M <= 80 else sorted(set(list(range(0, M, 7)) + [63, 64, 127, 128, M - 2, M - 1]) & set(range(M)))
    for r in check_rows:
        p = n_ctx + r
        for h in range(Hq):
            q = orc.rope_apply(qkv[p, h * hd:(h + 1) * hd], p, base)
            ref = orc.attention_head(q, K[:p + 1, h // G], V[:p + 1, h // G])
            worst = max(worst, float(np.max(np.abs(out[r, h * hd:(h + 1) * hd] - ref))))
    assert worst <= 2e-5, worst
    for h in range(Hq):
        q = orc.rope_apply(nxt[0, h * hd:(h + 1) * hd], n_tot, base)
        ref = orc.attention_head(q, K[:, h // G], V[:, h // G])
        assert np.max(np.abs(after[0, h * hd:(h + 1) * hd] - ref)) <= 2e-5


@pytest.mark.parametrize("hd,n_ctx,M", [(128, 2048 + 40, 2048), (64, 0, 2048 + 77)])
def test_prompt_attention_wide_form(T, hd, n_ctx, M):
    """Launches large enough for the form with 32 queries per wave (32 kv heads x >= 2048 queries): sampled
    heads and rows against the oracle's attention over the keys the cache holds, cache of those heads
    checked as above.  The prefix, where there is one, is itself written by a call of the same kind."""
    import paper_2604_12247_amd as sb
    Hq = Hkv = 32
    base = 1e4
    g = np.random.default_rng(900 + hd)
    n_tot = n_ctx + M
    n_pages = (n_tot + 15) // 16 + 3
    rows = (Hq + 2 * Hkv) * hd
    qkv = (g.standard_normal((n_tot, rows)) * 1.2).astype(np.float32)
    pool = T.empty(2 * n_pages * Hkv * 16 * hd * 2, dtype=T.uint8, device="cuda")
    pool.fill_(0xFF)
    table = _dev(T, g.permutation(n_pages).astype(np.int32))
    c, s = sb.rope_table(hd, base, n_pages * 16)
    cd, sd = _dev(T, c), _dev(T, s)
    if n_ctx:
        sb.op_prompt_attention(_dev(T, qkv[:n_ctx]), Hq, Hkv, hd, pool, table, 0, cd, sd, 0)
    out = sb.op_prompt_attention(_dev(T, qkv[n_ctx:]), Hq, Hkv, hd, pool, table, 0, cd, sd, n_ctx).cpu().numpy()
    raw = pool.view(T.int16).cpu().numpy().view(np.uint16).reshape(2, n_pages, Hkv, 16 * hd)
    tbl = table.cpu().numpy()
    for h in (0, 13, 31):
        Kc = np.stack([raw[0, tbl[t // 16], h].reshape(16, hd)[t % 16] for t in range(n_tot)])
        Vc = np.stack([raw[1, tbl[t // 16], h].reshape(hd, 16)[:, t % 16] for t in range(n_tot)])
        Ko = np.stack([si.round_to_bf16(orc.rope_apply(qkv[t, (Hq + h) * hd:(Hq + h + 1) * hd], t, base).astype(np.float32))
                       for t in range(n_tot)])
        Vo = si.round_to_bf16(np.ascontiguousarray(qkv[:, (Hq + Hkv + h) * hd:(Hq + Hkv + h + 1) * hd]))
        assert np.array_equal(Vc, Vo)
        _check_rotated_k_cache(Kc, Ko)
        K, V = si.bf16_to_f32(Kc), si.bf16_to_f32(Vc)
        for r in (0, 1, 31, 32, 63, 64, 127, 128, 129, 1000, 1023, 1024, M - 130, M - 2, M - 1):
            p_ = n_ctx + r
            q = orc.rope_apply(qkv[p_, h * hd:(h + 1) * hd], p_, base)
            ref = orc.attention_head(q, K[:p_ + 1], V[:p_ + 1])
            assert np.max(np.abs(out[r, h * hd:(h + 1) * hd] - ref)) <= 2e-5, (h, r)


@pytest.mark.parametrize("M", [1, 8])
def test_gemv_output_over_its_input(T, M):
    """y may be the memory of x (N == K): the same bits as with an output of its own."""
    import paper_2604_12247_amd as sb
    g = np.random.default_rng(31 + M)
    W = _dev(T, si.round_to_bf16((g.standard_normal((4096, 4096)) * 0.02).astype(np.float32)).view(np.int16))
    x = _dev(T, g.standard_normal((M, 4096)).astype(np.float32))
    P = sb.op_repack(W)
    ref = sb.op_gemv(P, x, sb.PROJ_MFMA_PACKED)
    scratch = T.empty(sb.lib().sb_op_gemv_scratch_bytes(M, 4096), dtype=T.uint8, device="cuda")
    rc = sb.lib().sb_op_gemv(P.data_ptr(), sb.BF16, 4096, 4096, x.data_ptr(), x.data_ptr(), M, sb.PROJ_MFMA_PACKED,
                             scratch.data_ptr(), T.cuda.current_stream().cuda_stream)
    assert rc == 0
    assert T.equal(x, ref)


@pytest.mark.parametrize("kernel", ["mfma", "mfma_packed"])
@pytest.mark.parametrize("entry", ["gemv", "gate_up", "head"])
@pytest.mark.parametrize("at", [0, 128, -128])   # the output begins with the input, inside it, before it
def test_projection_outputs_over_their_input(T, kernel, entry, at):
    """The outputs of every projection entry point (a head's logits among them) may lie over x: the same bits."""
    import paper_2604_12247_amd as sb
    L, n, M = sb.lib(), 1024, 5
    k = {"mfma": sb.PROJ_MFMA, "mfma_packed": sb.PROJ_MFMA_PACKED}[kernel]
    g = np.random.default_rng(37)
    W = _dev(T, _rand_w(g, 2 * n if entry == "gate_up" else n, n, True))
    W = sb.op_repack(W) if kernel == "mfma_packed" else W
    x0 = _dev(T, g.standard_normal((M, n)).astype(np.float32))
    buf = T.empty(M * n + 256, dtype=T.float32, device="cuda")
    x, y = buf[128:128 + M * n].view(M, n), buf[128 + at:128 + at + M * n].view(M, n)
    x.copy_(x0)
    st = T.cuda.current_stream().cuda_stream
    scratch = T.empty(max(L.sb_op_gemv_scratch_bytes(M, n), L.sb_op_head_scratch_bytes(M, n, n)), dtype=T.uint8, device="cuda")
    if entry == "head":
        am, cf, ref = sb.op_head(W, x0, 1.1, k, want_logits=True)
        am2, cf2 = T.empty_like(am), T.empty_like(cf)
        rc = L.sb_op_head(W.data_ptr(), sb.BF16, n, n, x.data_ptr(), M, 1.1, k, am2.data_ptr(), cf2.data_ptr(), y.data_ptr(), scratch.data_ptr(), st)
        assert rc == 0 and T.equal(am, am2) and T.equal(cf, cf2)
    else:
        ref = (sb.op_gemv if entry == "gemv" else sb.op_gate_up)(W, x0, k)
        call = L.sb_op_gemv if entry == "gemv" else L.sb_op_gate_up
        rc = call(W.data_ptr(), sb.BF16, n, n, x.data_ptr(), y.data_ptr(), M, k, scratch.data_ptr(), st)
        assert rc == 0
    assert T.equal(y, ref)


# launches between the two above: key tiles taken apart by the four waves of a block (257 blocks of 32 queries up to
# 319 of 128), with a prefix that ends inside a tile, fewer tiles than waves, a grouped-query shape whose
# blocks straddle rows; then the smallest launch of the wide form
@pytest.mark.parametrize("Hq,Hkv,hd,n_ctx,M", [(33, 33, 128, 0, 256), (40, 40, 64, 41, 213), (24, 8, 128, 70, 345), (32, 32, 64, 7, 1025),
                                               (32, 32, 128, 0, 1153)])
def test_prompt_attention_split_form(T, Hq, Hkv, hd, n_ctx, M):
    import paper_2604_12247_amd as sb
    base, G = 1e4, Hq // Hkv
    g = np.random.default_rng(1700 + hd + M)
    n_tot = n_ctx + M
    n_pages = (n_tot + 15) // 16 + 2
    qkv = (g.standard_normal((n_tot, (Hq + 2 * Hkv) * hd)) * 1.2).astype(np.float32)
    pool = T.empty(2 * n_pages * Hkv * 16 * hd * 2, dtype=T.uint8, device="cuda")
    pool.fill_(0xFF)
    table = _dev(T, g.permutation(n_pages).astype(np.int32))
    c, s = sb.rope_table(hd, base, n_pages * 16)
    cd, sd = _dev(T, c), _dev(T, s)
    if n_ctx:
        sb.op_prompt_attention(_dev(T, qkv[:n_ctx]), Hq, Hkv, hd, pool, table, 0, cd, sd, 0)
    out = sb.op_prompt_attention(_dev(T, qkv[n_ctx:]), Hq, Hkv, hd, pool, table, 0, cd, sd, n_ctx).cpu().numpy()
    raw = pool.view(T.int16).cpu().numpy().view(np.uint16).reshape(2, n_pages, Hkv, 16 * hd)
    tbl = table.cpu().numpy()
    for kvh in (0, Hkv - 1):
        K = si.bf16_to_f32(np.stack([raw[0, tbl[t // 16], kvh].reshape(16, hd)[t % 16] for t in range(n_tot)]))
        V = si.bf16_to_f32(np.stack([raw[1, tbl[t // 16], kvh].reshape(hd, 16)[:, t % 16] for t in range(n_tot)]))
        for r in sorted({0, 1, 10, 11, 31, 32, 127, 128, M // 2, M - 2, M - 1}):
            p_ = n_ctx + r
            for h in (kvh * G, kvh * G + G - 1):
                q = orc.rope_apply(qkv[p_, h * hd:(h + 1) * hd], p_, base)
                ref = orc.attention_head(q, K[:p_ + 1], V[:p_ + 1])
                assert np.max(np.abs(out[r, h * hd:(h + 1) * hd] - ref)) <= 2e-5, (h, r)


# one chunk (finished by the first stage, unless the output lies over the input), two chunks; grouped queries, whose output
# rows lie on other heads' keys; both caches
@pytest.mark.parametrize("Hq,Hkv,hd,bf16", [(32, 8, 128, True), (8, 8, 64, True), (32, 1, 128, True), (4, 4, 64, False), (16, 4, 128, False)])
@pytest.mark.parametrize("pos0", [0, 20, 56, 121])
def test_attention_output_over_its_input(T, Hq, Hkv, hd, bf16, pos0):
    """out may be the memory of qkv, from its start or from inside it: the same bits and the same cache as with an output of its own."""
    import paper_2604_12247_amd as sb
    kvd, M, n_pages = sb.BF16 if bf16 else sb.FP32, 7, 9
    g = np.random.default_rng(41 + Hq + pos0)
    c, s = sb.rope_table(hd, 1e4, n_pages * 16)
    cd, sd = _dev(T, c), _dev(T, s)
    table = _dev(T, g.permutation(n_pages).astype(np.int32))
    n = 2 * n_pages * Hkv * 16 * hd
    pool0 = _dev(T, g.standard_normal(n).astype(np.float32))
    pool0 = pool0.to(T.bfloat16) if bf16 else pool0
    qkv0 = _dev(T, g.standard_normal((M, (Hq + 2 * Hkv) * hd)).astype(np.float32))
    pool_ref = pool0.clone()
    ref = sb.op_attention(qkv0, Hq, Hkv, hd, kvd, pool_ref, table, 0, cd, sd, pos0)
    scratch = T.empty(sb.lib().sb_op_attention_scratch_bytes(Hq, hd, kvd, n_pages), dtype=T.uint8, device="cuda")
    for at in (0, hd, 2 * Hkv * hd):   # (the last: the end of out is the end of the first rows' keys and values)
        pool = pool0.clone()
        buf = T.empty(M * (Hq + 2 * Hkv) * hd + at, dtype=T.float32, device="cuda")
        qkv = buf[:qkv0.numel()].view_as(qkv0)
        qkv.copy_(qkv0)
        out = buf[at:at + M * Hq * hd].view(M, Hq * hd)
        rc = sb.lib().sb_op_attention(qkv.data_ptr(), Hq, Hkv, hd, kvd, pool.data_ptr(), table.data_ptr(), n_pages, 0, cd.data_ptr(),
                                      sd.data_ptr(), pos0, M, out.data_ptr(), scratch.data_ptr(), T.cuda.current_stream().cuda_stream)
        assert rc == 0
        assert T.equal(out, ref) and T.equal(pool.view(T.uint8), pool_ref.view(T.uint8)), at


# two launches of as many 128-row passes whose rows call for different numbers of blocks, at each form
@pytest.mark.parametrize("Hq,Hkv,hd,pos0,M,M2", [(40, 40, 64, 0, 190, 200), (16, 16, 64, 33, 390, 512), (32, 8, 128, 5, 1200, 1280),
                                                 (40, 40, 128, 0, 897, 1000)])
def test_prompt_attention_row_result_does_not_depend_on_the_rows_after_it(T, Hq, Hkv, hd, pos0, M, M2):
    import paper_2604_12247_amd as sb
    g = np.random.default_rng(59 + M)
    n_pages = (pos0 + M2 + 15) // 16
    c, s = sb.rope_table(hd, 1e4, n_pages * 16)
    cd, sd = _dev(T, c), _dev(T, s)
    table = _dev(T, g.permutation(n_pages).astype(np.int32))
    pool = _dev(T, g.standard_normal(2 * n_pages * Hkv * 16 * hd).astype(np.float32)).to(T.bfloat16)
    qkv = _dev(T, g.standard_normal((M2, (Hq + 2 * Hkv) * hd)).astype(np.float32))
    long = sb.op_prompt_attention(qkv, Hq, Hkv, hd, pool.clone(), table, 0, cd, sd, pos0)
    short = sb.op_prompt_attention(qkv[:M].contiguous(), Hq, Hkv, hd, pool.clone(), table, 0, cd, sd, pos0)
    assert T.equal(short, long[:M])


# one row, or one kv head whose rows fit one block of 64 queries: blocks of 32 would read queries that another has overwritten
@pytest.mark.parametrize("Hq,Hkv,hd,pos0,M", [(8, 8, 128, 70, 1), (64, 1, 128, 3, 1), (16, 1, 128, 40, 4), (32, 1, 64, 0, 2)])
def test_prompt_attention_output_over_its_input(T, Hq, Hkv, hd, pos0, M):
    import paper_2604_12247_amd as sb
    g = np.random.default_rng(61 + Hq + M)
    n_pages = (pos0 + M + 15) // 16
    c, s = sb.rope_table(hd, 1e4, n_pages * 16)
    cd, sd = _dev(T, c), _dev(T, s)
    table = _dev(T, g.permutation(n_pages).astype(np.int32))
    pool = _dev(T, g.standard_normal(2 * n_pages * Hkv * 16 * hd).astype(np.float32)).to(T.bfloat16)
    qkv = _dev(T, g.standard_normal((M, (Hq + 2 * Hkv) * hd)).astype(np.float32))
    ref = sb.op_prompt_attention(qkv, Hq, Hkv, hd, pool.clone(), table, 0, cd, sd, pos0)
    out = qkv.view(-1)[:M * Hq * hd].view(M, Hq * hd)
    rc = sb.lib().sb_op_prompt_attention(qkv.data_ptr(), Hq, Hkv, hd, pool.data_ptr(), table.data_ptr(), n_pages, 0, cd.data_ptr(),
                                         sd.data_ptr(), pos0, M, out.data_ptr(), T.cuda.current_stream().cuda_stream)
    assert rc == 0
    # another order of additions over <= 71 keys: fp32 sums and 16-bit pairs (2e-5 as everywhere)
    assert float((out - ref).abs().max()) <= 2e-5


# an fp32 cache, launches of 768 and 800, 1024 and 1056 blocks, where four to a CU are 1024 (a row alone and beside others may be on either side)
@pytest.mark.parametrize("hd,pos0", [(64, 3070), (64, 4095), (128, 1535), (128, 2047)])
def test_attention_fp32_cache_block_counts(T, hd, pos0):
    _, out6 = _attention_case(T, 32, 32, hd, False, pos0, 6, 1e4, True, seed=83 + pos0, oracle=False)
    for r in (0, 5):
        _, out1 = _attention_case(T, 32, 32, hd, False, pos0 + r, 1, 1e4, True, seed=83 + pos0, oracle=r == 5 and pos0 in (3070, 1535))
        assert np.array_equal(out1[0], out6[r]), r


@pytest.mark.parametrize("Hq,Hkv,hd,bf16", [(4, 4, 64, False), (2, 2, 128, False), (4, 2, 64, True), (4, 4, 128, True)])
def test_new_rows_at_every_place_of_a_chunk(T, Hq, Hkv, hd, bf16):
    """New rows on either side of half pages, pages, operand steps and chunks, from one to eight, as the chunk's first and last keys."""
    for pos0, M in ((0, 8), (7, 1), (8, 8), (13, 6), (15, 2), (31, 3), (57, 8), (63, 1), (64, 8), (95, 4), (120, 8), (121, 8), (127, 1), (128, 1)):
        worst, _ = _attention_case(T, Hq, Hkv, hd, bf16, pos0, M, 1e4, True, seed=pos0 * 9 + M)
        assert worst <= 2e-5, (pos0, M, worst)


@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("M", [1, 8])
def test_new_keys_bits(T, hd, bf16, M):
    """The last bit of an appended key is a property of its row and position, whatever form the kernel has."""
    import paper_2604_12247_amd as sb
    H, n_pages = 32, 64
    g = np.random.default_rng(67 + hd)
    c, s = sb.rope_table(hd, 1e4, n_pages * 16)
    for pos0 in (0, 121, 1000):
        pool = T.zeros(2 * n_pages * H * 16 * hd, dtype=T.bfloat16 if bf16 else T.float32, device="cuda")
        table = g.permutation(n_pages).astype(np.int32)
        qkv = g.standard_normal((M, 3 * H * hd)).astype(np.float32)
        sb.op_attention(_dev(T, qkv), H, H, hd, sb.BF16 if bf16 else sb.FP32, pool, _dev(T, table), 0, _dev(T, c), _dev(T, s), pos0)
        ref = _rotated(qkv[:, H * hd:2 * H * hd].reshape(M, H, hd), c[pos0:pos0 + M], s[pos0:pos0 + M])
        K = pool.float().cpu().numpy().reshape(2, n_pages, H, 16, hd)[0]
        K = np.stack([K[table[p // 16], :, p % 16] for p in range(pos0, pos0 + M)])
        assert np.array_equal(K, _bf16_value(ref) if bf16 else ref), pos0


# the three launches that take the key tiles apart
@pytest.mark.parametrize("H,hd", [(4, 64), (80, 64), (4, 128)])
def test_prompt_attention_query_parts(T, H, hd):
    """A query's low part is what its rounded value leaves over its high part.  Without rotation (cos 1, sin 0) two keys weigh one
    dim each by 1024, so that a last bit of a low part (2^-16 of a value near 1) is 2^-6 in the difference of the two scores."""
    import paper_2604_12247_amd as sb
    M, pos0, n_pages = 40, 2, 3
    g = np.random.default_rng(71 + hd)
    bf = _bf16_value
    c2 = np.float32(np.float32(1.4426950408889634) / np.sqrt(np.float32(hd)))
    x = g.uniform(5.5, 11, 400000).astype(np.float32)
    u = x * c2
    hi = bf(u)
    lo = bf(u - hi)
    at = np.flatnonzero(bf((np.longdouble(1) * x * c2 - hi).astype(np.float32)) != lo)   # where the unrounded product leaves another one
    assert len(at) >= 100
    a = at[np.arange(M * H) % len(at)].reshape(M, H)
    z = np.argsort(u)
    near = z[np.clip(np.searchsorted(u[z], u[a] + g.uniform(-1e-3, 1e-3, a.shape).astype(np.float32)), 0, len(z) - 1)]
    q = np.zeros((M, H, hd), np.float32)
    q[:, :, 0], q[:, :, 1] = x[a], x[near]
    pool = np.zeros((2, n_pages, H, 16 * hd), np.float32)
    pool[0].reshape(n_pages, H, 16, hd)[0, :, 0, 0] = 1024
    pool[0].reshape(n_pages, H, 16, hd)[0, :, 1, 1] = 1024
    pool[1].reshape(n_pages, H, hd, 16)[0, :, :, 0] = 1          # (values: transposed within a page; the other key's are 0)
    qkv = np.concatenate([q.reshape(M, -1), np.zeros((M, 2 * H * hd), np.float32)], 1)
    one, zero = np.ones((n_pages * 16, hd // 2), np.float32), np.zeros((n_pages * 16, hd // 2), np.float32)
    out = sb.op_prompt_attention(_dev(T, qkv), H, H, hd, _dev(T, pool).to(T.bfloat16), _dev(T, np.arange(n_pages, dtype=np.int32)), 0,
                                 _dev(T, one), _dev(T, zero), pos0).cpu().numpy().reshape(M, H, hd)

    def parts(i):
        return hi[i].astype(np.float64) + lo[i]

    ref = 1 / (1 + 2.0 ** (1024 * (parts(near) - parts(a))))     # (the other keys' scores are 1024 to 2048 lower)
    # scores near 2^11 as floats: 2^-13 of them, at most ln 2 / 4 of that in the result; probabilities as 16-bit pairs: 2^-17
    assert np.max(np.abs(out - ref[:, :, None])) <= 2 * 2.0 ** -13


# operands that wide loads may not read take the kernel's general form; new rows at every place of an eight-key operand and of a step, up to
# and across the end of a chunk, one to 64 queries per kv head
@pytest.mark.parametrize("Hq,Hkv,hd", [(4, 4, 128), (12, 4, 64), (8, 1, 128)])
@pytest.mark.parametrize("pos0", [0, 1, 6, 7, 8, 27, 121, 127, 128, 253])
def test_attention_unaligned_operands(T, Hq, Hkv, hd, pos0):
    import paper_2604_12247_amd as sb
    g = np.random.default_rng(Hq + hd + pos0)
    n_pages = (pos0 + 8 + 15) // 16
    c, s = sb.rope_table(hd, 1e4, n_pages * 16)
    table = _dev(T, g.permutation(n_pages).astype(np.int32))
    base = T.from_numpy(g.standard_normal((2 * n_pages * Hkv * 16, hd)).astype(np.float32)).cuda().to(T.bfloat16)

    def shifted(x):
        t = T.empty(x.size + 1, dtype=T.float32, device="cuda")[1:].view(x.shape)
        t.copy_(_dev(T, x))
        assert t.data_ptr() % 16 == 4
        return t

    for M in (1, 2, 5, 8):
        qkv = g.standard_normal((M, (Hq + 2 * Hkv) * hd)).astype(np.float32)
        got = []
        for put in (lambda x: _dev(T, x), shifted):
            pool = base.clone()
            out = sb.op_attention(put(qkv), Hq, Hkv, hd, sb.BF16, pool, table, 0, put(c), put(s), pos0)
            got.append((out.cpu().numpy(), pool.view(T.int16).cpu().numpy()))
        assert np.array_equal(got[0][1], got[1][1])                                  # what the cache holds, bit for bit
        assert np.max(np.abs(got[0][0] - got[1][0])) <= 4e-6, M                      # (float sums; a product may be fused in one form only)


# the fp32 cache's kernel in both forms: the same bits, with new rows in one page of a wave, in two, and across two waves and two chunks,
# first and last keys of a page, one to 32 queries per kv head (two groups), both chunk lengths
@pytest.mark.parametrize("Hq,Hkv,hd", [(4, 4, 64), (12, 4, 64), (8, 2, 128), (4, 1, 128)])
@pytest.mark.parametrize("pos0", [0, 9, 15, 16, 27, 31, 59, 64, 121, 127, 250])
def test_attention_fp32_unaligned_operands(T, Hq, Hkv, hd, pos0):
    import paper_2604_12247_amd as sb
    g = np.random.default_rng(Hq + hd + pos0)
    n_pages = (pos0 + 8 + 15) // 16
    c, s = sb.rope_table(hd, 1e4, n_pages * 16)
    table = _dev(T, g.permutation(n_pages).astype(np.int32))
    base = _dev(T, g.standard_normal((2 * n_pages * Hkv * 16, hd)).astype(np.float32))

    def shifted(x):
        t = T.empty(x.size + 1, dtype=T.float32, device="cuda")[1:].view(x.shape)
        t.copy_(_dev(T, x))
        return t

    for M in (1, 3, 8):
        qkv = g.standard_normal((M, (Hq + 2 * Hkv) * hd)).astype(np.float32)
        got = []
        for put in (lambda x: _dev(T, x), shifted):
            pool = base.clone()
            out = sb.op_attention(put(qkv), Hq, Hkv, hd, sb.FP32, pool, table, 0, put(c), put(s), pos0)
            got.append((out, pool))
        assert T.equal(got[0][0], got[1][0]) and T.equal(got[0][1], got[1][1]), M
        worst, _ = _attention_case(T, Hq, Hkv, hd, False, pos0, M, 1e4, True, seed=pos0 + M)
        assert worst <= 2e-5, M   # (as in test_new_rows_at_every_place_of_a_chunk)


def test_attention_row_result_does_not_depend_on_m(T):
    """The same position gives the same bits alone and inside a pass of 6 rows."""
    args = (8, 8, 128, True)
    _, out6 = _attention_case(T, *args, 250, 6, 1e4, True, seed=77)
    for r in (0, 3, 5):
        _, out1 = _attention_case(T, *args, 250 + r, 1, 1e4, True, seed=77)
        assert np.array_equal(out1[0], out6[r])
    # a pass whose rows straddle a chunk boundary (1024): the number of chunks a row sees is a
    # function of its own position, alone or beside rows that see one chunk less
    _, out6 = _attention_case(T, *args, 1021, 6, 1e4, True, seed=78)
    for r in (0, 2, 3, 5):
        _, out1 = _attention_case(T, *args, 1021 + r, 1, 1e4, True, seed=78)
        assert np.array_equal(out1[0], out6[r]), r
    # a pass of six rows with 32 kv heads x 25 chunks (more blocks than the chip holds at once) against
    # single rows with 24 and with 25 chunks
    args = (32, 32, 128, True)
    _, out6 = _attention_case(T, *args, 3070, 6, 1e4, True, seed=79, oracle=False)
    for r in (0, 1, 2, 5):
        _, out1 = _attention_case(T, *args, 3070 + r, 1, 1e4, True, seed=79, oracle=False)
        assert np.array_equal(out1[0], out6[r]), r

