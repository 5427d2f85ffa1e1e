"""GPU parity: the HIP path, called through the C ABI, against the CPU oracle.

Integer results (C_temp, S_B, column sums, flags, errCount) must match bit for bit.
The requantized uint8 output must equal the oracle's float32 evaluation exactly and
stay within one code of its float64 evaluation; the differing fraction is printed.
"""
import sys

import numpy as np
import pytest

from paper_2103_00130_amd import workloads as wlmod

pytestmark = pytest.mark.gpu


def say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def binding():
    import torch
    assert torch.cuda.is_available(), "these tests need the GPU"
    from paper_2103_00130_amd import binding as b   # raises if the HIP library is missing
    return b


@pytest.fixture(scope="module")
def gpu_util():
    import gpu_util
    return gpu_util


def operands(M, N, K, seed, relu_like=False, full_range_b=True):
    rng = np.random.Generator(np.random.PCG64(seed))
    A = wlmod.draw_a(rng, M, K, relu_like)
    B = rng.integers(-128, 128, size=(K, N), dtype=np.int8) if full_range_b else wlmod.draw_b(rng, K, N)
    return A, B


SHAPES = [(1, 1, 1), (3, 5, 7), (16, 48, 64), (64, 256, 512), (70, 300, 130), (129, 257, 65), (257, 513, 129),
          (300, 520, 200)]
TILE_VARIANTS = ["tile64", "tile128", "tile256", "auto"]


@pytest.mark.parametrize("transposed", [False, True])
@pytest.mark.parametrize("K,N", [(1, 1), (7, 5), (64, 256), (130, 300), (129, 513), (512, 256)])
def test_pack_checksum_and_colsum(binding, gpu_util, oracle, K, N, transposed):
    say(f"pack K={K} N={N} transposed={transposed}")
    _, B = operands(1, N, K, 100 + K + N)
    run = gpu_util.GpuRun(binding, B, transposed=transposed)
    assert np.array_equal(run.checksum(), oracle.b_checksum(B))
    assert np.array_equal(run.colsum(), oracle.b_colsum(B))
    assert binding.abft_packed_b_dims(run.Bp) == (K, N)


@pytest.mark.parametrize("variant", TILE_VARIANTS)
@pytest.mark.parametrize("M,N,K", SHAPES)
def test_checked_gemm_matches_oracle(binding, gpu_util, oracle, M, N, K, variant):
    say(f"gemm {M}x{N}x{K} variant={variant}")
    A, B = operands(M, N, K, 7 * M + 3 * N + K, relu_like=(M % 2 == 1))
    ref = oracle.checked_gemm(A, B)
    run = gpu_util.GpuRun(binding, B)
    out = run.gemm(A, variant=variant)
    assert np.array_equal(out["C"], ref.C)
    assert np.array_equal(out["flags"], ref.flags) and out["err_count"] == 0
    assert not out["ws"].any(), "workspace must be left zero"
    # same call without the check: same C, flags and count untouched
    out2 = run.gemm(A, variant=variant, check=False)
    assert np.array_equal(out2["C"], ref.C)
    assert (out2["flags"] == -1).all() and out2["err_count"] == -1


@pytest.mark.parametrize("variant", ["tile64", "tile256"])
def test_unaligned_and_strided_operands(binding, gpu_util, oracle, variant):
    import torch
    M, N, K = 37, 70, 83
    say(f"strided operands {M}x{N}x{K} variant={variant}")
    A, B = operands(M, N, K, 99)
    ref = oracle.checked_gemm(A, B)
    run = gpu_util.GpuRun(binding, B)
    # lda = K + 5 and a base pointer that is 1 byte off 16-byte alignment
    buf = torch.zeros(M * (K + 5) + 1, dtype=torch.uint8, device="cuda")
    A_dev = buf[1:1 + M * (K + 5)].view(M, K + 5)[:, :K]
    A_dev.copy_(gpu_util.dev(A))
    Cbuf = torch.full((M, N + 3), 55, dtype=torch.int32, device="cuda")
    C = Cbuf[:, :N]
    flags = torch.empty(M, dtype=torch.int32, device="cuda")
    cnt = torch.empty(1, dtype=torch.int32, device="cuda")
    ws = binding.Workspace(M, run.Bp)
    binding.abft_gemm_u8s8s32_checked(A_dev, run.Bp, C, flags, cnt, flags=gpu_util.VARIANTS[variant],
                                      workspace=ws.tensor)
    torch.cuda.synchronize()
    assert np.array_equal(C.cpu().numpy(), ref.C)
    assert (Cbuf[:, N:].cpu().numpy() == 55).all(), "columns past N must not be written"
    assert not flags.cpu().numpy().any() and int(cnt.item()) == 0


@pytest.mark.parametrize("variant", TILE_VARIANTS)
def test_c_flips_flag_exactly_their_rows(binding, gpu_util, oracle, variant):
    M, N, K = 150, 290, 140
    say(f"C flips {M}x{N}x{K} variant={variant}")
    A, B = operands(M, N, K, 5)
    run = gpu_util.GpuRun(binding, B)
    ws = binding.Workspace(M, run.Bp)
    rng = np.random.default_rng(3)
    for bit in list(range(32)) + [None]:
        if bit is None:   # several faults in one launch, two of them in the same row
            inj = [(3, 7, 1 << 31), (3, 200, 1 << 4), (149, 289, 1), (64, 128, 0x00F0F000)]
        else:
            inj = [(int(rng.integers(M)), int(rng.integers(N)), 1 << bit)]
        ref = oracle.checked_gemm(A, B, flips_c=inj)
        out = run.gemm(A, variant=variant, injections=inj, ws=ws)
        assert np.array_equal(out["C"], ref.C), f"bit {bit}"
        assert np.array_equal(out["flags"], ref.flags), f"bit {bit}"
        assert out["err_count"] == ref.err_count
        assert not out["ws"].any()
    # entries that name the same element compose (XOR of the masks), in either order, also to nothing
    for inj in ([(77, 100, 0x0000FF00), (5, 5, 2), (77, 100, 0x00F0F000)], [(20, 30, 0x80000001), (20, 30, 0x80000001)]):
        ref = oracle.checked_gemm(A, B, flips_c=inj)
        out = run.gemm(A, variant=variant, injections=inj, ws=ws)
        assert np.array_equal(out["C"], ref.C) and np.array_equal(out["flags"], ref.flags)
        assert out["err_count"] == ref.err_count and not out["ws"].any()
    # two flips in one row that cancel in the row sum (+2^5 and -2^5) are silent in both
    clean = oracle.gemm_u8s8s32(A, B)
    cols = [c for c in range(N) if not (clean[10, c] >> 5) & 1][:1] + [c for c in range(N) if (clean[10, c] >> 5) & 1][:1]
    inj = [(10, cols[0], 1 << 5), (10, cols[1], 1 << 5)]
    ref = oracle.checked_gemm(A, B, flips_c=inj)
    out = run.gemm(A, variant=variant, injections=inj, ws=ws)
    assert ref.err_count == 0 and out["err_count"] == 0 and np.array_equal(out["C"], ref.C)


@pytest.mark.parametrize("variant", ["tile64", "tile256"])
def test_b_and_a_flips(binding, gpu_util, oracle, variant):
    import torch
    M, N, K = 96, 300, 200
    say(f"A/B flips {M}x{N}x{K} variant={variant}")
    A, B = operands(M, N, K, 17, relu_like=True)
    run = gpu_util.GpuRun(binding, B)
    ws = binding.Workspace(M, run.Bp)
    rng = np.random.default_rng(8)
    for _ in range(12):
        k, j, bit = int(rng.integers(K)), int(rng.integers(N)), int(rng.integers(8))
        ref = oracle.checked_gemm(A, B, flips_b=[(k, j, bit)])
        binding.abft_packed_b_flip_bit(run.Bp, k, j, bit)
        out = run.gemm(A, variant=variant, ws=ws)
        binding.abft_packed_b_flip_bit(run.Bp, k, j, bit)
        assert np.array_equal(out["C"], ref.C) and np.array_equal(out["flags"], ref.flags)
        assert out["err_count"] == ref.err_count == int((A[:, k] != 0).sum())
    out = run.gemm(A, variant=variant, ws=ws)          # restored weight is clean again
    assert out["err_count"] == 0
    A_dev = gpu_util.dev(A)
    for _ in range(12):
        i, k, bit = int(rng.integers(M)), int(rng.integers(K)), int(rng.integers(8))
        ref = oracle.checked_gemm(A, B, flips_a=[(i, k, bit)])
        A_dev[i, k] ^= (1 << bit)
        out = run.gemm(A_dev, variant=variant, ws=ws)
        A_dev[i, k] ^= (1 << bit)
        assert np.array_equal(out["C"], ref.C)
        assert out["err_count"] == ref.err_count == 0
    torch.cuda.synchronize()


def test_checksum_entry_flip_flags_rows_it_touches(binding, gpu_util, oracle):
    # the paper assumes the encoded column error-free (Section IV-C); if S_B[k] is hit anyway,
    # row p differs by A[p][k] * (+-2^b) mod 2^32
    M, N, K = 80, 130, 70
    say("checksum entry flips")
    A, B = operands(M, N, K, 23, relu_like=True)
    run = gpu_util.GpuRun(binding, B)
    S = oracle.b_checksum(B)
    C = oracle.gemm_u8s8s32(A, B)
    rs = oracle.row_sums(C)
    for (k, bit) in [(0, 0), (5, 7), (69, 13), (33, 25), (12, 31)]:
        S2 = S.copy()
        S2.view(np.uint32)[k] ^= np.uint32(1 << bit)
        want, n = oracle.compare(rs, oracle.row_checksum(A, S2))
        binding.abft_packed_b_flip_checksum_bit(run.Bp, k, bit)
        out = run.gemm(A)
        assert np.array_equal(run.checksum(), S2)
        binding.abft_packed_b_flip_checksum_bit(run.Bp, k, bit)
        assert np.array_equal(out["flags"], want) and out["err_count"] == n
        assert np.array_equal(out["C"], C)
    assert np.array_equal(run.checksum(), S)
    assert run.gemm(A)["err_count"] == 0


@pytest.mark.parametrize("variant", ["tile64", "tile128", "tile256"])
@pytest.mark.parametrize("kind", ["tensor", "channel", "channel_bias"])
def test_requant_epilogue(binding, gpu_util, oracle, kind, variant):
    import torch
    M, N, K = 140, 270, 600
    say(f"requant {kind} variant={variant}")
    rng = np.random.default_rng(31)
    for zA, relu in ((128, False), (0, True), (17, False)):
        A, B = operands(M, N, K, 41 + zA, relu_like=relu, full_range_b=False)
        mult = wlmod.draw_mult(rng, N, "tensor" if kind == "tensor" else "channel")
        bias = rng.integers(-5000, 5000, size=N).astype(np.int32) if kind == "channel_bias" else None
        ref = oracle.checked_gemm(A, B)
        q32 = oracle.requantize(ref.C, ref.colsum, zA, 128, mult, bias, precision="f32")
        q64 = oracle.requantize(ref.C, ref.colsum, zA, 128, mult, bias, precision="f64")
        run = gpu_util.GpuRun(binding, B)
        both = run.gemm(A, variant=variant, requant=(zA, 128, mult, bias))
        only_q = run.gemm(A, variant=variant, requant=(zA, 128, mult, bias), want_c=False)
        assert np.array_equal(both["C"], ref.C) and both["err_count"] == 0 and only_q["err_count"] == 0
        for got in (both["Cq"], only_q["Cq"]):
            assert np.array_equal(got, q32)
            d = np.abs(got.astype(np.int32) - q64.astype(np.int32))
            assert d.max() <= 1
        say(f"  zA={zA}: fraction of codes differing from the float64 evaluation = {(both['Cq'] != q64).mean():.2e}")
        # stand-alone requantization of the stored C_temp
        mult_d = gpu_util.dev(np.atleast_1d(mult))
        bias_d = None if bias is None else gpu_util.dev(bias)
        rq = binding.make_requant(zA, 128, mult_d, bias_d)
        Cq = torch.zeros((M, N), dtype=torch.uint8, device="cuda")
        binding.abft_requantize_u8(gpu_util.dev(ref.C), run.Bp, rq, Cq)
        assert np.array_equal(Cq.cpu().numpy(), q32)
    # a fault in C_temp is flagged by the check and still requantized as it stands
    inj = [(9, 11, 1 << 30)]
    refi = oracle.checked_gemm(A, B, flips_c=inj)
    out = run.gemm(A, variant=variant, requant=(zA, 128, mult, bias), injections=inj)
    assert np.array_equal(out["flags"], refi.flags) and out["err_count"] == 1
    assert np.array_equal(out["Cq"], oracle.requantize(refi.C, refi.colsum, zA, 128, mult, bias, precision="f32"))


def test_verify_rows_and_row_checksum(binding, gpu_util, oracle):
    import torch
    M, N, K = 77, 301, 150
    say("verify_rows / row_checksum")
    A, B = operands(M, N, K, 61)
    ref = oracle.checked_gemm(A, B)
    run = gpu_util.GpuRun(binding, B)
    chk = torch.empty(M, dtype=torch.int32, device="cuda")
    binding.abft_row_checksum(gpu_util.dev(A), run.Bp, chk)
    assert np.array_equal(chk.cpu().numpy(), ref.chk)
    C_dev = gpu_util.dev(ref.C)
    flags = torch.empty(M, dtype=torch.int32, device="cuda")
    cnt = torch.empty(1, dtype=torch.int32, device="cuda")
    binding.abft_verify_rows(C_dev, chk, flags, cnt)
    assert not flags.cpu().numpy().any() and int(cnt.item()) == 0
    C_dev[5, 300] ^= (1 << 20)          # a stored intermediate picks up a flip after the GEMM
    C_dev[70, 0] ^= 1
    binding.abft_verify_rows(C_dev, chk, flags, cnt)
    want = np.zeros(M, np.int32)
    want[[5, 70]] = 1
    assert np.array_equal(flags.cpu().numpy(), want) and int(cnt.item()) == 2


@pytest.mark.parametrize("cfg", [0, 1, 2, 3, 4])
def test_paper_shaped_workloads_full_size(binding, gpu_util, oracle, cfg):
    """The five workloads at full size, in the launch configuration the benchmark times."""
    ops = wlmod.make_operands(cfg)
    wl = ops.wl
    say(f"workload {cfg}: {wl.name}")
    ref = oracle.checked_gemm(ops.A, ops.B)
    run = gpu_util.GpuRun(binding, ops.B)
    assert np.array_equal(run.checksum(), ref.S_B)
    assert np.array_equal(run.colsum(), ref.colsum)
    rq = None if ops.mult is None else (wl.zA, wl.zC, ops.mult, None)
    out = run.gemm(ops.A, requant=rq)
    assert np.array_equal(out["C"], ref.C)
    assert not out["flags"].any() and out["err_count"] == 0
    if rq is not None:
        q32 = oracle.requantize(ref.C, ref.colsum, wl.zA, wl.zC, ops.mult, precision="f32")
        q64 = oracle.requantize(ref.C, ref.colsum, wl.zA, wl.zC, ops.mult, precision="f64")
        assert np.array_equal(out["Cq"], q32)
        assert np.abs(out["Cq"].astype(np.int32) - q64.astype(np.int32)).max() <= 1
        say(f"  requantized codes differing from the float64 evaluation: {(out['Cq'] != q64).mean():.3e}")
    # one flip in C: exactly that row
    inj = [(wl.M - 1, wl.N - 1, 1 << 31)]
    out = run.gemm(ops.A, injections=inj)
    want = np.zeros(wl.M, np.int32)
    want[wl.M - 1] = 1
    assert np.array_equal(out["flags"], want) and out["err_count"] == 1
    assert out["C"][wl.M - 1, wl.N - 1] == np.int32(np.uint32(ref.C[wl.M - 1, wl.N - 1]) ^ np.uint32(1 << 31))
    # errCount as a counter that is added to, which is how the benchmark launches it
    acc = run.gemm(ops.A, requant=rq, accumulate_from=5)
    assert np.array_equal(acc["C"], ref.C) and not acc["flags"].any() and acc["err_count"] == 5
    if rq is not None:
        assert np.array_equal(acc["Cq"], q32)
    acc = run.gemm(ops.A, requant=rq, injections=inj, accumulate_from=5)
    assert np.array_equal(acc["flags"], want) and acc["err_count"] == 6


@pytest.mark.parametrize("M,N,K", [(300, 520, 1536), (16, 4096, 2048), (256, 512, 8192), (1040, 1100, 640), (46, 128, 13504), (64, 1345, 15376), (65, 5505, 4111)])
def test_graph_replays_match_oracle(binding, gpu_util, oracle, M, N, K):
    """Three checked launches captured in a graph (small tiles with row words, streaming kernel, 64x64 tiles, K split across
    workgroups on both tiles, a copy with padded rows ahead), replayed several times with eager work between the replays: every replay is compared with the
    oracle, clean and with a fault planted in the weight between two replays (the graph itself is unchanged)."""
    import torch
    say(f"graph replays {M}x{N}x{K}")
    b = binding
    A, B = operands(M, N, K, 13 * M + N + K, full_range_b=False)
    run = gpu_util.GpuRun(b, B)
    A_dev = gpu_util.dev(A)
    C = torch.empty((M, N), dtype=torch.int32, device="cuda")
    flags = torch.empty(M, dtype=torch.int32, device="cuda")
    cnt = torch.zeros(1, dtype=torch.int32, device="cuda")
    ws = b.Workspace(M, run.Bp)
    def launch():
        b.abft_gemm_u8s8s32_checked(A_dev, run.Bp, C, flags, cnt, flags=b.ABFT_CHECK | b.ABFT_ERRCOUNT_ACCUMULATE, workspace=ws.tensor)
    launch()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        for _ in range(3):
            launch()
    clean = oracle.checked_gemm(A, B)
    k, j, bit = K // 2 + 1, N // 3, 5
    hit = oracle.checked_gemm(A, B, flips_b=[(k, j, bit)])
    assert hit.err_count > 0
    for rep in range(4):
        faulty = rep in (1, 3)
        if faulty:
            b.abft_packed_b_flip_bit(run.Bp, k, j, bit)
        C.fill_(-3)
        flags.fill_(-3)
        cnt.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        want = hit if faulty else clean
        assert np.array_equal(C.cpu().numpy(), want.C), f"replay {rep}"
        assert np.array_equal(flags.cpu().numpy(), want.flags), f"replay {rep}"
        assert int(cnt.item()) == 3 * want.err_count, f"replay {rep}"
        if faulty:
            b.abft_packed_b_flip_bit(run.Bp, k, j, bit)
        # eager work between the replays: an unrelated checked launch through the same workspace
        launch()
        torch.cuda.synchronize()
        assert np.array_equal(C.cpu().numpy(), clean.C)


def test_deterministic_across_runs(binding, gpu_util):
    ops = wlmod.make_operands(3)
    say("determinism")
    run = gpu_util.GpuRun(binding, ops.B)
    a = run.gemm(ops.A)
    b = run.gemm(ops.A)
    assert np.array_equal(a["C"], b["C"]) and np.array_equal(a["flags"], b["flags"])


SMALLM_SHAPES = [(1, 16, 16), (1, 800, 3200), (5, 33, 80), (16, 48, 64), (16, 4096, 2048), (17, 100, 144),
                 (32, 512, 1024), (33, 70, 272), (64, 256, 512), (64, 1000, 1040),
                 # wide weights: a workgroup owns whole 32-column units (M <= 32, N >= 8192), ragged last unit
                 (16, 8192, 256), (9, 8217, 208), (32, 8240, 144), (17, 12000, 80),
                 # ... and two units (64 columns) from N = 16384 on (M <= 16)
                 (16, 16384, 128), (7, 16454, 80), (3, 16400, 2112)]


@pytest.mark.parametrize("M,N,K", SMALLM_SHAPES)
def test_streaming_kernel_matches_oracle(binding, gpu_util, oracle, M, N, K):
    say(f"streaming gemm {M}x{N}x{K}")
    A, B = operands(M, N, K, 11 * M + 5 * N + K, relu_like=(M % 2 == 1))
    rng = np.random.default_rng(M + N + K)
    run = gpu_util.GpuRun(binding, B)
    ws = binding.Workspace(M, run.Bp)
    ref = oracle.checked_gemm(A, B)
    for variant in ("smallm", "auto"):
        out = run.gemm(A, variant=variant, ws=ws)
        assert np.array_equal(out["C"], ref.C)
        assert np.array_equal(out["flags"], ref.flags) and out["err_count"] == 0
        assert not out["ws"].any(), "workspace must be left zero"
    out = run.gemm(A, variant="smallm", check=False)
    assert np.array_equal(out["C"], ref.C) and (out["flags"] == -1).all()
    # faults in C: single, and several at once
    for n_f in (1, 1, 3):
        inj = [(int(rng.integers(M)), int(rng.integers(N)), 1 << int(rng.integers(32))) for _ in range(n_f)]
        refi = oracle.checked_gemm(A, B, flips_c=inj)
        out = run.gemm(A, variant="smallm", injections=inj, ws=ws)
        assert np.array_equal(out["C"], refi.C) and np.array_equal(out["flags"], refi.flags)
        assert out["err_count"] == refi.err_count and not out["ws"].any()
    # a fault in B after packing, and one in A
    k, j, bit = int(rng.integers(K)), int(rng.integers(N)), int(rng.integers(8))
    refb = oracle.checked_gemm(A, B, flips_b=[(k, j, bit)])
    binding.abft_packed_b_flip_bit(run.Bp, k, j, bit)
    out = run.gemm(A, variant="smallm", ws=ws)
    binding.abft_packed_b_flip_bit(run.Bp, k, j, bit)
    assert np.array_equal(out["C"], refb.C) and np.array_equal(out["flags"], refb.flags)
    i, k, bit = int(rng.integers(M)), int(rng.integers(K)), int(rng.integers(8))
    refa = oracle.checked_gemm(A, B, flips_a=[(i, k, bit)])
    A2 = A.copy()
    A2[i, k] ^= np.uint8(1 << bit)
    out = run.gemm(A2, variant="smallm", ws=ws)
    assert np.array_equal(out["C"], refa.C) and out["err_count"] == 0
    # fused requantization
    mult = wlmod.draw_mult(rng, N, "channel")
    bias = rng.integers(-3000, 3000, size=N).astype(np.int32)
    q32 = oracle.requantize(ref.C, ref.colsum, 128, 128, mult, bias, precision="f32")
    for want_c in (True, False):
        out = run.gemm(A, variant="smallm", requant=(128, 128, mult, bias), want_c=want_c, ws=ws)
        assert np.array_equal(out["Cq"], q32) and out["err_count"] == 0
        if want_c:
            assert np.array_equal(out["C"], ref.C)


def test_streaming_variant_refuses_what_it_cannot_run(binding, gpu_util):
    import torch
    A, B = operands(70, 64, 64, 3)
    run = gpu_util.GpuRun(binding, B)
    with pytest.raises(binding.AbftError) as ei:
        run.gemm(A, variant="smallm")
    assert ei.value.code == binding.ABFT_EUNSUPPORTED
    A, B = operands(8, 64, 72, 4)       # K not a multiple of 16: forced streaming variant is refused,
    run = gpu_util.GpuRun(binding, B)   # the default choice falls back to the general tiled kernel
    with pytest.raises(binding.AbftError):
        run.gemm(A, variant="smallm")
    assert run.gemm(A)["err_count"] == 0
    torch.cuda.synchronize()


@pytest.mark.gpu
def test_calibration_copy_is_a_copy(binding):
    import torch
    g = torch.Generator(device="cpu").manual_seed(7)
    src = torch.randint(-2**31, 2**31 - 1, ((1 << 20) + 12,), dtype=torch.int32, generator=g).cuda()
    dst = torch.zeros_like(src)
    binding.abft_calib_copy(src, dst)
    torch.cuda.synchronize()
    assert torch.equal(src, dst)


@pytest.mark.gpu
@pytest.mark.parametrize("variant", ["tile256w2x4", "tile256w4x2"])
def test_eight_wavefront_variants(binding, gpu_util, oracle, variant):
    M, N, K = 300, 520, 384
    say(f"8-wavefront variant {variant} {M}x{N}x{K}")
    A, B = operands(M, N, K, 41)
    run = gpu_util.GpuRun(binding, B)
    inj = [(299, 519, 1 << 30), (0, 0, 1), (131, 260, 0x00010000)]
    ref = oracle.checked_gemm(A, B, flips_c=inj)
    out = run.gemm(A, variant=variant, injections=inj)
    assert np.array_equal(out["C"], ref.C) and np.array_equal(out["flags"], ref.flags)
    assert out["err_count"] == ref.err_count == 3 and not out["ws"].any()
    mult = np.full(N, 3e-4, np.float32)
    clean = oracle.checked_gemm(A, B)
    out = run.gemm(A, variant=variant, requant=(128, 128, mult, None), want_c=False)
    want = oracle.requantize(clean.C, clean.colsum, 128, 128, mult, precision="f32")
    assert np.array_equal(out["Cq"], want) and out["err_count"] == 0


# ---- Algorithm 1 with its printed modulus (ABFT_MOD127) -----------------------------------

@pytest.mark.gpu
@pytest.mark.parametrize("variant", ["auto", "tile64", "tile128", "tile256"])
def test_mod127_matches_oracle(binding, gpu_util, oracle, variant):
    import torch
    M, N, K = 150, 290, 144            # the modulus is implemented on the aligned path: K a multiple of 16
    say(f"mod 127: {M}x{N}x{K} variant={variant}")
    A, B = operands(M, N, K, 17, relu_like=True)
    A[3, 9], A[40, 9], A[41, 9] = 127, 254, 0      # operands on which a B fault at k = 9 is invisible modulo 127
    run = gpu_util.GpuRun(binding, B)
    rs = torch.empty(K, dtype=torch.int32, device="cuda")
    binding.abft_packed_b_get_checksum_mod127(run.Bp, rs)
    assert np.array_equal(rs.cpu().numpy(), oracle.b_checksum_mod127(B).astype(np.int32))
    ws = binding.Workspace(M, run.Bp)
    C0, flags0, n0 = oracle.checked_gemm_mod127(A, B)
    out = run.gemm(A, variant=variant, mod127=True, ws=ws)
    assert n0 == 0 and out["err_count"] == 0 and not out["flags"].any()
    assert np.array_equal(out["C"], C0) and not out["ws"].any()
    # C faults: every bit of the 32 (127 does not divide 2^b), several per launch, composed masks
    rng = np.random.default_rng(5)
    for bit in list(range(32)) + [None]:
        inj = [(3, 7, 1 << 31), (3, 200, 1 << 4), (149, 289, 1), (64, 128, 0x00F0F000)] if bit is None else \
              [(int(rng.integers(M)), int(rng.integers(N)), 1 << bit)]
        Cw, fw, nw = oracle.checked_gemm_mod127(A, B, flips_c=inj)
        out = run.gemm(A, variant=variant, mod127=True, injections=inj, ws=ws)
        assert np.array_equal(out["C"], Cw) and np.array_equal(out["flags"], fw) and out["err_count"] == nw
        assert bit is None or nw == 1
    # a mask whose value change is a multiple of 127 is missed by both
    clean = oracle.gemm_u8s8s32(A, B)
    r, c = 20, 30
    for delta in (127, 254, 127 * 4096):
        mask = int(np.uint32(clean[r, c]) ^ np.uint32(np.int64(clean[r, c]) + delta))
        Cw, fw, nw = oracle.checked_gemm_mod127(A, B, flips_c=[(r, c, mask)])
        out = run.gemm(A, variant=variant, mod127=True, injections=[(r, c, mask)], ws=ws)
        assert nw == 0 and out["err_count"] == 0 and np.array_equal(out["C"], Cw)
    # B faults after the checksum was taken: flags follow the oracle row by row, misses included
    missed_rows = 0
    for (k, j, bit) in [(9, 11, 0), (9, 250, 7), (0, 0, 3), (139, 289, 6), (77, 128, 1)]:
        Cw, fw, nw = oracle.checked_gemm_mod127(A, B, flips_b=[(k, j, bit)])
        binding.abft_packed_b_flip_bit(run.Bp, k, j, bit)
        out = run.gemm(A, variant=variant, mod127=True, ws=ws)
        binding.abft_packed_b_flip_bit(run.Bp, k, j, bit)
        assert np.array_equal(out["C"], Cw) and np.array_equal(out["flags"], fw) and out["err_count"] == nw
        corrupted = (Cw != clean).any(axis=1)
        missed_rows += int((corrupted & (fw == 0)).sum())
    assert missed_rows >= 2, "rows with A = 127 or 254 at the faulty k are corrupted yet pass modulo 127"
    out = run.gemm(A, variant=variant, ws=ws)           # the exact check on the same workspace afterwards
    assert out["err_count"] == 0 and not out["ws"].any()


@pytest.mark.gpu
def test_mod127_full_size_and_refusals(binding, gpu_util, oracle):
    import torch
    ops = wlmod.make_operands(3)
    say("mod 127: workload 3 full size")
    run = gpu_util.GpuRun(binding, ops.B)
    inj = [(1000, 1000, 1 << 20), (5, 6, 0x7)]
    Cw, fw, nw = oracle.checked_gemm_mod127(ops.A, ops.B, flips_c=inj)
    out = run.gemm(ops.A, mod127=True, injections=inj)
    assert np.array_equal(out["C"], Cw) and np.array_equal(out["flags"], fw) and out["err_count"] == nw == 2
    # unaligned operands do not implement the modulus
    A, B = operands(16, 64, 64, 1)
    small = gpu_util.GpuRun(binding, B)
    out = small.gemm(A, mod127=True)
    assert out["err_count"] == 0 and np.array_equal(out["C"], oracle.gemm_u8s8s32(A, B))
    buf = torch.zeros(16 * 64 + 1, dtype=torch.uint8, device="cuda")
    with pytest.raises(binding.AbftError):
        small.gemm(buf[1:].view(16, 64), mod127=True)


# ---- recovery: recompute the flagged rows ---------------------------------------------------

@pytest.mark.gpu
def test_recompute_flagged_rows(binding, gpu_util, oracle):
    import torch
    b = binding
    M, N, K = 300, 520, 384
    say(f"recovery {M}x{N}x{K}")
    A, B = operands(M, N, K, 43)
    clean = oracle.checked_gemm(A, B)
    run = gpu_util.GpuRun(b, B)
    A_dev = gpu_util.dev(A)
    mult = gpu_util.dev(np.full(N, 2e-4, np.float32))
    rq = b.make_requant(128, 128, mult)
    want_q = oracle.requantize(clean.C, clean.colsum, 128, 128, np.full(N, 2e-4, np.float32), precision="f32")
    C = torch.empty((M, N), dtype=torch.int32, device="cuda")
    Cq = torch.empty((M, N), dtype=torch.uint8, device="cuda")
    flags = torch.empty(M, dtype=torch.int32, device="cuda")
    cnt = torch.empty(1, dtype=torch.int32, device="cuda")
    ws = b.Workspace(M, run.Bp)
    # transient faults in the 32-bit intermediate: five rows flagged, all five recovered
    inj = [(0, 0, 1 << 31), (17, 300, 1 << 3), (17, 301, 1 << 9), (128, 519, 0x00FF0000), (255, 256, 1), (299, 1, 1 << 20)]
    b.abft_gemm_u8s8s32_checked(A_dev, run.Bp, C, flags, cnt, rq=rq, Cq=Cq, inj=b.make_injections(inj), n_inj=len(inj),
                                workspace=ws.tensor)
    assert int(cnt.item()) == 5 and not np.array_equal(C.cpu().numpy(), clean.C)
    before, after = b.abft_recompute_flagged_rows(A_dev, run.Bp, C, flags, cnt, rq=rq, Cq=Cq, max_rows_per_pass=2)
    assert (before, after) == (5, 0) and int(cnt.item()) == 0 and not flags.any().item()
    assert np.array_equal(C.cpu().numpy(), clean.C) and np.array_equal(Cq.cpu().numpy(), want_q)
    before, after = b.abft_recompute_flagged_rows(A_dev, run.Bp, C, flags, cnt)       # nothing to do
    assert (before, after) == (0, 0) and np.array_equal(C.cpu().numpy(), clean.C)
    # a fault that sits in the weight is still there when the rows are recomputed: flags stay
    b.abft_packed_b_flip_bit(run.Bp, 100, 200, 6)
    bad = oracle.checked_gemm(A, B, flips_b=[(100, 200, 6)])
    b.abft_gemm_u8s8s32_checked(A_dev, run.Bp, C, flags, cnt, workspace=ws.tensor)
    assert np.array_equal(flags.cpu().numpy(), bad.flags) and bad.err_count > 200
    before, after = b.abft_recompute_flagged_rows(A_dev, run.Bp, C, flags, cnt, max_rows_per_pass=64)   # several passes
    assert before == after == bad.err_count == int(cnt.item())
    assert np.array_equal(flags.cpu().numpy(), bad.flags) and np.array_equal(C.cpu().numpy(), bad.C)
    b.abft_packed_b_flip_bit(run.Bp, 100, 200, 6)                     # repair the weight: now recovery succeeds
    before, after = b.abft_recompute_flagged_rows(A_dev, run.Bp, C, flags, cnt, max_rows_per_pass=64)
    assert (before, after) == (bad.err_count, 0) and np.array_equal(C.cpu().numpy(), clean.C)


@pytest.mark.gpu
def test_seeded_sweep_of_shapes_variants_and_faults(binding, gpu_util, oracle):
    """120 seeded cases: ragged and tiny shapes, every kernel family, aligned and unaligned K, clean and
    faulty runs, with and without requantization; everything compared with the oracle."""
    rng = np.random.default_rng(20210300130)
    n_cases = 120
    for case in range(n_cases):
        M = int(rng.choice([1, 2, 15, 16, 17, 33, 64, 65, 100, 129, 255, 256, 257, 300, 513]))
        N = int(rng.choice([1, 3, 16, 31, 32, 33, 64, 100, 128, 255, 256, 257, 300, 520]))
        K = int(rng.choice([16, 32, 48, 64, 80, 128, 144, 256, 272, 384, 1, 7, 63, 65, 130, 200]))
        variant = str(rng.choice(["auto", "tile64", "tile128", "tile256", "tile256w2x4", "tile256w4x2"] + (["smallm"] if M <= 64 else [])))
        aligned = K % 16 == 0
        if variant == "smallm" and not aligned:
            variant = "auto"
        mod127 = bool(aligned and variant != "smallm" and rng.random() < 0.25)
        n_inj = int(rng.choice([0, 0, 1, 3]))
        inj = [(int(rng.integers(M)), int(rng.integers(N)), int(rng.integers(1, 2**32))) for _ in range(n_inj)]
        with_q = bool(rng.random() < 0.3) and not mod127
        say(f"sweep {case}: {M}x{N}x{K} {variant} mod127={mod127} inj={n_inj} requant={with_q}")
        A, B = operands(M, N, K, 1000 + case, relu_like=bool(rng.random() < 0.3), full_range_b=bool(rng.random() < 0.3))
        run = gpu_util.GpuRun(binding, B)
        rq = None
        if with_q:
            mult = wlmod.draw_mult(rng, N, "channel")
            bias = rng.integers(-5000, 5000, size=N, dtype=np.int32)
            rq = (int(rng.choice([0, 128])), 128, mult, bias)
        out = run.gemm(A, variant=variant, injections=inj, requant=rq, mod127=mod127)
        if mod127:
            Cw, fw, nw = oracle.checked_gemm_mod127(A, B, flips_c=inj)
        else:
            ref = oracle.checked_gemm(A, B, flips_c=inj)
            Cw, fw, nw = ref.C, ref.flags, ref.err_count
        assert np.array_equal(out["C"], Cw), f"case {case}: C"
        assert np.array_equal(out["flags"], fw) and out["err_count"] == nw, f"case {case}: flags"
        assert not out["ws"].any(), f"case {case}: workspace not restored"
        if with_q:
            want = oracle.requantize(Cw, oracle.b_colsum(B), rq[0], rq[1], rq[2], bias=rq[3], precision="f32")
            assert np.array_equal(out["Cq"], want), f"case {case}: Cq"


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K", [(20000, 384, 160), (513, 9000, 272), (70000, 64, 64)])
def test_long_and_wide_ragged_shapes(binding, gpu_util, oracle, M, N, K):
    """Many tile rows or tile columns (several rounds of workgroups per compute unit, hundreds of
    arrivals per workspace word), ragged in both dimensions."""
    say(f"long/wide {M}x{N}x{K}")
    A, B = operands(M, N, K, M + N + K)
    inj = [(M - 1, N - 1, 1 << 31), (0, 0, 1), (M // 2, N // 2, 0x00100000)]
    ref = oracle.checked_gemm(A, B, flips_c=inj)
    run = gpu_util.GpuRun(binding, B)
    out = run.gemm(A, injections=inj)
    assert np.array_equal(out["C"], ref.C) and np.array_equal(out["flags"], ref.flags)
    assert out["err_count"] == ref.err_count == 3 and not out["ws"].any()


# (grids that do not fill the chip, on the tiles of gemm_tile_wk.h either way; 64x64 tiles with four stages in flight, in whole rounds of them and with
# one and three left over; 289 of them with two)
@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K", [(200, 300, 2304), (1000, 1000, 4096), (65, 64, 2048), (1000, 1000, 1024), (1000, 1000, 640), (1000, 990, 1408), (1040, 1088, 2064)])
@pytest.mark.parametrize("variant", ["auto", "tile64"])
def test_small_grid_long_k(binding, gpu_util, oracle, M, N, K, variant):
    """Grids of a few hundred tiles and several stages of K, with injections, in the exact check and modulo 127."""
    say(f"small grid, long K {M}x{N}x{K} {variant}")
    A, B = operands(M, N, K, 3 * M + N + K)
    inj = [(M - 1, N - 1, 1 << 30), (0, 0, 1), (M // 2, N // 3, 0x00020000)]
    ref = oracle.checked_gemm(A, B, flips_c=inj)
    run = gpu_util.GpuRun(binding, B)
    out = run.gemm(A, variant=variant, injections=inj)
    assert np.array_equal(out["C"], ref.C) and np.array_equal(out["flags"], ref.flags)
    assert out["err_count"] == ref.err_count == 3 and not out["ws"].any()
    clean = run.gemm(A, variant=variant)
    assert clean["err_count"] == 0 and not clean["flags"].any()
    C127, flags127, count127 = oracle.checked_gemm_mod127(A, B, flips_c=inj)
    out127 = run.gemm(A, variant=variant, injections=inj, mod127=True)
    assert np.array_equal(out127["C"], C127) and np.array_equal(out127["flags"], flags127) and out127["err_count"] == count127


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K", [(200, 130, 2000), (192, 64, 1792), (130, 200, 3008), (300, 520, 1536)])
def test_k_split_between_wavefronts(binding, gpu_util, oracle, M, N, K):
    """Few tiles and a K of twelve stages and more, in rounds among the wavefronts of a workgroup: a K that ends inside
    the last stage, tile columns whose checksum shares lie in every wavefront's stages, ragged M and N, injections, faults in
    the weight early and late in K, requantized output, and the check modulo 127."""
    say(f"K split {M}x{N}x{K}")
    A, B = operands(M, N, K, 7 * M + N + K, full_range_b=False)
    inj = [(M - 1, N - 1, 1 << 29), (0, 0, 1 << 3), (M // 2, N // 2, 0x00400000)]
    ref = oracle.checked_gemm(A, B, flips_c=inj)
    run = gpu_util.GpuRun(binding, B)
    out = run.gemm(A, variant="tile64", injections=inj)
    assert np.array_equal(out["C"], ref.C) and np.array_equal(out["flags"], ref.flags)
    assert out["err_count"] == ref.err_count == 3 and not out["ws"].any()
    auto = run.gemm(A)
    assert np.array_equal(auto["C"], oracle.checked_gemm(A, B).C) and auto["err_count"] == 0 and not auto["flags"].any()
    rng = np.random.default_rng(K)
    mult = wlmod.draw_mult(rng, N, "channel")
    bias = rng.integers(-5000, 5000, size=N).astype(np.int32)
    q = run.gemm(A, variant="tile64", requant=(128, 128, mult, bias), want_c=False)
    clean = oracle.checked_gemm(A, B)
    assert np.array_equal(q["Cq"], oracle.requantize(clean.C, clean.colsum, 128, 128, mult, bias, precision="f32"))
    assert q["err_count"] == 0
    C127, flags127, count127 = oracle.checked_gemm_mod127(A, B, flips_c=inj)
    out127 = run.gemm(A, variant="tile64", injections=inj, mod127=True)
    assert np.array_equal(out127["C"], C127) and np.array_equal(out127["flags"], flags127) and out127["err_count"] == count127
    for k, j, bit in ((5, N // 3, 6), (K - 3, N - 1, 2)):
        binding.abft_packed_b_flip_bit(run.Bp, k, j, bit)
        refb = oracle.checked_gemm(A, B, flips_b=[(k, j, bit)])
        outb = run.gemm(A, variant="tile64")
        assert np.array_equal(outb["C"], refb.C) and np.array_equal(outb["flags"], refb.flags) and outb["err_count"] == refb.err_count
        binding.abft_packed_b_flip_bit(run.Bp, k, j, bit)


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K", [(200, 130, 2064), (64, 64, 2048), (130, 200, 3008), (320, 1000, 4096), (1000, 1024, 2176), (70, 190, 4112),
                                   (1000, 1000, 1296), (1024, 1150, 1424)])
def test_small_grid_long_k_every_feature(binding, gpu_util, oracle, M, N, K):
    """Grids of up to 288 tiles of 64x64 with every feature, on gemm_tile_wk.h and, where its forms do not take the grid, on the
    64x64 tiles with four stages in flight (1000x1000x1296) and with two (1024x1150x1424): odd and even numbers of stages, a K that
    ends inside the last stage, shares of the checksum product of one and two stages and empty ones, ragged M and N, injections in
    every quadrant of a tile, faults in the weight early, late and in the middle of K and in the checksum column, both outputs with
    requantization, the unchecked launch, the check modulo 127."""
    say(f"small grid, long K, every feature {M}x{N}x{K}")
    A, B = operands(M, N, K, 11 * M + N + K, full_range_b=False)
    inj = [(M - 1, N - 1, 1 << 29), (0, 0, 1 << 3), (M // 2, N // 2, 0x00400000), (40, 10, 1 << 31), (5, 50, 1 << 12)]
    ref = oracle.checked_gemm(A, B, flips_c=inj)
    run = gpu_util.GpuRun(binding, B)
    out = run.gemm(A, variant="tile64", injections=inj)
    assert np.array_equal(out["C"], ref.C) and np.array_equal(out["flags"], ref.flags)
    assert out["err_count"] == ref.err_count == len(set(r for r, _, _ in inj)) and not out["ws"].any()
    auto = run.gemm(A)
    clean = oracle.checked_gemm(A, B)
    assert np.array_equal(auto["C"], clean.C) and auto["err_count"] == 0 and not auto["flags"].any()
    unchecked = run.gemm(A, variant="tile64", check=False)
    assert np.array_equal(unchecked["C"], clean.C)
    rng = np.random.default_rng(K)
    mult = wlmod.draw_mult(rng, N, "channel")
    bias = rng.integers(-5000, 5000, size=N).astype(np.int32)
    q = run.gemm(A, variant="tile64", requant=(128, 128, mult, bias))
    assert np.array_equal(q["C"], clean.C)
    assert np.array_equal(q["Cq"], oracle.requantize(clean.C, clean.colsum, 128, 128, mult, bias, precision="f32"))
    assert q["err_count"] == 0
    C127, flags127, count127 = oracle.checked_gemm_mod127(A, B, flips_c=inj)
    out127 = run.gemm(A, variant="tile64", injections=inj, mod127=True)
    assert np.array_equal(out127["C"], C127) and np.array_equal(out127["flags"], flags127) and out127["err_count"] == count127
    for k, j, bit in ((5, N // 3, 6), (K - 3, N - 1, 2), (K // 2 + 33, 0, 7)):
        binding.abft_packed_b_flip_bit(run.Bp, k, j, bit)
        refb = oracle.checked_gemm(A, B, flips_b=[(k, j, bit)])
        outb = run.gemm(A, variant="tile64")
        assert np.array_equal(outb["C"], refb.C) and np.array_equal(outb["flags"], refb.flags) and outb["err_count"] == refb.err_count
        binding.abft_packed_b_flip_bit(run.Bp, k, j, bit)
    # a fault in the checksum column itself: every row whose A entry at that k is not zero is flagged, C is clean
    k = K // 3
    S2 = oracle.b_checksum(B)
    S2.view(np.uint32)[k] ^= np.uint32(1 << 9)
    want, n = oracle.compare(oracle.row_sums(clean.C), oracle.row_checksum(A, S2))
    binding.abft_packed_b_flip_checksum_bit(run.Bp, k, 9)
    outc = run.gemm(A, variant="tile64")
    binding.abft_packed_b_flip_checksum_bit(run.Bp, k, 9)
    assert np.array_equal(outc["C"], clean.C) and np.array_equal(outc["flags"], want) and outc["err_count"] == n and n > 0


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K,variant", [(100, 64, 8320, "tile64"), (16450, 33, 4240, "tile64"), (300, 256, 12288, "tile256"), (130, 128, 4224, "tile128")])
def test_long_checksum_share(binding, gpu_util, oracle, M, N, K, variant):
    """One tile column and a long K: its share of the checksum product is longer than one lot of
    digits in LDS (32 stages of 128), so the digits are staged in several lots (64x64 tiles: from 257 of them on; fewer
    run on gemm_tile_wk.h, which fetches a stage's digits with it)."""
    say(f"long checksum share {M}x{N}x{K} {variant}")
    A, B = operands(M, N, K, 5 * M + N + K)
    inj = [(M - 1, N - 1, 1 << 31), (0, 0, 1 << 5)]
    ref = oracle.checked_gemm(A, B, flips_c=inj)
    run = gpu_util.GpuRun(binding, B)
    out = run.gemm(A, variant=variant, injections=inj)
    assert np.array_equal(out["C"], ref.C) and np.array_equal(out["flags"], ref.flags)
    assert out["err_count"] == ref.err_count == 2 and not out["ws"].any()
    assert run.gemm(A, variant=variant)["err_count"] == 0
    # a fault in the weight, late in K (second lot of digits): the rows it corrupts, as the oracle says
    k, j = K - 7, N // 2
    binding.abft_packed_b_flip_bit(run.Bp, k, j, 6)
    refb = oracle.checked_gemm(A, B, flips_b=[(k, j, 6)])
    outb = run.gemm(A, variant=variant)
    assert np.array_equal(outb["C"], refb.C) and np.array_equal(outb["flags"], refb.flags) and outb["err_count"] == refb.err_count


@pytest.mark.gpu
def test_output_beyond_4_gib(binding, gpu_util, oracle):
    """C of 40000 x 30000 int32 (4.8 GB): element offsets that do not fit 32 bits.  The rows the oracle
    recomputes are a sample (rows are independent in product and check); flags and count are complete."""
    import torch
    M, N, K = 40000, 30000, 32
    say(f"large output {M}x{N}x{K}")
    A, B = operands(M, N, K, 77)
    inj = [(M - 1, N - 1, 1 << 29), (12345, 6789, 1 << 3)]
    Bp = binding.abft_pack_b_checksum(gpu_util.dev(B))
    C = torch.empty((M, N), dtype=torch.int32, device="cuda")
    flags = torch.empty(M, dtype=torch.int32, device="cuda")
    cnt = torch.empty(1, dtype=torch.int32, device="cuda")
    ws = binding.Workspace(M, Bp)
    binding.abft_gemm_u8s8s32_checked(gpu_util.dev(A), Bp, C, flags, cnt, inj=binding.make_injections(inj), n_inj=2,
                                      workspace=ws.tensor)
    torch.cuda.synchronize()
    rows = np.unique(np.concatenate([[0, 1, 255, 256, 12345, M - 257, M - 2, M - 1],
                                     np.random.default_rng(5).integers(0, M, size=56)]))
    sub = {int(r): i for i, r in enumerate(rows)}
    ref = oracle.checked_gemm(A[rows], B, flips_c=[(sub[r], c, m) for (r, c, m) in inj])
    got = C[torch.from_numpy(rows).cuda()].cpu().numpy()
    assert np.array_equal(got, ref.C)
    f = flags.cpu().numpy()
    assert f.sum() == 2 and f[M - 1] == 1 and f[12345] == 1 and int(cnt.item()) == 2
    assert np.array_equal(f[rows], ref.flags) and not ws.tensor.any().item()
    del C
    Bp.destroy()


# ---- further cases ---------------------------------------------------------------------------

@pytest.mark.gpu
def test_standalone_requantize_beyond_65535_rows(binding, gpu_util, oracle):
    """More rows than the second grid dimension holds: the stand-alone requantization must equal the
    fused epilogue and the oracle on every row."""
    import torch
    M, N, K = 70000, 64, 64
    say(f"stand-alone requantization, {M} rows")
    A, B = operands(M, N, K, 404, full_range_b=False)
    mult = wlmod.draw_mult(np.random.default_rng(9), N, "channel")
    run = gpu_util.GpuRun(binding, B)
    out = run.gemm(A, requant=(128, 128, mult, None))
    ref = oracle.checked_gemm(A, B)
    q32 = oracle.requantize(ref.C, ref.colsum, 128, 128, mult, precision="f32")
    assert np.array_equal(out["C"], ref.C) and np.array_equal(out["Cq"], q32)
    mult_d = gpu_util.dev(mult)
    rq = binding.make_requant(128, 128, mult_d)
    Cq = torch.zeros((M, N), dtype=torch.uint8, device="cuda")
    binding.abft_requantize_u8(gpu_util.dev(ref.C), run.Bp, rq, Cq)
    assert np.array_equal(Cq.cpu().numpy(), q32)


@pytest.mark.gpu
@pytest.mark.parametrize("variant", ["auto", "tile64", "tile128", "tile256"])
def test_accumulator_entries_wrap_on_the_matrix_cores(binding, gpu_util, oracle, variant):
    """Constant operands that drive the matrix cores' 32-bit accumulators past 2^31: with a = 0 the
    shifted operand is -128 and b = -128 gives 16384 per k, 2.29e9 after K = 140032 (the true entry is 0);
    with a = 255, b = 127 both the accumulator (127 * 127 * K) and the true entry (255 * 127 * K) wrap.
    Equality with the oracle shows that the accumulation is modulo 2^32 and does not saturate."""
    M, N, K = 20, 24, 140032
    say(f"accumulator wrap: {M}x{N}x{K} variant={variant}")
    A = np.zeros((M, K), np.uint8)
    B = np.full((K, N), -128, np.int8)
    A[5:10] = 255
    B[:, 8:16] = 127
    A[10:15, ::2] = 1           # mixed rows: small entries next to wrapped ones
    A[15:] = 128                # shifted operand 0: accumulator stays 0, the add-back alone carries the entry
    ref = oracle.checked_gemm(A, B)
    assert ref.err_count == 0
    assert int(ref.C[5, 8]) != 255 * 127 * K and (255 * 127 * K - int(ref.C[5, 8])) % (1 << 32) == 0   # wrapped indeed
    run = gpu_util.GpuRun(binding, B)
    assert np.array_equal(run.checksum(), ref.S_B)
    out = run.gemm(A, variant=variant)
    assert np.array_equal(out["C"], ref.C)
    assert not out["flags"].any() and out["err_count"] == 0 and not out["ws"].any()
    inj = [(0, 0, 1 << 31), (7, 9, 1), (19, 23, 1 << 16)]
    refi = oracle.checked_gemm(A, B, flips_c=inj)
    out = run.gemm(A, variant=variant, injections=inj)
    assert np.array_equal(out["C"], refi.C) and np.array_equal(out["flags"], refi.flags) and out["err_count"] == 3


@pytest.mark.gpu
def test_mod127_rowsum_entry_flip(binding, gpu_util, oracle):
    """A fault in the stored 8-bit checksum entry itself (Section IV-C assumes there is none): flags follow
    the oracle row by row, and a second call of the hook restores the column."""
    import torch
    M, N, K = 150, 290, 144
    say("mod 127: checksum entry flips")
    A, B = operands(M, N, K, 19, relu_like=True)
    A[3, 9], A[40, 9] = 127, 254
    run = gpu_util.GpuRun(binding, B)
    rs0 = oracle.b_checksum_mod127(B).astype(np.int32)
    rs = torch.empty(K, dtype=torch.int32, device="cuda")
    hits = 0
    for (k, bit) in [(9, 0), (9, 7), (0, 3), (143, 6), (77, 5)]:
        Cw, fw, nw = oracle.checked_gemm_mod127(A, B, flips_rowsum=[(k, bit)])
        binding.abft_packed_b_flip_checksum_bit_mod127(run.Bp, k, bit)
        binding.abft_packed_b_get_checksum_mod127(run.Bp, rs)
        want_entry = np.array([rs0[k]], np.int32).astype(np.uint8) ^ np.uint8(1 << bit)
        assert int(rs.cpu().numpy()[k]) == int(want_entry.view(np.int8)[0])
        out = run.gemm(A, mod127=True)
        exact = run.gemm(A)                       # the int32 column is a different column: untouched
        binding.abft_packed_b_flip_checksum_bit_mod127(run.Bp, k, bit)
        assert np.array_equal(out["C"], Cw) and np.array_equal(out["flags"], fw) and out["err_count"] == nw
        assert exact["err_count"] == 0
        hits += nw
    assert hits > 0
    binding.abft_packed_b_get_checksum_mod127(run.Bp, rs)
    assert np.array_equal(rs.cpu().numpy(), rs0)
    assert run.gemm(A, mod127=True)["err_count"] == 0


@pytest.mark.gpu
def test_mod127_on_the_tall_skinny_workload(binding, gpu_util, oracle):
    """Algorithm 1 with its printed modulus on workload 2's shape (M = 16), through whichever kernel the
    library picks for it: clean, C faults, B faults including rows that pass modulo 127."""
    ops = wlmod.make_operands(2)
    A = ops.A.copy()
    A[3, 100], A[7, 100], A[9, 100] = 127, 254, 0
    say("mod 127: workload 2 shape")
    run = gpu_util.GpuRun(binding, ops.B)
    C0, f0, n0 = oracle.checked_gemm_mod127(A, ops.B)
    out = run.gemm(A, mod127=True)
    assert n0 == 0 and np.array_equal(out["C"], C0) and out["err_count"] == 0 and not out["flags"].any()
    for inj in ([(15, 4095, 1 << 31)], [(0, 0, 1), (8, 2000, 1 << 13)]):
        Cw, fw, nw = oracle.checked_gemm_mod127(A, ops.B, flips_c=inj)
        out = run.gemm(A, mod127=True, injections=inj)
        assert np.array_equal(out["C"], Cw) and np.array_equal(out["flags"], fw) and out["err_count"] == nw == len(inj)
    for (k, j, bit) in [(100, 17, 0), (100, 4000, 7), (2047, 4095, 5), (0, 0, 6)]:
        Cw, fw, nw = oracle.checked_gemm_mod127(A, ops.B, flips_b=[(k, j, bit)])
        binding.abft_packed_b_flip_bit(run.Bp, k, j, bit)
        out = run.gemm(A, mod127=True)
        binding.abft_packed_b_flip_bit(run.Bp, k, j, bit)
        assert np.array_equal(out["C"], Cw) and np.array_equal(out["flags"], fw) and out["err_count"] == nw
    assert not out["ws"].any()


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K,variant", [(300, 520, 200, "tile64"), (300, 520, 200, "tile128"), (300, 520, 256, "tile256"),
                                           (200, 300, 2304, "auto"), (16, 4096, 2048, "auto"), (40, 100, 144, "smallm"),
                                           (129, 257, 65, "auto"), (100, 64, 272, "tile64"), (13, 16, 64, "smallm")])
def test_errcount_as_a_counter_and_without_one(binding, gpu_util, oracle, M, N, K, variant):
    """ABFT_ERRCOUNT_ACCUMULATE: the flagged rows are added to the caller's counter (Algorithm 1's errCount++),
    a clean launch leaves it alone; err_count = NULL: flags only.  Every kernel family, including shapes with a
    single tile column / column block (whose rows are judged inside one workgroup)."""
    say(f"errCount modes: {M}x{N}x{K} variant={variant}")
    A, B = operands(M, N, K, 3 * M + N + K)
    run = gpu_util.GpuRun(binding, B)
    ws = binding.Workspace(M, run.Bp)
    inj = [(0, 0, 1 << 31), (M - 1, N - 1, 1), (M // 2, N // 3, 1 << 9), (M // 2, N // 2, 1 << 3)]
    ref = oracle.checked_gemm(A, B, flips_c=inj)
    clean = oracle.checked_gemm(A, B)
    out = run.gemm(A, variant=variant, ws=ws, accumulate_from=5)
    assert np.array_equal(out["C"], clean.C) and not out["flags"].any() and out["err_count"] == 5
    out = run.gemm(A, variant=variant, ws=ws, injections=inj, accumulate_from=5)
    assert np.array_equal(out["C"], ref.C) and np.array_equal(out["flags"], ref.flags)
    assert out["err_count"] == 5 + ref.err_count == 8
    out = run.gemm(A, variant=variant, ws=ws, injections=inj, want_count=False)
    assert np.array_equal(out["C"], ref.C) and np.array_equal(out["flags"], ref.flags) and out["err_count"] == -1
    out = run.gemm(A, variant=variant, ws=ws, injections=inj)        # the overwriting form on the same workspace
    assert np.array_equal(out["flags"], ref.flags) and out["err_count"] == 3 and not out["ws"].any()


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K", [(1, 800, 3200), (16, 48, 64), (17, 100, 144), (33, 70, 272), (64, 1000, 1040), (13, 16, 64),
                                   (12, 8230, 96), (5, 16420, 64)])
def test_mod127_on_the_streaming_kernel(binding, gpu_util, oracle, M, N, K):
    """Algorithm 1 as printed through the streaming kernel (Section VI-A-1 names m = 1 among its shapes):
    clean, every bit of a C element, value changes that are multiples of 127 (missed by both sides), B faults
    including operand values 127 and 254 at the faulty k, a fault in the 8-bit checksum entry."""
    say(f"mod 127, streaming kernel: {M}x{N}x{K}")
    A, B = operands(M, N, K, M + 3 * N + K, relu_like=(M % 2 == 0))
    k0 = K // 2
    A[0, k0] = 127
    if M > 2:
        A[1, k0], A[2, k0] = 254, 0
    run = gpu_util.GpuRun(binding, B)
    ws = binding.Workspace(M, run.Bp)
    C0, f0, n0 = oracle.checked_gemm_mod127(A, B)
    out = run.gemm(A, variant="smallm", mod127=True, ws=ws)
    assert n0 == 0 and np.array_equal(out["C"], C0) and out["err_count"] == 0 and not out["flags"].any() and not out["ws"].any()
    rng = np.random.default_rng(M * N)
    for bit in range(32):
        inj = [(int(rng.integers(M)), int(rng.integers(N)), 1 << bit)]
        Cw, fw, nw = oracle.checked_gemm_mod127(A, B, flips_c=inj)
        out = run.gemm(A, variant="smallm", mod127=True, injections=inj, ws=ws)
        assert np.array_equal(out["C"], Cw) and np.array_equal(out["flags"], fw) and out["err_count"] == nw == 1
    r, c = M - 1, N - 1
    for delta in (127, 254 * 4096):
        mask = int(np.uint32(C0[r, c]) ^ np.uint32(np.int64(C0[r, c]) + delta))
        Cw, fw, nw = oracle.checked_gemm_mod127(A, B, flips_c=[(r, c, mask)])
        out = run.gemm(A, variant="smallm", mod127=True, injections=[(r, c, mask)], ws=ws)
        assert nw == 0 and out["err_count"] == 0 and np.array_equal(out["C"], Cw)
    for (k, j, bit) in [(k0, 0, 0), (k0, N - 1, 7), (0, N // 2, 3), (K - 1, N - 1, 6)]:
        Cw, fw, nw = oracle.checked_gemm_mod127(A, B, flips_b=[(k, j, bit)])
        binding.abft_packed_b_flip_bit(run.Bp, k, j, bit)
        out = run.gemm(A, variant="smallm", mod127=True, ws=ws)
        binding.abft_packed_b_flip_bit(run.Bp, k, j, bit)
        assert np.array_equal(out["C"], Cw) and np.array_equal(out["flags"], fw) and out["err_count"] == nw
    Cw, fw, nw = oracle.checked_gemm_mod127(A, B, flips_rowsum=[(k0, 5)])
    binding.abft_packed_b_flip_checksum_bit_mod127(run.Bp, k0, 5)
    out = run.gemm(A, variant="smallm", mod127=True, ws=ws)
    binding.abft_packed_b_flip_checksum_bit_mod127(run.Bp, k0, 5)
    assert np.array_equal(out["flags"], fw) and out["err_count"] == nw
    out = run.gemm(A, variant="smallm", ws=ws)           # the exact check on the same workspace afterwards
    assert out["err_count"] == 0 and not out["ws"].any()


@pytest.mark.gpu
def test_recompute_flagged_rows_without_a_host_round_trip(binding, gpu_util, oracle):
    """abft_recompute_flagged_rows_async: the count of flagged rows stays on the device.  Transient faults are
    recovered bit for bit; more flagged rows than the pass holds leave the rest flagged; a fault that sits in
    the weight stays flagged."""
    import torch
    b = binding
    M, N, K = 300, 520, 384
    say(f"recovery without synchronisation {M}x{N}x{K}")
    A, B = operands(M, N, K, 47)
    clean = oracle.checked_gemm(A, B)
    run = gpu_util.GpuRun(b, B)
    A_dev = gpu_util.dev(A)
    mult_np = wlmod.draw_mult(np.random.default_rng(4), N, "channel")
    mult = gpu_util.dev(mult_np)
    rq = b.make_requant(128, 128, mult)
    want_q = oracle.requantize(clean.C, clean.colsum, 128, 128, mult_np, precision="f32")
    C = torch.empty((M, N), dtype=torch.int32, device="cuda")
    Cq = torch.empty((M, N), dtype=torch.uint8, device="cuda")
    flags = torch.empty(M, dtype=torch.int32, device="cuda")
    cnt = torch.empty(1, dtype=torch.int32, device="cuda")
    ws = b.Workspace(M, run.Bp)
    inj = [(0, 0, 1 << 31), (17, 300, 1 << 3), (128, 519, 0x00FF0000), (255, 256, 1), (299, 1, 1 << 20)]
    for max_rows in (64, 5, 16):
        b.abft_gemm_u8s8s32_checked(A_dev, run.Bp, C, flags, cnt, rq=rq, Cq=Cq, inj=b.make_injections(inj), n_inj=len(inj),
                                    workspace=ws.tensor)
        status = b.abft_recompute_flagged_rows_async(A_dev, run.Bp, C, flags, cnt, rq=rq, Cq=Cq, max_rows=max_rows)
        torch.cuda.synchronize()
        assert status.cpu().tolist() == [5, 0] and int(cnt.item()) == 0 and not flags.any().item()
        assert np.array_equal(C.cpu().numpy(), clean.C) and np.array_equal(Cq.cpu().numpy(), want_q)
    # nothing flagged: nothing changes
    status = b.abft_recompute_flagged_rows_async(A_dev, run.Bp, C, flags, cnt, rq=rq, Cq=Cq)
    torch.cuda.synchronize()
    assert status.cpu().tolist() == [0, 0] and np.array_equal(C.cpu().numpy(), clean.C)
    # a pass of three rows against five flagged ones: three are recovered, two keep their flag
    b.abft_gemm_u8s8s32_checked(A_dev, run.Bp, C, flags, cnt, rq=rq, Cq=Cq, inj=b.make_injections(inj), n_inj=len(inj),
                                workspace=ws.tensor)
    status = b.abft_recompute_flagged_rows_async(A_dev, run.Bp, C, flags, cnt, rq=rq, Cq=Cq, max_rows=3)
    torch.cuda.synchronize()
    f = flags.cpu().numpy()
    assert status.cpu().tolist() == [5, 2] and int(cnt.item()) == 2 and int(f.sum()) == 2
    Cn = C.cpu().numpy()
    for r in (0, 17, 128, 255, 299):
        assert np.array_equal(Cn[r], clean.C[r]) == (f[r] == 0)
    status = b.abft_recompute_flagged_rows_async(A_dev, run.Bp, C, flags, cnt, rq=rq, Cq=Cq, max_rows=3)
    torch.cuda.synchronize()
    assert status.cpu().tolist() == [2, 0] and np.array_equal(C.cpu().numpy(), clean.C) and np.array_equal(Cq.cpu().numpy(), want_q)
    # a fault in the weight persists through the recomputation
    A1 = A.copy()
    A1[:, 100] = 0
    A1[[5, 9], 100] = 3
    A1_dev = gpu_util.dev(A1)
    bad = oracle.checked_gemm(A1, B, flips_b=[(100, 200, 6)])
    b.abft_packed_b_flip_bit(run.Bp, 100, 200, 6)
    b.abft_gemm_u8s8s32_checked(A1_dev, run.Bp, C, flags, cnt, workspace=ws.tensor)
    status = b.abft_recompute_flagged_rows_async(A1_dev, run.Bp, C, flags, cnt)
    torch.cuda.synchronize()
    assert bad.err_count == 2 and status.cpu().tolist() == [2, 2] and int(cnt.item()) == 2
    assert np.array_equal(flags.cpu().numpy(), bad.flags) and np.array_equal(C.cpu().numpy(), bad.C)
    b.abft_packed_b_flip_bit(run.Bp, 100, 200, 6)


# (32x32 tiles in two, three, four, seven, eight and sixteen slices, rows of whole chunks and of any length; 64x64 tiles in three, eight and
# eleven; shapes next to them that run unsplit)
@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K,split", [(65, 64, 3072, True), (65, 64, 6144, True), (46, 128, 13504, True), (100, 500, 8208, True), (128, 128, 16384, True), (40, 32, 32000, True),
                                         (45, 1000, 5001, True), (32, 240, 12600, True), (64, 1100, 9008, True), (20, 2500, 9104, True), (250, 500, 9008, True), (33, 4161, 7712, True), (64, 1345, 15376, True), (49, 1345, 20496, True), (130, 1640, 11600, True),
                                         (256, 512, 8192, False), (200, 300, 5120, False), (130, 70, 5264, False), (100, 1000, 8192, False)])
def test_k_split_across_workgroups(binding, gpu_util, oracle, M, N, K, split):
    """Few tiles and a long K: the library splits K across workgroups, the slices of a tile meet through the
    workspace, and every slice contributes its share of the checksum product on its own.  Bit-exact against the
    oracle: clean, C faults in several tiles, B faults early and late in K (different slices), A faults, the
    requantization epilogue, the printed modulus, errCount as a counter - and the same shapes unsplit, which is
    what a workspace without room for the partial tiles gets."""
    import torch
    say(f"split-K across workgroups: {M}x{N}x{K}")
    A, B = operands(M, N, K, M + 2 * N + K, relu_like=(K % 256 == 0))
    run = gpu_util.GpuRun(binding, B)
    ws = binding.Workspace(M, run.Bp)
    scratch = gpu_util.WS_SCRATCH

    class SmallWs:
        tensor = torch.zeros(binding.lib.abft_gemm_workspace_bytes(M, None) // 4, dtype=torch.int32, device="cuda")
    ref = oracle.checked_gemm(A, B)
    for w in (ws, SmallWs):
        out = run.gemm(A, ws=w)
        assert np.array_equal(out["C"], ref.C) and not out["flags"].any() and out["err_count"] == 0
        assert not out["ws"].any(), "row words, counting words and tickets must be left zero"
        if w is ws:     # the parts of the slices stay behind in the scratch, in whose first ints nothing else lies
            assert ws.tensor[scratch:scratch + 1280].any().item() == split
        out = run.gemm(A, ws=w, check=False)
        assert np.array_equal(out["C"], ref.C) and not out["ws"].any()
    rng = np.random.default_rng(K + M)
    inj = [(0, 0, 1 << 31), (M - 1, N - 1, 1), (M // 2, N // 2, 1 << 17), (M // 2, N // 3, 1 << 5), (1, N - 1, 0xFFFF0000)]
    refi = oracle.checked_gemm(A, B, flips_c=inj)
    out = run.gemm(A, ws=ws, injections=inj)
    assert np.array_equal(out["C"], refi.C) and np.array_equal(out["flags"], refi.flags) and out["err_count"] == refi.err_count
    out = run.gemm(A, ws=ws, injections=inj, accumulate_from=2)
    assert np.array_equal(out["flags"], refi.flags) and out["err_count"] == 2 + refi.err_count
    for (k, j, bit) in [(0, 0, 7), (K - 1, N - 1, 0), (K // 2 + 3, N // 2, 6), (K // 4, 5, 3)]:
        refb = oracle.checked_gemm(A, B, flips_b=[(k, j, bit)])
        binding.abft_packed_b_flip_bit(run.Bp, k, j, bit)
        out = run.gemm(A, ws=ws)
        binding.abft_packed_b_flip_bit(run.Bp, k, j, bit)
        assert np.array_equal(out["C"], refb.C) and np.array_equal(out["flags"], refb.flags) and out["err_count"] == refb.err_count
    i, k, bit = int(rng.integers(M)), int(rng.integers(K)), int(rng.integers(8))
    refa = oracle.checked_gemm(A, B, flips_a=[(i, k, bit)])
    A2 = A.copy()
    A2[i, k] ^= np.uint8(1 << bit)
    out = run.gemm(A2, ws=ws)
    assert np.array_equal(out["C"], refa.C) and out["err_count"] == 0
    # a fault in the checksum column late in K: the slice that holds that stage's share shows it
    S2 = ref.S_B.copy()
    S2.view(np.uint32)[K - 2] ^= np.uint32(1 << 9)
    want, n = oracle.compare(ref.rsum, oracle.row_checksum(A, S2))
    binding.abft_packed_b_flip_checksum_bit(run.Bp, K - 2, 9)
    out = run.gemm(A, ws=ws)
    binding.abft_packed_b_flip_checksum_bit(run.Bp, K - 2, 9)
    assert np.array_equal(out["flags"], want) and out["err_count"] == n
    # requantization epilogue, with and without C
    mult = wlmod.draw_mult(rng, N, "channel")
    bias = rng.integers(-3000, 3000, size=N).astype(np.int32)
    q32 = oracle.requantize(ref.C, ref.colsum, 128, 128, mult, bias, precision="f32")
    for want_c in (True, False):
        out = run.gemm(A, ws=ws, requant=(128, 128, mult, bias), want_c=want_c)
        assert np.array_equal(out["Cq"], q32) and out["err_count"] == 0
    # Algorithm 1 with its printed modulus
    if K % 16 == 0 and K <= 65536:
        Cw, fw, nw = oracle.checked_gemm_mod127(A, B, flips_c=inj[:3])
        out = run.gemm(A, ws=ws, mod127=True, injections=inj[:3])
        assert np.array_equal(out["C"], Cw) and np.array_equal(out["flags"], fw) and out["err_count"] == nw
    out = run.gemm(A, ws=ws)
    assert out["err_count"] == 0 and not out["ws"].any()


# (edges of the 16-byte chunk, of the 128-wide stage, of one and of several stages; streaming kernel, 64x64 kernel with loads
# through registers, copy with padded rows - with a K split behind it too - and each of them where a smaller workspace has
# no room for the copy)
@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K", [(5, 40, 3), (70, 70, 15), (2000, 1500, 13), (7, 100, 17), (33, 8200, 63), (64, 1100, 4001), (130, 70, 31), (65, 129, 127),
                                   (100, 65, 129), (128, 64, 255), (129, 200, 257), (64, 64, 385), (200, 130, 2687), (70, 200, 5121),
                                   (1000, 1300, 1249), (1, 300, 2001), (8, 700, 1999), (1, 4203, 6205), (7, 4999, 1021), (65, 5505, 4111)])
def test_rows_that_are_no_whole_chunks(binding, gpu_util, oracle, M, N, K):
    """A whose rows start and end at any byte: clean, with C and B faults, requantized, contiguous and as a view one byte
    into rows that are longer; nothing past the operand may count."""
    import torch
    say(f"rows of {K} bytes: {M}x{N}")
    A, B = operands(M, N, K, M + N + K)
    ref = oracle.checked_gemm(A, B)
    run = gpu_util.GpuRun(binding, B)
    inj = [(M - 1, N - 1, 1 << 31), (M // 2, N // 2, 1 << 3)]
    refi = oracle.checked_gemm(A, B, flips_c=inj)
    flip = (K - 1, N // 2, 6)
    refb = oracle.checked_gemm(A, B, flips_b=[flip])
    base_ints = 64 + max(2 * ((M + 63) // 64 * 64), 2 * (32 * 64 + 64))

    class SmallWs:
        tensor = torch.zeros(base_ints, dtype=torch.int32, device="cuda")
    buf = torch.full((M * (K + 6) + 1,), 255, dtype=torch.uint8, device="cuda")
    view = buf[1:].view(M, K + 6)[:, :K]
    view.copy_(gpu_util.dev(A))
    for ws in (None, SmallWs):
        for operand in (A, view):
            out = run.gemm(operand, ws=ws)
            assert np.array_equal(out["C"], ref.C) and not out["flags"].any() and out["err_count"] == 0 and not out["ws"].any()
        out = run.gemm(view, ws=ws, injections=inj, accumulate_from=1)
        assert np.array_equal(out["C"], refi.C) and np.array_equal(out["flags"], refi.flags) and out["err_count"] == 1 + refi.err_count
        binding.abft_packed_b_flip_bit(run.Bp, *flip)
        out = run.gemm(A, ws=ws)
        assert np.array_equal(out["C"], refb.C) and np.array_equal(out["flags"], refb.flags)
        assert np.array_equal(run.gemm(view, ws=ws, check=False)["C"], refb.C)
        binding.abft_packed_b_flip_bit(run.Bp, *flip)
        mult = wlmod.draw_mult(np.random.default_rng(K), N, "channel")
        out = run.gemm(A, ws=ws, requant=(128, 128, mult, None), want_c=False)
        assert np.array_equal(out["Cq"], oracle.requantize(ref.C, ref.colsum, 128, 128, mult, precision="f32"))


# (one and several tile columns; two to sixteen slices)
@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K", [(65, 64, 3001), (64, 32, 32001), (129, 40, 9001), (64, 64, 16383), (256, 200, 9001), (512, 100, 9001),
                                   (64, 4161, 7690)])
def test_padded_copy_and_k_split_in_one_call(binding, gpu_util, oracle, M, N, K):
    """64x64 tiles asked for, rows that are no whole chunks, few tiles and a long K: the rows are copied into the workspace and K is
    split across workgroups, whose parts go there too, beside the copy.  One workspace for all calls, tickets left zero."""
    import torch
    say(f"copy and K split: {M}x{N}x{K}")
    A, B = operands(M, N, K, M + N + K)
    run = gpu_util.GpuRun(binding, B)
    ws = binding.Workspace(M, run.Bp)
    scratch = gpu_util.WS_SCRATCH
    clean = oracle.checked_gemm(A, B)
    inj = [(M - 1, N - 1, 1 << 31), (M // 2, N // 3, 1 << 7)]
    refi = oracle.checked_gemm(A, B, flips_c=inj)
    flip = (K - 1, N // 2, 6)
    refb = oracle.checked_gemm(A, B, flips_b=[flip])
    for _ in range(4):
        ws.tensor[scratch:].zero_()
        out = run.gemm(A, variant="tile64", ws=ws)
        assert np.array_equal(out["C"], clean.C) and not out["flags"].any() and out["err_count"] == 0
        assert not out["ws"].any() and ws.tensor[scratch:scratch + 1280].any(), "the parts of a split come first"
        assert np.array_equal(run.gemm(A, variant="tile64", ws=ws, check=False)["C"], clean.C)
        out = run.gemm(A, variant="tile64", ws=ws, injections=inj, accumulate_from=3)
        assert np.array_equal(out["C"], refi.C) and np.array_equal(out["flags"], refi.flags) and out["err_count"] == 3 + refi.err_count
    binding.abft_packed_b_flip_bit(run.Bp, *flip)
    out = run.gemm(A, variant="tile64", ws=ws)
    assert np.array_equal(out["C"], refb.C) and np.array_equal(out["flags"], refb.flags) and out["err_count"] == refb.err_count
    assert not out["ws"].any()


@pytest.mark.gpu
def test_one_workspace_for_calls_of_different_sizes(binding, gpu_util, oracle):
    """A K split's partial tiles and a padded copy of A are left behind in the workspace: the next call, of other sizes and
    with words of its own where a smaller call's scratch could lie, starts from zeros all the same."""
    import torch
    shapes = [(128, 128, 16384), (5000, 96, 64), (300, 520, 1999), (5000, 96, 64), (256, 512, 8192), (16, 700, 320)]
    runs, need = [], 0
    for M, N, K in shapes:
        A, B = operands(M, N, K, M + K)
        run = gpu_util.GpuRun(binding, B)
        need = max(need, binding.abft_gemm_workspace_bytes(M, run.Bp) // 4)
        runs.append((A, oracle.checked_gemm(A, B, flips_c=[(M - 1, 1, 1 << 20)]), run))

    class Shared:
        tensor = torch.zeros(need, dtype=torch.int32, device="cuda")
    for A, ref, run in runs:
        out = run.gemm(A, ws=Shared, injections=[(A.shape[0] - 1, 1, 1 << 20)])
        assert np.array_equal(out["C"], ref.C) and np.array_equal(out["flags"], ref.flags) and out["err_count"] == 1


@pytest.mark.gpu
def test_many_rows_after_calls_that_left_scratch(binding, gpu_util, oracle):
    """Row words beyond 131072 rows lie where a K split's partial tiles and a padded copy of A are left: a call of that many
    rows starts from zeros all the same, overwriting and adding to errCount, and leaves zeros."""
    import torch
    M, N, K = 150000, 258, 32
    A, B = operands(M, N, K, 5)
    inj = [(M - 1, 1, 1 << 20), (131600, N - 1, 1 << 3), (7, 0, 1 << 31)]
    ref, refi = oracle.checked_gemm(A, B), oracle.checked_gemm(A, B, flips_c=inj)
    run, A_dev = gpu_util.GpuRun(binding, B), gpu_util.dev(A)

    class Shared:
        tensor = torch.zeros(400064, dtype=torch.int32, device="cuda")   # what 200000 rows need without a weight
    for m, n, k in ((128, 64, 3072), (500, 4160, 1001)):
        a, b = operands(m, n, k, m)
        small = gpu_util.GpuRun(binding, b)
        want = oracle.checked_gemm(a, b)
        out = small.gemm(a, ws=Shared)
        assert np.array_equal(out["C"], want.C) and not out["flags"].any() and out["err_count"] == 0
        assert Shared.tensor[gpu_util.WS_SCRATCH:].any(), "the call left no scratch: this test has lost its point"
        out = run.gemm(A_dev, ws=Shared)
        assert np.array_equal(out["C"], ref.C) and not out["flags"].any() and out["err_count"] == 0
        assert not Shared.tensor[:64 + 2 * M].any()
        out = small.gemm(a, ws=Shared)
        out = run.gemm(A_dev, ws=Shared, injections=inj, accumulate_from=4)
        assert np.array_equal(out["flags"], refi.flags) and out["err_count"] == 4 + refi.err_count


# (edges of the 16-byte chunk, of the 128 x 256 tile that a workgroup packs, rows shorter than a chunk)
@pytest.mark.gpu
@pytest.mark.parametrize("transposed", [False, True])
@pytest.mark.parametrize("K,N", [(3, 300), (300, 3), (15, 17), (17, 255), (127, 256), (128, 257), (129, 15), (385, 530), (1000, 16)])
def test_pack_of_strided_weights(binding, gpu_util, oracle, K, N, transposed):
    """A weight that lies one byte into longer rows, either way round: its sums, its residues modulo 127, and the product
    with it (every packed byte, the digits and their total take part in that)."""
    import torch
    A, B = operands(70, N, K, K * N)
    src = B.T if transposed else B
    rows, cols = src.shape
    buf = torch.full((rows * (cols + 5) + 1,), 77, dtype=torch.int8, device="cuda")
    view = buf[1:].view(rows, cols + 5)[:, :cols]
    view.copy_(gpu_util.dev(src))
    run = gpu_util.GpuRun(binding, B)
    run.Bp = binding.abft_pack_b_checksum(view, b_is_transposed=transposed)
    S_B = oracle.b_checksum(B)
    assert np.array_equal(run.checksum(), S_B) and np.array_equal(run.colsum(), oracle.b_colsum(B))
    r127 = torch.empty(K, dtype=torch.int32, device="cuda")
    binding.abft_packed_b_get_checksum_mod127(run.Bp, r127)
    assert np.array_equal(r127.cpu().numpy(), S_B % 127)
    ref = oracle.checked_gemm(A, B)
    out = run.gemm(A)
    assert np.array_equal(out["C"], ref.C) and not out["flags"].any()
    if K % 16 == 0:
        out = run.gemm(A, mod127=True)
        assert np.array_equal(out["C"], ref.C) and not out["flags"].any()


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K,words_only", [(1, 800, 4095, True), (32, 300, 2049, True), (40, 1000, 3071, True), (48, 4096, 2048, True), (33, 8192, 4095, False),
                                              (41, 1000, 3071, False), (64, 512, 4096, False)])
def test_workspace_holds_what_calls_use(binding, gpu_util, M, N, K, words_only):
    """Shapes that neither split K nor copy A are asked for the row and counting words alone, others for scratch as well; either way
    the call runs on what was asked for and leaves the words zero."""
    A, B = operands(M, N, K, M)
    run = gpu_util.GpuRun(binding, B)
    assert (binding.abft_gemm_workspace_bytes(M, run.Bp) == (64 + 2 * (32 * 64 + 64)) * 4) == words_only
    out = run.gemm(A)
    assert np.array_equal(out["C"], A.astype(np.int32) @ B.astype(np.int32)) and not out["flags"].any() and not out["ws"].any()


@pytest.mark.gpu
def test_refused_variant_enqueues_nothing(binding, gpu_util):
    """An unknown variant on rows that a copy would be made of: refused, and the workspace stays as it was."""
    import torch
    A, B = operands(500, 4160, 1001, 3)
    run = gpu_util.GpuRun(binding, B)
    ws = binding.Workspace(500, run.Bp).tensor
    C, flags = torch.zeros((500, 4160), dtype=torch.int32, device="cuda"), torch.zeros(500, dtype=torch.int32, device="cuda")
    with pytest.raises(binding.AbftError) as e:
        binding.abft_gemm_u8s8s32_checked(gpu_util.dev(A), run.Bp, C, flags, None, flags=0x700, workspace=ws)
    assert e.value.code == binding.ABFT_EINVAL
    torch.cuda.synchronize()
    assert ws.numel() > 263232 and not ws.any() and not C.any()


@pytest.mark.gpu
def test_operands_of_the_native_call(binding, gpu_util, oracle, monkeypatch):
    """The natively marshalled call takes what the Python code takes - views, single rows, an explicit stream, no errCount -
    and leaves to it, errors and all, what it does not: the native function says which (a return code, or None)."""
    import torch
    native, said = binding._fastcall.gemm, []

    def watched(*args):
        said.append(native(*args))
        return said[-1]
    monkeypatch.setattr(binding._fastcall, "gemm", watched)
    M, N, K = 70, 65, 130
    A, B = operands(M, N, K, 17)
    ref = oracle.checked_gemm(A, B)
    run = gpu_util.GpuRun(binding, B)
    ws = binding.Workspace(M, run.Bp).tensor
    wide = torch.zeros((M, K + 7), dtype=torch.uint8, device="cuda")
    wide[:, 3:3 + K] = gpu_util.dev(A)
    Cw = torch.zeros((M, N + 2), dtype=torch.int32, device="cuda")
    flags = torch.full((M + 4,), 9, dtype=torch.int32, device="cuda")
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    call = binding.abft_gemm_u8s8s32_checked
    call(wide[:, 3:3 + K], run.Bp, Cw[:, 1:1 + N], flags, None, workspace=ws, stream=side)
    with torch.cuda.stream(side):
        one = torch.zeros((1, N), dtype=torch.int32, device="cuda")
        call(wide[5:6, 3:3 + K], run.Bp, one, flags[M:], None, workspace=ws)
    side.synchronize()
    assert said == [binding.ABFT_OK] * 2
    assert np.array_equal(Cw[:, 1:1 + N].cpu().numpy(), ref.C) and not Cw[:, 0].any() and np.array_equal(one.cpu().numpy()[0], ref.C[5])
    assert flags.cpu().tolist() == [0] * (M + 1) + [9] * 3
    A_dev, C, cnt = gpu_util.dev(A), torch.zeros((M, N), dtype=torch.int32, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda")
    for bad, error in (((A_dev.cpu(), C, flags), TypeError), ((A_dev.int(), C, flags), TypeError), ((A_dev[:, :-1], C, flags), ValueError),
                       ((A_dev, C[:, :-1], flags), ValueError), ((A_dev, C, flags[:M - 1]), ValueError), ((A_dev, C.float(), flags), TypeError),
                       ((A_dev, None, flags), binding.AbftError), ((A_dev, C, None), binding.AbftError)):
        with pytest.raises(error):
            call(bad[0], run.Bp, bad[1], bad[2], cnt, workspace=ws)
        assert said.pop() == (binding.ABFT_EINVAL if error is binding.AbftError else None)
    with pytest.raises(ValueError):
        call(A_dev, run.Bp, C, flags, cnt, inj=torch.zeros(2, dtype=torch.int32, device="cuda"), n_inj=1, workspace=ws)
    assert said.pop() is None
    with pytest.raises(binding.AbftError) as e:
        call(A_dev, run.Bp, C, flags, cnt, workspace=ws[:64])
    assert e.value.code == binding.ABFT_EINVAL and "workspace" in str(e.value)
    assert said.pop() == binding.ABFT_EINVAL
    call(A_dev, run.Bp, C, flags, cnt, flags=np.int64(0), workspace=ws)     # (a number that is no plain int)
    assert said.pop() is None
    mult = torch.full((N,), 1e-3, device="cuda")
    Cq = torch.zeros((M, N), dtype=torch.uint8, device="cuda")
    call(A_dev, run.Bp, None, flags, cnt, rq=binding.make_requant(0, 0, mult), Cq=Cq, inj=binding.make_injections([(0, 0, 1)]), n_inj=1, workspace=ws)
    assert said.pop() == binding.ABFT_OK
    torch.cuda.synchronize()
    assert np.array_equal(C.cpu().numpy(), ref.C)


# (K slices across workgroups that are not all equally long: 24, 25, 41, 61, 105 and 161 stages in 4, 2 or 3, 8 and 16 slices;
# two K groups of unequal length inside a workgroup: 13 and 25 stages; three row blocks and 64 columns per workgroup on the
# streaming kernel)
@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K", [(100, 64, 3072), (100, 200, 3200), (700, 500, 5136), (130, 70, 7696), (61, 496, 13440), (65, 64, 20496),
                                   (700, 900, 1664), (500, 1300, 3200), (33, 1000, 1040), (48, 333, 2048), (40, 4096, 784), (20, 8250, 96),
                                   (32, 16390, 64), (9, 12330, 160), (64, 4200, 1024)])
def test_unequal_runs_and_wide_blocks(binding, gpu_util, oracle, M, N, K):
    """Bit for bit against the oracle: clean, faults in C, in B and in the checksum column, requantized, modulo 127."""
    say(f"unequal runs: {M}x{N}x{K}")
    A, B = operands(M, N, K, M + N + K)
    ref = oracle.checked_gemm(A, B)
    run = gpu_util.GpuRun(binding, B)
    ws = binding.Workspace(M, run.Bp)
    out = run.gemm(A, ws=ws)
    assert np.array_equal(out["C"], ref.C) and not out["flags"].any() and out["err_count"] == 0 and not out["ws"].any()
    assert np.array_equal(run.gemm(A, ws=ws, check=False)["C"], ref.C)
    inj = [(0, 0, 1 << 31), (M - 1, N - 1, 1), (M // 2, N // 3, 1 << 9), (M // 2, N // 2, 1 << 3)]
    refi = oracle.checked_gemm(A, B, flips_c=inj)
    out = run.gemm(A, ws=ws, injections=inj, accumulate_from=3)
    assert np.array_equal(out["C"], refi.C) and np.array_equal(out["flags"], refi.flags) and out["err_count"] == 3 + refi.err_count
    for (k, j, bit) in [(0, 0, 7), (K - 1, N - 1, 0), (K // 2 + 3, N // 2, 6)]:
        refb = oracle.checked_gemm(A, B, flips_b=[(k, j, bit)])
        binding.abft_packed_b_flip_bit(run.Bp, k, j, bit)
        out = run.gemm(A, ws=ws)
        binding.abft_packed_b_flip_bit(run.Bp, k, j, bit)
        assert np.array_equal(out["C"], refb.C) and np.array_equal(out["flags"], refb.flags) and out["err_count"] == refb.err_count
    for k in (1, K // 3, K - 2):     # a fault in the checksum column, in the share of different runs and tile columns
        S2 = ref.S_B.copy()
        S2.view(np.uint32)[k] ^= np.uint32(1 << 9)
        want, n = oracle.compare(ref.rsum, oracle.row_checksum(A, S2))
        binding.abft_packed_b_flip_checksum_bit(run.Bp, k, 9)
        out = run.gemm(A, ws=ws)
        binding.abft_packed_b_flip_checksum_bit(run.Bp, k, 9)
        assert np.array_equal(out["flags"], want) and out["err_count"] == n
    mult = wlmod.draw_mult(np.random.default_rng(K), N, "channel")
    out = run.gemm(A, ws=ws, requant=(128, 128, mult, None), want_c=False)
    assert np.array_equal(out["Cq"], oracle.requantize(ref.C, ref.colsum, 128, 128, mult, precision="f32"))
    Cw, fw, nw = oracle.checked_gemm_mod127(A, B, flips_c=inj[:3])
    out = run.gemm(A, ws=ws, mod127=True, injections=inj[:3])
    assert np.array_equal(out["C"], Cw) and np.array_equal(out["flags"], fw) and out["err_count"] == nw and not out["ws"].any()


# (one to fifteen tile columns, eight and more with every remainder by eight; one tile row, two, and a strip of four and one more; each form)
@pytest.mark.gpu
@pytest.mark.parametrize("M,width,K", [(20, 32, 144), (20, 32, 1168), (150, 32, 144), (150, 32, 2321), (2500, 32, 144), (1300, 64, 1296), (40, 480, 144)])
def test_grids_of_any_number_of_tiles(binding, gpu_util, oracle, M, width, K):
    """Every tile is computed once, whatever their number: the XCDs' blocks of tiles are of two lengths where it is no multiple of eight."""
    A, B = operands(M, 15 * width, K, M + K)
    ref = oracle.checked_gemm(A, B)
    for n in range(1, 16):
        N = n * width - (n % 3)
        run = gpu_util.GpuRun(binding, np.ascontiguousarray(B[:, :N]))
        out = run.gemm(A)
        assert np.array_equal(out["C"], ref.C[:, :N]) and not out["flags"].any() and out["err_count"] == 0 and not out["ws"].any(), N


# (widths around four columns, a quad of lanes, 32-column blocks and whole tiles; one to four rows past the last whole quad)
@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K,variant", [(5, 1, 64, "auto"), (20, 67, 128, "auto"), (33, 130, 1040, "auto"), (70, 3, 64, "tile64"), (129, 65, 96, "tile64"),
                                           (66, 257, 97, "auto"), (131, 254, 64, "tile128"), (258, 515, 64, "tile256"), (512, 512, 64, "tile256")])
def test_requantized_quads(binding, gpu_util, oracle, M, N, K, variant):
    """The uint8 output, stored four columns at a time, in rows that start at any byte: every value as the oracle's, faults and
    multipliers that are zero, negative, infinite or no number included, and nothing written beside it."""
    import torch
    say(f"requantized quads: {M}x{N}x{K} {variant}")
    A, B = operands(M, N, K, 3 * M + N)
    inj = [(M - 1, N - 1, 1 << 20), (0, 0, 1 << 12), (M // 2, N // 2, 1 << 31)]
    ref = oracle.checked_gemm(A, B, flips_c=inj)
    run = gpu_util.GpuRun(binding, B)
    ws = binding.Workspace(M, run.Bp).tensor
    rng = np.random.default_rng(N)
    mult = wlmod.draw_mult(rng, N, "channel")
    mult[::7] = [np.float32(v) for v in (0.0, -1e-3, np.inf, -np.inf, np.nan, 1e30)][N % 6]
    bias = rng.integers(-3000, 3000, size=N).astype(np.int32)
    with np.errstate(all="ignore"):
        t = (ref.C.astype(np.int64) - 128 * ref.colsum.astype(np.int64) + bias).astype(np.uint32).view(np.int32).astype(np.float32)
        want = np.fmin(np.fmax(np.rint(t * mult) + np.float32(7), np.float32(0)), np.float32(255)).astype(np.uint8)
    keep = (gpu_util.dev(mult), gpu_util.dev(bias))
    rq = binding.make_requant(128, 7, *keep)
    A_dev, inj_dev = gpu_util.dev(A), binding.make_injections(inj)
    for want_c in (False, True):
        buf = torch.full((M * (N + 5) + 3,), 99, dtype=torch.uint8, device="cuda")
        Cq = buf[3:].view(M, N + 5)[:, :N]
        C = torch.zeros((M, N), dtype=torch.int32, device="cuda") if want_c else None
        flags = torch.empty(M, dtype=torch.int32, device="cuda")
        binding.abft_gemm_u8s8s32_checked(A_dev, run.Bp, C, flags, None, rq=rq, Cq=Cq, inj=inj_dev, n_inj=len(inj),
                                          flags=gpu_util.VARIANTS[variant], workspace=ws)
        torch.cuda.synchronize()
        assert np.array_equal(Cq.cpu().numpy(), want) and np.array_equal(flags.cpu().numpy(), ref.flags)
        assert (buf[:3] == 99).all() and (buf[3:].view(M, N + 5)[:, N:] == 99).all()
        if want_c:
            assert np.array_equal(C.cpu().numpy(), ref.C)


@pytest.mark.gpu
def test_requantized_full_grid(binding, gpu_util, oracle):
    """The uint8 output alone on a grid of 256 tiles of 256x256, whole ones (byte by byte) beside cut ones (by fours): checked with
    faults in both, and unchecked, whose faults move Cq all the same; rows that start at any byte, nothing written beside them."""
    import torch
    M, N, K = 4094, 4093, 64
    A, B = operands(M, N, K, 9)
    inj = [(M - 1, N - 1, 1 << 20), (0, 0, 1 << 12), (M // 2, N // 2, 1 << 31), (700, 4092, 1 << 15), (4093, 900, 1 << 14)]
    ref = oracle.checked_gemm(A, B, flips_c=inj)
    mult = wlmod.draw_mult(np.random.default_rng(N), N, "channel")
    want = oracle.requantize(ref.C, ref.colsum, 128, 7, mult, precision="f32")
    run = gpu_util.GpuRun(binding, B)
    ws = binding.Workspace(M, run.Bp).tensor
    keep = gpu_util.dev(mult)
    rq = binding.make_requant(128, 7, keep)
    A_dev, inj_dev = gpu_util.dev(A), binding.make_injections(inj)
    for how in (binding.ABFT_CHECK, binding.ABFT_NOCHECK):
        buf = torch.full((M * (N + 5) + 3,), 99, dtype=torch.uint8, device="cuda")
        Cq = buf[3:].view(M, N + 5)[:, :N]
        flags = torch.zeros(M, dtype=torch.int32, device="cuda")
        binding.abft_gemm_u8s8s32_checked(A_dev, run.Bp, None, flags, None, rq=rq, Cq=Cq, inj=inj_dev, n_inj=len(inj), flags=how, workspace=ws)
        torch.cuda.synchronize()
        assert np.array_equal(Cq.cpu().numpy(), want)
        assert (buf[:3] == 99).all() and (buf[3:].view(M, N + 5)[:, N:] == 99).all()
        assert np.array_equal(flags.cpu().numpy(), ref.flags if how == binding.ABFT_CHECK else np.zeros(M, np.int32))


# (each tile form with one stage, stages that no wavefront, some or all wavefronts have, tiles and stages cut off, rows of whole chunks
# and of any length; slots for 64, 128 and 256 rows; K split across workgroups; weights of more than 96 MiB, which pass the caches by)
@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K", [(1, 1, 16), (17, 33, 17), (31, 31, 128), (33, 65, 1008), (100, 129, 1153), (257, 95, 2049), (65, 200, 4111),
                                   (300, 900, 304), (320, 1000, 1553), (257, 1025, 3090), (1000, 1000, 1296), (1023, 963, 1290), (130, 3500, 70),
                                   (16, 1600, 80), (5, 8000, 200), (64, 1537, 1201), (65, 3200, 250), (128, 3105, 1040), (129, 1700, 144), (256, 1569, 90),
                                   (40, 70, 8192), (129, 40, 3000), (33, 200, 5001), (3, 100, 9000), (1030, 40, 112), (3001, 80, 160), (1030, 40, 300), (3001, 80, 400), (2100, 300, 1552), (1100, 1800, 131), (700, 1950, 1279),
                                   (16, 12000, 9008), (3, 12100, 8999), (9, 8192, 12400), (2, 7900, 13003)])
def test_k_split_among_wavefronts(binding, gpu_util, oracle, M, N, K):
    """Grids that do not fill the chip: clean, C and B faults early and late in K and in the last row and column, both outputs,
    unchecked, errCount overwritten, added to and absent, the printed modulus where rows are whole chunks."""
    say(f"K split among wavefronts {M}x{N}x{K}")
    A, B = operands(M, N, K, 3 * M + N + K)
    run = gpu_util.GpuRun(binding, B)
    clean = oracle.checked_gemm(A, B)
    mult = wlmod.draw_mult(np.random.default_rng(K), N, "channel")
    bias = np.random.default_rng(M).integers(-9000, 9000, size=N).astype(np.int32)
    out = run.gemm(A, requant=(128, 128, mult, bias))
    assert np.array_equal(out["C"], clean.C) and not out["flags"].any() and out["err_count"] == 0 and not out["ws"].any()
    assert np.array_equal(out["Cq"], oracle.requantize(clean.C, clean.colsum, 128, 128, mult, bias, precision="f32"))
    out = run.gemm(A, requant=(128, 128, mult, bias), want_c=False, want_count=False)
    assert np.array_equal(out["Cq"], oracle.requantize(clean.C, clean.colsum, 128, 128, mult, bias, precision="f32")) and not out["flags"].any()
    assert np.array_equal(run.gemm(A, check=False)["C"], clean.C)
    inj = [(M - 1, N - 1, 1 << 31), (0, 0, 1 << 3), (M // 2, N // 3, 0x00400000)]
    ref = oracle.checked_gemm(A, B, flips_c=inj)
    for accumulate in (None, 5):
        out = run.gemm(A, injections=inj, accumulate_from=accumulate)
        assert np.array_equal(out["C"], ref.C) and np.array_equal(out["flags"], ref.flags) and out["err_count"] == (accumulate or 0) + ref.err_count
    for flip in ((0, N - 1, 6), (K - 1, N // 2, 7), (K // 2, 0, 2)):
        binding.abft_packed_b_flip_bit(run.Bp, *flip)
        ref = oracle.checked_gemm(A, B, flips_b=[flip])
        out = run.gemm(A)
        assert np.array_equal(out["C"], ref.C) and np.array_equal(out["flags"], ref.flags) and out["err_count"] == ref.err_count
        binding.abft_packed_b_flip_bit(run.Bp, *flip)
    if K % 16 == 0:
        C127, flags127, count127 = oracle.checked_gemm_mod127(A, B, flips_c=inj)
        out = run.gemm(A, injections=inj, mod127=True)
        assert np.array_equal(out["C"], C127) and np.array_equal(out["flags"], flags127) and out["err_count"] == count127
    assert not run.gemm(A)["flags"].any()


# (64x64 tiles on grids beyond the chip, with one, two and more stages than the two that LDS holds, rows of whole chunks, of any length
# and shorter than a chunk)
@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K", [(1100, 1030, 16), (1100, 1030, 128), (1025, 1100, 144), (1100, 1030, 256), (1090, 1030, 272), (1100, 1030, 640), (2100, 1030, 100),
                                   (2100, 1030, 131), (2100, 1030, 300), (2100, 1030, 401), (2100, 1030, 13), (8200, 130, 384),
                                   # (slots between many tile columns and a row's word: 32, 8 and 4 of them, at the last number of rows for each, and none)
                                   (40, 17000, 256), (128, 9000, 128), (150, 1630, 272), (192, 6500, 160), (193, 8000, 131), (384, 3200, 144), (385, 3200, 144),
                                   # (more tiles than two to a compute unit on the kernel that splits K among wavefronts: 32x64 and 64x64 tiles, rows of whole
                                   # chunks and of any length, with and without a copy ahead; large grids and a short K on 64x64 tiles)
                                   (215, 4173, 1690), (90, 8237, 1040), (1100, 1001, 2064), (1350, 900, 2500), (700, 3100, 1313), (396, 4325, 2309), (1423, 1227, 303), (2300, 3000, 300), (1953, 4100, 96)])
def test_64x64_tiles_of_few_stages(binding, gpu_util, oracle, M, N, K):
    test_k_split_among_wavefronts(binding, gpu_util, oracle, M, N, K)


@pytest.mark.gpu
def test_weights_replaced_while_others_are_in_use(binding, gpu_util, oracle):
    """Blocks of destroyed weights serve later ones: never while work enqueued before still reads them, on whatever stream, from several
    threads at once, blocks of other sizes among them; all memory is given back with the last weight."""
    import threading

    import torch

    say("weights replaced while others are in use")
    M, N, K = 40, 700, 1500
    rng = np.random.default_rng(5)
    A = rng.integers(0, 256, size=(M, K), dtype=np.uint8)
    weights = [rng.integers(-127, 128, size=(K, N), dtype=np.int8) for _ in range(6)]
    wants = [torch.from_numpy(oracle.checked_gemm(A, B).C).cuda() for B in weights]
    A_dev, B_dev = gpu_util.dev(A), [gpu_util.dev(B) for B in weights]
    torch.cuda.synchronize()
    free0 = torch.cuda.mem_get_info()[0]
    failed = []

    def work(first):
        try:
            stream, side = torch.cuda.Stream(), torch.cuda.Stream()
            done = []
            with torch.cuda.stream(stream):
                Bp, ws = None, None
                for r in range(40):
                    w = (first + r) % len(weights)
                    if r % 9 == 8:    # another size in between
                        binding.abft_pack_b_checksum(B_dev[0][: K // 3].contiguous())
                    Bp = binding.abft_pack_b_checksum(B_dev[w])    # (the one before is destroyed; its products may not even have begun)
                    ws = binding.Workspace(M, Bp) if ws is None else ws
                    side.wait_stream(stream)
                    C = [torch.empty(M, N, dtype=torch.int32, device="cuda") for _ in range(12)]
                    flags = torch.empty(M, dtype=torch.int32, device="cuda")
                    with torch.cuda.stream(side):
                        for c in C:
                            binding.abft_gemm_u8s8s32_checked(A_dev, Bp, c, flags, None, workspace=ws.tensor)
                    done.append((w, C, flags, Bp if r == 39 else None))
            side.synchronize()
            for w, C, flags, _ in done:
                if not all(torch.equal(c, wants[w]) for c in C) or bool(flags.any()):
                    failed.append(("wrong product", first, w))
        except Exception as e:    # (a failure in a thread is the test's)
            failed.append(repr(e))

    work(0)
    threads = [threading.Thread(target=work, args=(i,)) for i in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not failed, failed[:3]
    big = [binding.abft_pack_b_checksum(torch.zeros(8192, 9000, dtype=torch.int8, device="cuda")) for _ in range(6)]    # more than is kept
    del big
    torch.cuda.empty_cache()
    torch.cuda.synchronize()
    assert torch.cuda.mem_get_info()[0] >= free0 - (96 << 20)    # (torch's own pools of the new streams; six blocks of 74 MB were there)


@pytest.mark.gpu
@pytest.mark.parametrize("late,others", [(False, 0), (True, 0), (True, 18)])
def test_weights_replaced_back_to_back(binding, gpu_util, oracle, late, others):
    """Replacements with nothing else between them, each used once on another stream: the kept blocks run full, and the one wait that follows comes
    before any of them is written again.  late: that stream has work of some milliseconds ahead of the first product.  others: so many weights of
    other sizes have been destroyed before, whose blocks fill the list."""
    import torch

    say(f"weights replaced back to back, late={late}, others={others}")
    M, N, K = 24, 700, 1500
    rng = np.random.default_rng(6)
    A = rng.integers(0, 256, size=(M, K), dtype=np.uint8)
    weights = [rng.integers(-127, 128, size=(K, N), dtype=np.int8) for _ in range(5)]
    wants = [torch.from_numpy(oracle.checked_gemm(A, B).C).cuda() for B in weights]
    A_dev, B_dev = gpu_util.dev(A), [gpu_util.dev(B) for B in weights]
    Bp = binding.abft_pack_b_checksum(B_dev[0])
    ws = binding.Workspace(M, Bp)
    C = [torch.full((M, N), -7, dtype=torch.int32, device="cuda") for _ in range(60)]
    flags = [torch.full((M,), -1, dtype=torch.int32, device="cuda") for _ in C]
    side = torch.cuda.Stream()
    busy = torch.zeros(1 << 28, dtype=torch.int32, device="cuda")
    spare = [binding.abft_pack_b_checksum(torch.zeros(2000 + 300 * i, 700, dtype=torch.int8, device="cuda")) for i in range(others)]
    del spare
    torch.cuda.synchronize()
    if late:
        with torch.cuda.stream(side):
            for _ in range(30):
                busy.add_(1)
    for r in range(len(C)):
        Bp = binding.abft_pack_b_checksum(B_dev[r % len(weights)])
        side.wait_stream(torch.cuda.current_stream())
        binding.abft_gemm_u8s8s32_checked(A_dev, Bp, C[r], flags[r], None, workspace=ws.tensor, stream=side)
    torch.cuda.synchronize()
    for r in range(len(C)):
        assert torch.equal(C[r], wants[r % len(weights)]), r
        assert not bool(flags[r].any()), r


@pytest.mark.gpu
def test_pack_while_streams_are_captured(binding, gpu_util, oracle):
    """Kept blocks change nothing there: a weight packed on a captured stream gets a block of its own, into which every replay packs anew; a call that
    another stream's capture forbids is refused although a block is kept."""
    import ctypes
    import types

    import torch

    say("pack while streams are captured")
    M, N, K = 40, 300, 700
    rng = np.random.default_rng(8)
    A = rng.integers(0, 256, size=(M, K), dtype=np.uint8)
    weights = [rng.integers(-127, 128, size=(K, N), dtype=np.int8) for _ in range(3)]
    wants = [torch.from_numpy(oracle.checked_gemm(A, B).C).cuda() for B in weights]
    A_dev, B_dev = gpu_util.dev(A), [gpu_util.dev(B) for B in weights]
    held = binding.abft_pack_b_checksum(B_dev[0])
    ws = binding.Workspace(M, held)
    C = torch.full((M, N), -7, dtype=torch.int32, device="cuda")
    flags = torch.full((M,), -1, dtype=torch.int32, device="cuda")
    into = B_dev[0].clone()
    for _ in range(2):    # blocks are kept, waited for and not
        spare = [binding.abft_pack_b_checksum(B_dev[1]) for _ in range(3)]
        del spare
        torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, capture_error_mode="relaxed"):
        captured = binding.abft_pack_b_checksum(into)
        binding.abft_gemm_u8s8s32_checked(A_dev, captured, C, flags, None, workspace=ws.tensor)
    for r in range(6):
        into.copy_(B_dev[r % 3])
        graph.replay()
        others = [binding.abft_pack_b_checksum(B) for B in B_dev]    # (between the replays, other weights come and go)
        assert torch.equal(C, wants[r % 3]) and not bool(flags.any())
        for B, want in zip(others, wants):
            binding.abft_gemm_u8s8s32_checked(A_dev, B, C, flags, None, workspace=ws.tensor)
            assert torch.equal(C, want)
        del others
    torch.cuda.synchronize()
    del graph, captured

    with open("/proc/self/maps") as maps:
        runtime = next(line.split()[-1] for line in maps if "libamdhip64.so" in line)
    hip = ctypes.CDLL(runtime)
    stream = ctypes.c_void_p()
    assert hip.hipStreamCreateWithFlags(ctypes.byref(stream), 1) == 0
    assert hip.hipStreamBeginCapture(stream, 0) == 0    # (global: unsafe calls of any thread are refused, and end the capture)
    current = types.SimpleNamespace(cuda_stream=torch._C._cuda_getCurrentRawStream(0))
    with pytest.raises(binding.AbftError) as refused:
        binding.abft_pack_b_checksum(B_dev[0], stream=current)
    assert refused.value.code == binding.ABFT_EHIP
    recorded = ctypes.c_void_p()
    hip.hipStreamEndCapture(stream, ctypes.byref(recorded))
    hip.hipGetLastError()
    assert hip.hipStreamDestroy(stream) == 0
    again = binding.abft_pack_b_checksum(B_dev[2])
    binding.abft_gemm_u8s8s32_checked(A_dev, again, C, flags, None, workspace=ws.tensor)
    assert torch.equal(C, wants[2])


@pytest.mark.gpu
def test_kept_memory_is_given_back(binding):
    import torch

    say("kept memory is given back")
    held = binding.abft_pack_b_checksum(torch.zeros(64, 64, dtype=torch.int8, device="cuda"))
    B = torch.zeros(8192, 8192, dtype=torch.int8, device="cuda")
    binding.abft_packed_b_trim()
    free = torch.cuda.mem_get_info()[0]
    weights = [binding.abft_pack_b_checksum(B) for _ in range(3)]
    del weights
    torch.cuda.synchronize()
    assert torch.cuda.mem_get_info()[0] < free - (180 << 20)    # (three blocks of 64 MiB and more)
    binding.abft_packed_b_trim()
    assert torch.cuda.mem_get_info()[0] > free - (8 << 20)
    held.destroy()


@pytest.mark.gpu
@pytest.mark.parametrize("transposed", [False, True])
def test_pack_into_blocks_of_other_weights(binding, gpu_util, oracle, transposed):
    """The sums of a weight meet in accumulators that the one before it has left at zero, or, where that one's lay elsewhere in the block, that are cleared
    first: weights of the same tiles, of others whose block is of about the same size, with what was flipped in between and where it takes a new one."""
    import torch

    say(f"pack into blocks of other weights, transposed={transposed}")
    rng = np.random.default_rng(12)
    held = binding.abft_pack_b_checksum(gpu_util.dev(rng.integers(-127, 128, size=(64, 64), dtype=np.int8)))
    sizes = [(3000, 700), (2999, 690), (3000, 700), (2900, 700), (3060, 513), (2900, 768), (16384, 20), (16300, 256), (20, 16385), (100, 16400), (3000, 700)]
    for r in range(3):
        for K, N in sizes:
            B = rng.integers(-128, 128, size=(K, N)).astype(np.int8)
            run = gpu_util.GpuRun(binding, B, transposed)
            wide = B.astype(np.int64)
            assert np.array_equal(run.checksum(), wide.sum(1)) and np.array_equal(run.colsum(), wide.sum(0)), (r, K, N)
            residues = torch.empty(K, dtype=torch.int32, device="cuda")
            binding.abft_packed_b_get_checksum_mod127(run.Bp, residues)
            assert np.array_equal(residues.cpu().numpy(), wide.sum(1) % 127)
            A = rng.integers(0, 256, size=(3, K), dtype=np.uint8)
            out = run.gemm(A)
            assert np.array_equal(out["C"], oracle.checked_gemm(A, B).C) and not out["flags"].any()
            binding.abft_packed_b_flip_checksum_bit(run.Bp, K // 2, r)
            binding.abft_packed_b_flip_bit(run.Bp, K // 3, N // 2, r)
    assert held


# (weights of many tiles in a row or a column)
@pytest.mark.gpu
@pytest.mark.parametrize("transposed", [False, True])
@pytest.mark.parametrize("K,N", [(64, 20), (300, 1100), (16384, 20), (16385, 20), (20, 16384), (20, 16385)])
def test_pack_of_many_tiles(binding, gpu_util, oracle, K, N, transposed):
    test_pack_of_strided_weights(binding, gpu_util, oracle, K, N, transposed)
