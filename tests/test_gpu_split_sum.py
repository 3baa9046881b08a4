"""A split of K over the grid that the product kernel sums itself (the block that takes the last ticket of a tile, counted
in the output) gives the bits of the separate sum kernel, which outputs that are not 8-byte aligned still take -- whatever
the output holds before the call, call after call, on two streams at once and replayed from a graph."""
import pytest

from gpu_util import kernels_of, torch_mod

pytestmark = pytest.mark.gpu

# (rows, K, N, bits, g, type): the smallest call; one and several column groups per block, with and without k-workers; a last
# block with column tiles past the end; two and three row tiles with ragged rows
SHAPES = [(4, 1024, 1024, 4, 128, "f16"), (1, 15744, 1248, 4, 128, "bf16"), (13, 6528, 3728, 4, 32, "f16"),
          (16, 8192, 10000, 8, 128, "bf16"), (3, 2048, 16, 3, 64, "f16"), (21, 3200, 4400, 4, 64, "f16"),
          (30, 7296, 2432, 8, 64, "f16"), (43, 7552, 1584, 4, 32, "bf16"), (48, 10240, 5264, 4, 128, "bf16")]


def _case(M, K, N, bits, g, act, seed=1):
    from paper_2308_09723_amd import fq
    torch = torch_mod()
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    W = (torch.randn((K, N), generator=gen, device="cuda") * 0.02).to(torch.float16)
    codes, scales = fq.quantize(W, bits, g)
    A = torch.randn((M, K), generator=gen, device="cuda").to(torch.float16 if act == "f16" else torch.bfloat16)
    need = fq.gemm_workspace_bytes(M, N, K, bits, g)
    assert need > 0, "the product does not split K"
    return A, codes, scales, torch.empty(need, dtype=torch.uint8, device="cuda")


def _outputs(M, N, dtype):
    """An aligned output and one that starts two bytes past an aligned address."""
    torch = torch_mod()
    return torch.empty((M, N), dtype=dtype, device="cuda"), torch.empty(M * N + 4, dtype=dtype, device="cuda")[1:1 + M * N].view(M, N)


@pytest.mark.parametrize("M,K,N,bits,g,act", SHAPES)
def test_same_bits_as_the_separate_sum(M, K, N, bits, g, act):
    from paper_2308_09723_amd import fq
    torch = torch_mod()
    A, codes, scales, ws = _case(M, K, N, bits, g, act)
    C, apart = _outputs(M, N, A.dtype)
    assert C.data_ptr() % 8 == 0 and apart.data_ptr() % 8 == 2
    want = fq.gemm(A, codes, scales, bits, g, out=apart, workspace=ws).clone()
    fq.gemm(A, codes, scales, bits, g, out=C, workspace=ws)
    assert kernels_of(lambda: fq.gemm(A, codes, scales, bits, g, out=C, workspace=ws)) == 1
    assert kernels_of(lambda: fq.gemm(A, codes, scales, bits, g, out=apart, workspace=ws)) == 2
    exact = A.double() @ (fq.unpack(codes, K, N, bits).double() * scales.double().repeat_interleave(g, 0))
    assert float((want.double() - exact).norm() / exact.norm()) < (1.2e-3 if act == "f16" else 7e-3)
    # zeros, the results themselves, NaNs, and words that look like tickets of other calls, full and begun
    fills = [lambda: C.zero_(), lambda: None, lambda: C.fill_(float("nan")), lambda: C.view(torch.int16).fill_(-91)]
    fills += [lambda n=n: C.view(torch.int64).fill_((-91 << 48) | n) for n in (0, 1, 7, 0x12345600)]
    for i, fill in enumerate(fills * 3):
        fill()
        assert torch.equal(fq.gemm(A, codes, scales, bits, g, out=C, workspace=ws).view(torch.int16), want.view(torch.int16)), i


def test_two_streams_at_once():
    from paper_2308_09723_amd import fq
    torch = torch_mod()
    cases = [_case(4, 1024, 1024, 4, 128, "f16", 3) + (4, 128), _case(21, 3200, 4400, 4, 64, "f16", 4) + (4, 64)]
    wants = [fq.gemm(A, c, s, b, g) for A, c, s, ws, b, g in cases]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in cases]
    got = [[] for _ in cases]
    for _ in range(20):
        for i, (A, c, s, ws, b, g) in enumerate(cases):
            with torch.cuda.stream(streams[i]):
                got[i].append(fq.gemm(A, c, s, b, g, workspace=ws))
    torch.cuda.synchronize()
    for want, outs in zip(wants, got):
        assert all(torch.equal(o, want) for o in outs)


def test_replayed_with_the_tag_it_was_captured_with():
    from paper_2308_09723_amd import fq
    torch = torch_mod()
    A, codes, scales, ws = _case(13, 6528, 3728, 4, 32, "f16")
    C = torch.empty((13, 3728), dtype=A.dtype, device="cuda")
    fq.gemm(A, codes, scales, 4, 32, out=C, workspace=ws)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        fq.gemm(A, codes, scales, 4, 32, out=C, workspace=ws)
    for rep in range(5):
        A.mul_(1.5)
        want = fq.gemm(A, codes, scales, 4, 32)        # eager work between the replays
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(C, want), rep


@pytest.mark.parametrize("M,K,N,g,act", [(4, 4096, 1024, 128, "f16"), (1, 8448, 1024, 128, "bf16"), (16, 16256, 1808, 32, "f16"),
                                         (13, 15744, 2048, 96, "bf16"), (43, 7040, 1472, 32, "bf16"), (52, 15744, 1552, 64, "f16"),
                                         (130, 16384, 1040, 128, "bf16")])
def test_integer_path_same_bits_as_the_separate_sum(M, K, N, g, act):
    from paper_2308_09723_amd import fq
    torch = torch_mod()
    gen = torch.Generator(device="cuda")
    gen.manual_seed(2)
    dtype = torch.float16 if act == "f16" else torch.bfloat16
    codes, z, t = fq.quantize_w4a8((torch.randn((K, N), generator=gen, device="cuda") * 0.02).to(torch.float16), g)
    Aq, alpha = fq.quantize_act_i8(torch.randn((M, K), generator=gen, device="cuda").to(dtype))
    need = fq.gemm_w4a8_workspace_bytes(M, N, K, g)
    assert need > 0, "the product does not split K"
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    C, apart = _outputs(M, N, dtype)
    want = fq.gemm_w4a8(Aq, alpha, codes, z, t, g, dtype, out=apart, workspace=ws).clone()
    fq.gemm_w4a8(Aq, alpha, codes, z, t, g, dtype, out=C, workspace=ws)
    assert kernels_of(lambda: fq.gemm_w4a8(Aq, alpha, codes, z, t, g, dtype, out=C, workspace=ws)) == 1
    assert kernels_of(lambda: fq.gemm_w4a8(Aq, alpha, codes, z, t, g, dtype, out=apart, workspace=ws)) == 2
    for fill in (lambda: C.zero_(), lambda: None, lambda: C.fill_(float("nan")), lambda: C.view(torch.int64).fill_((-91 << 48) | 3)) * 4:
        fill()
        got = fq.gemm_w4a8(Aq, alpha, codes, z, t, g, dtype, out=C, workspace=ws)
        assert torch.equal(got.view(torch.int16), want.view(torch.int16))
    alpha[0], alpha[M // 2] = float("nan"), float("inf")         # (row 0 holds the tickets)
    want = fq.gemm_w4a8(Aq, alpha, codes, z, t, g, dtype, out=apart, workspace=ws).clone()
    for _ in range(3):
        got = fq.gemm_w4a8(Aq, alpha, codes, z, t, g, dtype, out=C, workspace=ws)
        assert torch.equal(got.view(torch.int16), want.view(torch.int16)) and not torch.isfinite(got[0]).any()


@pytest.mark.parametrize("M,K,N,bits,g,kernels", [(30, 4864, 1824, 4, 32, 1), (28, 5120, 2048, 4, 128, 1), (36, 4480, 2576, 4, 64, 2),
                                                  (32, 5248, 1776, 3, 32, 2), (16, 8192, 28672, 8, 128, 2)])
def test_tiles_of_more_than_80_KiB_of_partial_sums_are_summed_by_a_second_kernel(M, K, N, bits, g, kernels):
    """78.8, 73.5, 81, 84 and 180 KiB per tile: the kernel that runs, and the results of either."""
    from paper_2308_09723_amd import fq
    torch = torch_mod()
    A, codes, scales, ws = _case(M, K, N, bits, g, "f16")
    C, apart = _outputs(M, N, A.dtype)
    want = fq.gemm(A, codes, scales, bits, g, out=apart, workspace=ws)
    assert torch.equal(fq.gemm(A, codes, scales, bits, g, out=C, workspace=ws), want)
    assert kernels_of(lambda: fq.gemm(A, codes, scales, bits, g, out=C, workspace=ws)) == kernels


@pytest.mark.parametrize("M,K,N,bits,g,act", [SHAPES[0], SHAPES[1], SHAPES[4], SHAPES[5], SHAPES[7]])
def test_results_that_are_not_finite_have_the_bits_of_the_separate_sum(M, K, N, bits, g, act):
    """Infinities and NaNs in row 0, whose first results hold the tickets, among them the NaN that a ticket's upper bits are."""
    from paper_2308_09723_amd import fq
    torch = torch_mod()
    A, codes, scales, ws = _case(M, K, N, bits, g, act)
    C, apart = _outputs(M, N, A.dtype)
    A[M - 1, K // 2] = float("inf")
    for first in (float("inf"), float("-inf"), float("nan"), -91):
        if first == -91:
            A.view(torch.int16)[0, 5] = first
        else:
            A[0, 5] = first
        want = fq.gemm(A, codes, scales, bits, g, out=apart, workspace=ws).clone()
        for _ in range(3):
            got = fq.gemm(A, codes, scales, bits, g, out=C, workspace=ws)
            assert torch.equal(got.view(torch.int16), want.view(torch.int16)) and not torch.isfinite(got[0]).all()


def test_a_product_over_its_own_activations_sums_in_a_second_kernel():
    """C on memory that the product reads: tickets there would change what other blocks still read, so the separate kernel adds
    the partial sums once everything is read, and the result is that of an output of its own."""
    from paper_2308_09723_amd import fq
    torch = torch_mod()
    A, codes, scales, ws = _case(4, 1024, 1024, 4, 128, "f16")
    def product(a, c):
        return fq.gemm(a, codes, scales, 4, 128, out=c, workspace=ws)

    C = torch.empty_like(A)
    want = product(A, C).clone()
    rows = torch.cat([A, A])                 # the output begins in the middle of the activations
    assert kernels_of(lambda: product(A, C)) == 1
    assert kernels_of(lambda: product(A, A)) == kernels_of(lambda: product(rows[:4], rows[2:6])) == 2
    product(rows[:4], rows[2:6])
    assert torch.equal(rows[2:6], want) and torch.equal(rows[:2], A[:2]) and torch.equal(rows[6:], A[2:])
    product(A, A)
    assert torch.equal(A, want)


def test_integer_path_over_its_own_activations_sums_in_a_second_kernel():
    from paper_2308_09723_amd import fq
    torch = torch_mod()
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)
    codes, z, t = fq.quantize_w4a8((torch.randn((4096, 1024), generator=gen, device="cuda") * 0.02).to(torch.float16), 128)
    Aq, alpha = fq.quantize_act_i8(torch.randn((4, 4096), generator=gen, device="cuda").to(torch.float16))
    ws = torch.empty(fq.gemm_w4a8_workspace_bytes(4, 1024, 4096, 128), dtype=torch.uint8, device="cuda")
    C, over = torch.empty((4, 1024), dtype=torch.float16, device="cuda"), Aq.view(torch.float16).view(-1)[:4096].view(4, 1024)

    def product(c):
        return fq.gemm_w4a8(Aq, alpha, codes, z, t, 128, torch.float16, out=c, workspace=ws)

    want = product(C).clone()
    assert kernels_of(lambda: product(C)) == 1 and kernels_of(lambda: product(over)) == 2
    assert torch.equal(product(over), want)


def test_outputs_and_scratch_in_host_memory_are_summed_by_a_second_kernel():
    """Tickets are counted with atomics of the device: C in pinned host memory is only stored to, and partial sums there are read
    by a later kernel."""
    from paper_2308_09723_amd import fq
    torch = torch_mod()
    A, codes, scales, ws = _case(4, 1024, 1024, 4, 128, "f16")
    C, host = torch.empty_like(A), torch.zeros((4, 1024), dtype=torch.float16, pin_memory=True)

    def product(c, scratch=ws):
        return fq.gemm(A, codes, scales, 4, 128, out=c, workspace=scratch)

    want = product(C).clone()
    host_ws = torch.zeros(ws.numel(), dtype=torch.uint8, pin_memory=True)
    assert kernels_of(lambda: product(C)) == 1 and kernels_of(lambda: product(host)) == kernels_of(lambda: product(C, host_ws)) == 2
    product(host)
    product(C.zero_(), host_ws)
    torch.cuda.synchronize()
    assert torch.equal(host, want.cpu()) and torch.equal(C, want)
    codes, z, t = fq.quantize_w4a8((torch.randn((4096, 1024), device="cuda") * 0.02).to(torch.float16), 128)
    Aq, alpha = fq.quantize_act_i8(torch.randn((4, 4096), device="cuda").to(torch.float16))
    ws = torch.empty(fq.gemm_w4a8_workspace_bytes(4, 1024, 4096, 128), dtype=torch.uint8, device="cuda")

    def integer(c):
        return fq.gemm_w4a8(Aq, alpha, codes, z, t, 128, torch.float16, out=c, workspace=ws)

    want = integer(C).clone()
    assert kernels_of(lambda: integer(C)) == 1 and kernels_of(lambda: integer(host)) == 2
    integer(host)
    torch.cuda.synchronize()
    assert torch.equal(host, want.cpu())


def test_the_librarys_own_scratch_is_plain_memory():
    """fq_gemm_noalloc adds its splits in one kernel, too."""
    from paper_2308_09723_amd import fq
    torch = torch_mod()
    A, codes, scales, ws = _case(4, 1024, 1024, 4, 128, "f16")
    C = torch.empty_like(A)

    def noalloc():
        assert fq.gemm_noalloc_raw(A.data_ptr(), fq.FQ_F16, 4, 1024, 1024, codes.data_ptr(), scales.data_ptr(), 4, 128, C.data_ptr(),
                                   torch.cuda.current_stream().cuda_stream) == fq.FQ_OK

    noalloc()
    assert torch.equal(C, fq.gemm(A, codes, scales, 4, 128, workspace=ws)) and kernels_of(noalloc) == 1
