"""Parity of each HIP kernel, called through the C ABI, against the CPU oracle on the same seeded inputs."""
import ctypes as C

import numpy as np
import pytest
import torch

import flover_synth as synth
from oracle import oracle as orc

pytestmark = pytest.mark.gpu

fl = None


@pytest.fixture(scope="module", autouse=True)
def _lib():
    global fl
    assert torch.cuda.is_available(), "these tests need the MI355X"
    import paper_2305_13484_amd as m
    fl = m
    m.load_library()


TDT = synth.TORCH_DTYPE


# ---------------------------------------------------------------- weight GEMM

@pytest.mark.parametrize("dtype", [synth.DT_BF16, synth.DT_F16, synth.DT_F32])
@pytest.mark.parametrize("M,N,K", [(1, 64, 64), (5, 100, 96), (16, 256, 512), (17, 1000, 256), (33, 130, 1024),
                                   (70, 320, 2048), (128, 192, 4096), (200, 64, 160), (300, 320, 1024),
                                   (513, 130, 512), (48, 200, 512), (90, 130, 1024), (100, 320, 512)])
def test_gemm_matches_oracle(dtype, M, N, K):
    print("gemm", dtype, M, N, K, flush=True)
    g = torch.Generator().manual_seed(100 + M + N)
    x = torch.randn((M, K), generator=g).to(TDT[dtype])
    W = (torch.randn((N, K), generator=g) * 0.05).to(TDT[dtype])
    ref = orc.gemm(dtype, x, W)
    got = fl.k_gemm(x.cuda(), W.cuda()).cpu().double().numpy()
    bound = (x.double().abs() @ W.double().abs().T).numpy()       # sum of |terms| per output
    assert np.all(np.abs(got - ref) <= 4e-6 * bound + 1e-30)


@pytest.mark.parametrize("dtype", [synth.DT_BF16, synth.DT_F16])
def test_gemm_row_result_does_not_depend_on_other_rows(dtype):
    g = torch.Generator().manual_seed(5)
    K, N = 1024, 448
    x = torch.randn((600, K), generator=g).to(TDT[dtype]).cuda()
    W = (torch.randn((N, K), generator=g) * 0.05).to(TDT[dtype]).cuda()
    tw = fl.binding.TiledWeight(W)
    full = fl.k_gemm(x, tw)
    for M in (1, 16, 17, 32, 48, 64, 65, 81, 96, 100, 112, 128, 129, 256, 257, 400, 513):   # every count of 16-row tiles up to 8
        part = fl.k_gemm(x[:M].contiguous(), tw)
        assert torch.equal(part, full[:M]), M
    alone = fl.k_gemm(x[77:78].contiguous(), tw)
    assert torch.equal(alone[0], full[77])


@pytest.mark.parametrize("M", [8, 24, 48, 72, 96, 112, 128, 600])
def test_gemm_full_size_sampled_columns(M):
    """The 7B shapes the benchmark runs, at row counts that select each kernel variant (<=16 direct, <=32 / <=64 / <=128
    LDS-staged with 4 or 8 waves, above that the 256-row blocks of a context pass with a ragged last block); sampled
    output columns from the oracle."""
    dtype = synth.DT_BF16
    for (N, K) in [(12288, 4096), (4096, 11008), (22016, 4096), (32000, 4096)]:
        print("gemm full", M, N, K, flush=True)
        g = torch.Generator(device="cuda").manual_seed(N + M)
        x = torch.randn((M, K), generator=g, device="cuda").to(TDT[dtype])
        W = (torch.randn((N, K), generator=g, device="cuda") * 0.02).to(TDT[dtype])
        got = fl.k_gemm(x, W)
        cols = np.random.default_rng(N).choice(N, size=24, replace=False)
        cols = np.concatenate([cols, [0, N - 1]]).astype(np.int32)
        xh, Wh = x.cpu(), W[torch.as_tensor(cols, device="cuda").long()].cpu().contiguous()
        ref = orc.gemm(dtype, xh, Wh)
        bound = (xh.double().abs() @ Wh.double().abs().T).numpy()
        err = np.abs(got[:, torch.as_tensor(cols, device="cuda").long()].cpu().double().numpy() - ref)
        assert np.all(err <= 4e-6 * bound)
        del W


@pytest.mark.parametrize("dtype", [synth.DT_BF16, synth.DT_F16])
@pytest.mark.parametrize("M,N,K", [(129, 70, 32), (191, 130, 64), (257, 320, 96), (130, 4100, 160), (300, 2050, 512), (513, 8192, 288),
                                   (700, 8192, 1024), (900, 12288, 2048), (1024, 22016, 256)])
def test_gemm_of_more_than_128_rows_every_block_shape(dtype, M, N, K):
    """Ragged last row blocks, slices shorter than the copy ring, columns past the last full block, at the shapes' own choice of
    block (which blocks there are is pinned in the next test); the bound is fp32 accumulation (4e-6 of the sum of magnitudes)
    against fp64."""
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    x = torch.randn((M, K), generator=g, device="cuda").to(TDT[dtype])
    W = (torch.randn((N, K), generator=g, device="cuda") * 0.05).to(TDT[dtype])
    got = fl.k_gemm(x, W).double()
    xd, Wd = x.double(), W.double()
    assert torch.all((got - xd @ Wd.T).abs() <= 4e-6 * (xd.abs() @ Wd.abs().T) + 1e-30)


@pytest.mark.parametrize("dtype", [synth.DT_BF16, synth.DT_F32])
@pytest.mark.parametrize("M,N", [(5, 96), (20, 98), (100, 128), (140, 100)])
def test_gemm_takes_rows_as_they_are(dtype, M, N):
    """Rows that end with the allocation, that are a strided view, and that start off the 16-byte grid give the same bits."""
    K = 256
    g = torch.Generator(device="cuda").manual_seed(M)
    x = torch.randn((M, K), generator=g, device="cuda").to(TDT[dtype])
    tw = fl.binding.TiledWeight(torch.randn((N, K), generator=g, device="cuda").to(TDT[dtype]))
    ref = fl.k_gemm(x, tw)
    wide = torch.zeros((M, 2 * K), dtype=x.dtype, device="cuda")
    wide[:, :K] = x
    flat = torch.zeros(M * K + 1, dtype=x.dtype, device="cuda")
    flat[1:] = x.reshape(-1)
    for other in (wide[:, :K], flat[1:].view(M, K)):
        assert torch.equal(fl.k_gemm(other, tw), ref)


@pytest.mark.parametrize("dtype", [synth.DT_BF16, synth.DT_F16])
@pytest.mark.parametrize("group,block_rows,block_columns,M,N,K", [
    (32, 64, 64, 191, 130, 64), (32, 64, 128, 150, 6000, 64), (32, 128, 128, 131, 1000, 2048), (32, 128, 256, 257, 10000, 512),
    (32, 256, 256, 257, 2050, 8192), (64, 64, 128, 129, 33000, 288), (64, 128, 256, 257, 33000, 512), (64, 256, 256, 130, 50257, 1024)])
def test_gemm_of_more_than_128_rows_each_block_and_group_width(dtype, group, block_rows, block_columns, M, N, K):
    """One shape for every block and both widths of the layout's column groups, ragged in rows and columns; the shape's choice
    is asserted, so that a new rule cannot leave one out unnoticed.  Bound as above."""
    assert fl.binding.k_gemm_block(dtype, N, K, M) == (group, block_rows, block_columns)
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    x = torch.randn((M, K), generator=g, device="cuda").to(TDT[dtype])
    W = (torch.randn((N, K), generator=g, device="cuda") * 0.05).to(TDT[dtype])
    got = fl.k_gemm(x, W).double()
    xd, Wd = x.double(), W.double()
    assert torch.all((got - xd @ Wd.T).abs() <= 4e-6 * (xd.abs() @ Wd.abs().T) + 1e-30)


@pytest.mark.parametrize("dtype", [synth.DT_BF16, synth.DT_F16])
def test_gemm_of_256_row_blocks_with_three_k_blocks_in_the_last_turn(dtype):
    """The weight ring turns four k-blocks at a time; slices of 4n + 3 read row copies in the last turn that only that turn's own
    waits cover.  Every row of the three row blocks, the last one of a single live row tile: the bits of calls of at most 128 rows,
    which another kernel serves, and the bound as above."""
    M, N, K = 513, 4096, 2336
    assert fl.binding.k_gemm_block(dtype, N, K, M)[1:] == (256, 256) and fl.binding.k_gemm_plan(dtype, N, K)[1] % 4 == 3
    g = torch.Generator(device="cuda").manual_seed(4)
    x = torch.randn((M, K), generator=g, device="cuda").to(TDT[dtype])
    W = (torch.randn((N, K), generator=g, device="cuda") * 0.05).to(TDT[dtype])
    tw = fl.binding.TiledWeight(W)
    got = fl.k_gemm(x, tw)
    assert torch.equal(got, torch.cat([fl.k_gemm(x[m:m + 128].contiguous(), tw) for m in range(0, M, 128)]))
    xd, Wd = x.double(), W.double()
    assert torch.all((got.double() - xd @ Wd.T).abs() <= 4e-6 * (xd.abs() @ Wd.abs().T) + 1e-30)


def _at_element(t, at):
    """A copy of t that starts `at` elements behind a 16-byte boundary."""
    room = torch.zeros(t.numel() + 8, dtype=t.dtype, device="cuda")
    room[at:at + t.numel()].copy_(t.reshape(-1))
    return room[at:at + t.numel()].view(t.shape)


@pytest.mark.parametrize("dtype,M,N,K", [(synth.DT_F32, 5, 70, 96), (synth.DT_F32, 20, 260, 1056), (synth.DT_BF16, 9, 130, 160),
                                         (synth.DT_F16, 30, 98, 96), (synth.DT_BF16, 77, 320, 512), (synth.DT_BF16, 300, 200, 1024),
                                         (synth.DT_F16, 129, 24576, 256), (synth.DT_BF16, 260, 24576, 8192)])
def test_gemm_c_entry_takes_rows_at_any_element(dtype, M, N, K):
    """flover_k_gemm itself (the binding copies such rows) with x that starts off the 16-byte grid: the bits of aligned rows, at
    both group widths and on either side of 128 rows."""
    g = torch.Generator(device="cuda").manual_seed(M)
    x = torch.randn((M, K), generator=g, device="cuda").to(TDT[dtype])
    tw = fl.binding.TiledWeight((torch.randn((N, K), generator=g, device="cuda") * 0.05).to(TDT[dtype]))
    ref = fl.k_gemm(x, tw)
    n = C.c_uint64()
    lib = fl.load_library()
    assert lib.flover_k_gemm_workspace_bytes(dtype, M, N, K, C.byref(n)) == 0
    ws = torch.empty(int(n.value), dtype=torch.uint8, device="cuda")
    for at in (1, 2, 3):
        xo, y = _at_element(x, at), torch.empty_like(ref)
        assert xo.data_ptr() % 16
        assert lib.flover_k_gemm(dtype, xo.data_ptr(), tw.buf.data_ptr(), M, N, K, y.data_ptr(), ws.data_ptr(), n.value,
                                 torch.cuda.current_stream().cuda_stream) == 0
        assert torch.equal(y, ref), at


@pytest.mark.parametrize("dtype,M,N,K", [(synth.DT_F32, 9, 96, 64), (synth.DT_BF16, 20, 512, 2048), (synth.DT_F16, 200, 1030, 512)])
def test_gemm_result_at_any_float(dtype, M, N, K):
    """Results that start off the 16-byte grid hold the same bits, and nothing beside them is written."""
    g = torch.Generator(device="cuda").manual_seed(N)
    tw = fl.binding.TiledWeight(torch.randn((N, K), generator=g, device="cuda").to(TDT[dtype]))
    x = torch.randn((M, K), generator=g, device="cuda").to(TDT[dtype])
    ref = fl.k_gemm(x, tw)
    for at in (0, 1, 2, 3):
        room = torch.full((M * N + 8,), 7.0, dtype=torch.float32, device="cuda")
        assert torch.equal(fl.k_gemm(x, tw, room[at:at + M * N].view(M, N)), ref)
        assert torch.all(room[:at] == 7.0) and torch.all(room[at + M * N:] == 7.0)


@pytest.mark.parametrize("dtype,M,N,K", [(synth.DT_F32, 40, 256, 256), (synth.DT_F32, 7, 96, 1024), (synth.DT_BF16, 24, 40, 96),
                                         (synth.DT_F16, 150, 8192, 32)])
def test_gemm_result_may_share_memory_with_the_rows(dtype, M, N, K):
    """y over the memory that x lies in, at shapes taken in one slice (elsewhere the sums go through the workspace anyway):
    the same bits as into memory of its own."""
    assert fl.binding.k_gemm_plan(dtype, N, K)[0] == 1
    g = torch.Generator(device="cuda").manual_seed(M + N)
    tw = fl.binding.TiledWeight(torch.randn((N, K), generator=g, device="cuda").to(TDT[dtype]))
    x0 = torch.randn((M, K), generator=g, device="cuda").to(TDT[dtype])
    ref = fl.k_gemm(x0, tw)
    x_bytes, y_bytes = M * K * x0.element_size(), M * N * 4
    room = torch.zeros(x_bytes + y_bytes, dtype=torch.uint8, device="cuda")
    for x_at, y_at in ((0, 0), (0, x_bytes - 16), (y_bytes - 16, 0)):
        x = room[x_at:x_at + x_bytes].view(TDT[dtype]).view(M, K)
        x.copy_(x0)
        y = room[y_at:y_at + y_bytes].view(torch.float32).view(M, N)
        assert torch.equal(fl.k_gemm(x, tw, y), ref), (x_at, y_at)


# ---------------------------------------------------------------- gated MLP input (contraction + activation, one launch)

@pytest.mark.parametrize("M,F,K,context", [(7, 96, 512, 0), (100, 96, 512, 0), (200, 96, 512, 0), (200, 96, 4096, 1), (200, 1376, 512, 1), (300, 11008, 1024, 1)])
def test_gated_c_entry_takes_rows_at_any_element(M, F, K, context):
    """flover_k_gated_mlp itself with x off the 16-byte grid.  An iteration's rows give the bits of aligned rows, and so do a
    context pass's with slices; with one slice they are the iteration's, which add up K in two halves."""
    dtype = synth.DT_BF16
    g = torch.Generator(device="cuda").manual_seed(M)
    gw = fl.binding.GatedWeight(*[(torch.randn((F, K), generator=g, device="cuda") * 0.05).to(TDT[dtype]) for _ in range(2)])
    x = torch.randn((M, K), generator=g, device="cuda").to(TDT[dtype])
    halves = not context or fl.binding.k_gemm_plan(dtype, 2 * F, K, M)[0] == 1
    ref = fl.binding.k_gated_mlp(x, gw, context_pass=not halves)
    n = C.c_uint64()
    lib = fl.load_library()
    assert lib.flover_k_gated_workspace_bytes(dtype, M, F, K, C.byref(n)) == 0
    ws = torch.empty(max(int(n.value), 16), dtype=torch.uint8, device="cuda")
    for at in (1, 5):
        xo, act = _at_element(x, at), torch.empty_like(ref)
        assert lib.flover_k_gated_mlp(dtype, xo.data_ptr(), gw.buf.data_ptr(), M, F, K, context, act.data_ptr(), ws.data_ptr(), n.value,
                                      torch.cuda.current_stream().cuda_stream) == 0
        assert torch.equal(act, ref), at


@pytest.mark.parametrize("M", [5, 40, 100, 200])
def test_gated_mlp_result_may_share_memory_with_the_rows(M):
    """The activations over the memory that x lies in give the same bits as into memory of their own."""
    dtype, F, K = synth.DT_BF16, 512, 512
    g = torch.Generator(device="cuda").manual_seed(M)
    gw = fl.binding.GatedWeight(*[(torch.randn((F, K), generator=g, device="cuda") * 0.05).to(TDT[dtype]) for _ in range(2)])
    x0 = torch.randn((M, K), generator=g, device="cuda").to(TDT[dtype])
    for context in (False, True):
        ref = fl.binding.k_gated_mlp(x0, gw, context_pass=context)
        room = torch.zeros(M * K + 64, dtype=TDT[dtype], device="cuda")
        x, out = room[:M * K].view(M, K), room[64:].view(M, F)
        for o in (x, out):
            x.copy_(x0)
            assert torch.equal(fl.binding.k_gated_mlp(x, gw, o, context_pass=context), ref)


def _gated_reference(dtype, x, Wg, Wu):
    """fp64 silu(g) * u before the final rounding, and a bound on what fp32 accumulation may move it by."""
    g, u = orc.gemm(dtype, x, Wg), orc.gemm(dtype, x, Wu)
    eg = 4e-6 * (x.double().abs() @ Wg.double().abs().T).numpy()
    eu = 4e-6 * (x.double().abs() @ Wu.double().abs().T).numpy()
    sg = g / (1.0 + np.exp(-g))
    ref = sg * u
    slack = 1.1 * np.abs(u) * eg + np.abs(sg) * eu          # |d silu / dg| <= 1.1
    return ref, slack


def _gated_check(dtype, got, ref, slack):
    half_ulp = 2.0 ** -8 if dtype == synth.DT_BF16 else 2.0 ** -11       # relative, of the rounding to the model dtype
    tiny = 0.0 if dtype == synth.DT_BF16 else 2.0 ** -25                  # fp16 subnormal spacing
    assert np.all(np.abs(got - ref) <= half_ulp * np.abs(ref) * 1.001 + slack * (1 + half_ulp) + tiny + 1e-30)


@pytest.mark.parametrize("dtype", [synth.DT_BF16, synth.DT_F16])
@pytest.mark.parametrize("M,F,K", [(1, 32, 512), (7, 96, 512), (16, 352, 1024), (17, 64, 1024), (32, 160, 512),
                                   (33, 96, 2048), (64, 224, 512), (65, 128, 1024), (128, 96, 512), (129, 64, 512),
                                   (300, 160, 1024), (48, 96, 512), (90, 160, 1024), (110, 64, 512)])
def test_gated_mlp_matches_oracle(dtype, M, F, K):
    print("gated", dtype, M, F, K, flush=True)
    g = torch.Generator().manual_seed(300 + M + F)
    x = torch.randn((M, K), generator=g).to(TDT[dtype])
    Wg = (torch.randn((F, K), generator=g) * 0.05).to(TDT[dtype])
    Wu = (torch.randn((F, K), generator=g) * 0.05).to(TDT[dtype])
    ref, slack = _gated_reference(dtype, x, Wg, Wu)
    gw = fl.binding.GatedWeight(Wg.cuda(), Wu.cuda())
    got = fl.k_gated_mlp(x.cuda(), gw).cpu().double().numpy()
    _gated_check(dtype, got, ref, slack)


@pytest.mark.parametrize("dtype", [synth.DT_BF16, synth.DT_F16])
def test_gated_mlp_row_result_does_not_depend_on_other_rows(dtype):
    g = torch.Generator().manual_seed(6)
    K, F = 1024, 416
    x = torch.randn((300, K), generator=g).to(TDT[dtype]).cuda()
    gw = fl.binding.GatedWeight((torch.randn((F, K), generator=g) * 0.05).to(TDT[dtype]).cuda(),
                                (torch.randn((F, K), generator=g) * 0.05).to(TDT[dtype]).cuda())
    full = fl.k_gated_mlp(x, gw)
    for M in (1, 16, 17, 32, 33, 48, 64, 65, 81, 96, 100, 112, 128, 129, 200, 257):   # every count of 16-row tiles up to 8
        part = fl.k_gated_mlp(x[:M].contiguous(), gw)
        assert torch.equal(part, full[:M]), M
    alone = fl.k_gated_mlp(x[77:78].contiguous(), gw)
    assert torch.equal(alone[0], full[77])


@pytest.mark.parametrize("dtype", [synth.DT_BF16, synth.DT_F16])
@pytest.mark.parametrize("M,F,K", [(40, 96, 512), (130, 352, 1024), (300, 160, 1024), (600, 224, 512)])
def test_gated_mlp_of_a_context_pass_matches_oracle(dtype, M, F, K):
    g = torch.Generator().manual_seed(400 + M + F)
    x = torch.randn((M, K), generator=g).to(TDT[dtype])
    Wg = (torch.randn((F, K), generator=g) * 0.05).to(TDT[dtype])
    Wu = (torch.randn((F, K), generator=g) * 0.05).to(TDT[dtype])
    ref, slack = _gated_reference(dtype, x, Wg, Wu)
    gw = fl.binding.GatedWeight(Wg.cuda(), Wu.cuda())
    got = fl.k_gated_mlp(x.cuda(), gw, context_pass=True).cpu().double().numpy()
    _gated_check(dtype, got, ref, slack)


@pytest.mark.parametrize("M,context", [(8, False), (24, False), (48, False), (64, False), (72, False), (96, False),
                                       (112, False), (128, False), (300, True), (513, True), (1024, True)])
def test_gated_mlp_full_size_sampled_columns(M, context):
    """The 7B gate|up shape at row counts that select each variant of the one-launch form (1 to 8 row tiles); as a
    context pass: one slice with the activation as the 256-row-block kernel's epilogue (300, 513 and
    1024 rows, incl. ragged last blocks) -- sampled MLP columns from the oracle."""
    dtype, F, K = synth.DT_BF16, 11008, 4096
    print("gated full", M, context, flush=True)
    if context:
        from paper_2305_13484_amd.binding import k_gemm_plan
        # the plan of the plain 2F-column matrix is a lower bound of how attractive one slice is for the paired one
        print("slices of a plain matrix of this shape:", k_gemm_plan(dtype, 2 * F, K, M))
    g = torch.Generator(device="cuda").manual_seed(F + M)
    x = torch.randn((M, K), generator=g, device="cuda").to(TDT[dtype])
    Wg = (torch.randn((F, K), generator=g, device="cuda") * 0.02).to(TDT[dtype])
    Wu = (torch.randn((F, K), generator=g, device="cuda") * 0.02).to(TDT[dtype])
    got = fl.k_gated_mlp(x, fl.binding.GatedWeight(Wg, Wu), context_pass=context)
    cols = np.concatenate([np.random.default_rng(M).choice(F, size=24, replace=False), [0, 15, 16, F - 1]])
    ci = torch.as_tensor(cols, device="cuda").long()
    ref, slack = _gated_reference(dtype, x.cpu(), Wg[ci].cpu().contiguous(), Wu[ci].cpu().contiguous())
    _gated_check(dtype, got[:, ci].cpu().double().numpy(), ref, slack)


@pytest.mark.parametrize("dtype,F,K", [
    (synth.DT_BF16, 4128, 2560), (synth.DT_F16, 8192, 512), (synth.DT_BF16, 8224, 1536), (synth.DT_F16, 12288, 512), (synth.DT_BF16, 12320, 2560),
    (synth.DT_F16, 16384, 1536), (synth.DT_BF16, 16416, 2560), (synth.DT_F16, 20480, 512), (synth.DT_BF16, 20512, 1536)])
def test_gated_mlp_blocks_of_every_width(dtype, F, K):
    """First and last F of 2, 3, 4, 5 and 8 groups per block, the last block short or whole, K of one to five turns of the deepest weight
    ring in a half: sampled columns from the oracle, and at every count of row tiles the bits of the two launches that 129 rows take."""
    g = torch.Generator(device="cuda").manual_seed(F)
    x = torch.randn((129, K), generator=g, device="cuda").to(TDT[dtype])
    Wg, Wu = [(torch.randn((F, K), generator=g, device="cuda") * 0.05).to(TDT[dtype]) for _ in range(2)]
    gw = fl.binding.GatedWeight(Wg, Wu)
    full = fl.k_gated_mlp(x, gw)
    for M in (1, 16, 17, 33, 64, 65, 81, 97, 113, 128):
        print("gated width", F, M, flush=True)
        assert torch.equal(fl.k_gated_mlp(x[:M].contiguous(), gw), full[:M]), M
    cols = np.concatenate([np.random.default_rng(F).choice(F, size=20, replace=False), [0, 16, F - 17, F - 1]])
    ci = torch.as_tensor(cols, device="cuda").long()
    ref, slack = _gated_reference(dtype, x[:48].cpu(), Wg[ci].cpu().contiguous(), Wu[ci].cpu().contiguous())
    _gated_check(dtype, full[:48, ci].cpu().double().numpy(), ref, slack)


def test_gated_mlp_at_the_30b_shape_sampled_columns_and_row_invariance():
    """F = 17920, K = 6656, blocks of five groups: sampled MLP columns from the oracle, and every row count gives the same bits
    for a row."""
    dtype, F, K = synth.DT_BF16, 17920, 6656
    g = torch.Generator(device="cuda").manual_seed(30)
    x = torch.randn((100, K), generator=g, device="cuda").to(TDT[dtype])
    Wg = (torch.randn((F, K), generator=g, device="cuda") * 0.02).to(TDT[dtype])
    Wu = (torch.randn((F, K), generator=g, device="cuda") * 0.02).to(TDT[dtype])
    gw = fl.binding.GatedWeight(Wg, Wu)
    full = fl.k_gated_mlp(x, gw)
    for M in (8, 24, 48, 64, 65, 100):
        print("gated 30b", M, flush=True)
        assert torch.equal(fl.k_gated_mlp(x[:M].contiguous(), gw), full[:M]), M
    cols = np.concatenate([np.random.default_rng(3).choice(F, size=20, replace=False), [0, 16, F - 1]])
    ci = torch.as_tensor(cols, device="cuda").long()
    ref, slack = _gated_reference(dtype, x[:48].cpu(), Wg[ci].cpu().contiguous(), Wu[ci].cpu().contiguous())
    _gated_check(dtype, full[:48, ci].cpu().double().numpy(), ref, slack)


def test_gated_mlp_rejects_shapes_it_does_not_serve():
    lib = fl.load_library()
    assert lib.flover_k_gated_mlp(2, None, None, 4, 48, 512, 0, None, None, 0, None) == -1       # F not a multiple of 32
    assert lib.flover_k_gated_mlp(2, None, None, 4, 64, 256, 0, None, None, 0, None) == -1       # K not a multiple of 512
    assert lib.flover_k_gated_mlp(0, None, None, 4, 64, 512, 0, None, None, 0, None) == -1       # fp32


# ---------------------------------------------------------------- ragged decode attention

ATT_TOL = {synth.DT_F32: 2e-5, synth.DT_F16: 1.5e-3, synth.DT_BF16: 1e-2}   # |err| / max|ref row|: rounding of the output
                                                                            # to dtype (2^-11, 2^-8 half-ulps) + fp32 softmax


@pytest.mark.parametrize("dtype", [synth.DT_BF16, synth.DT_F16, synth.DT_F32])
@pytest.mark.parametrize("d", [64, 128])
def test_attention_matches_oracle(dtype, d):
    print("attention", dtype, d, flush=True)
    M, Cn, nh, S = 11, 14, 8, 700
    q, k, v, slots, lens = synth.attention_case(17 + d, M, Cn, nh, d, S, dtype, 1, S)
    lens[:5] = [1, 2, 255, 256, 257]       # single row, chunk boundaries
    lens[5] = S
    # rows at or beyond len hold garbage that must not be read into the result
    for s_, n_ in zip(slots.tolist(), lens.tolist()):
        k[s_, :, n_:] = float("nan")
        v[s_, :, n_:] = float("nan")
    pairs = [(m, h) for m in range(M) for h in range(nh)]
    ref = orc.attention(dtype, q, k, v, slots, lens, pairs).reshape(M, nh, d)
    got = fl.k_decode_attention(q.cuda(), k.cuda(), v.cuda(), slots, lens).cpu().double().numpy()
    assert np.isfinite(got).all()
    scale = np.abs(ref).max(axis=2, keepdims=True)
    assert (np.abs(got - ref) / scale).max() <= ATT_TOL[dtype]


def test_attention_row_result_does_not_depend_on_other_rows():
    dtype, d = synth.DT_BF16, 128
    M, Cn, nh, S = 9, 12, 4, 600
    q, k, v, slots, lens = synth.attention_case(3, M, Cn, nh, d, S, dtype, 1, S)
    qd, kd, vd = q.cuda(), k.cuda(), v.cuda()
    full = fl.k_decode_attention(qd, kd, vd, slots, lens)
    for m in range(M):
        one = fl.k_decode_attention(qd[m:m + 1].contiguous(), kd, vd, slots[m:m + 1], lens[m:m + 1])
        assert torch.equal(one[0], full[m])


@pytest.mark.parametrize("dtype,d", [(synth.DT_BF16, 128), (synth.DT_F16, 64), (synth.DT_F32, 64)])
def test_attention_rows_by_argument_by_list_and_by_copy_give_the_same_bits(dtype, d):
    """300 rows come as a list copied from the host, 256 and fewer as a kernel argument; in both a block takes all chunks of a row.  20 rows
    take a block per chunk and a merge, 16 without a second chunk no merge: a row's result is the same in all of them."""
    M, Cn, nh, S = 300, 301, 4, 1100
    q, k, v, slots, lens = synth.attention_case(31, M, Cn, nh, d, S, dtype, 1, S)
    lens[:4] = [1, 256, 257, S]
    lens[4:20] = np.minimum(lens[4:20], 256)
    qd, kd, vd = q.cuda(), k.cuda(), v.cuda()
    full = fl.k_decode_attention(qd, kd, vd, slots, lens)
    for lo, hi in ((0, 256), (0, 20), (4, 20), (3, 4), (0, 1)):
        part = fl.k_decode_attention(qd[lo:hi].contiguous(), kd, vd, slots[lo:hi], lens[lo:hi])
        assert torch.equal(part, full[lo:hi]), (lo, hi)


@pytest.mark.parametrize("dtype,d", [(synth.DT_BF16, 128), (synth.DT_F16, 64), (synth.DT_F32, 64)])
def test_attention_chunks_by_argument_and_by_list_give_the_same_bits(dtype, d):
    """A block per chunk and a merge: 256 rows of several chunks found by the argument's search (the call that cannot allocate), 300 from
    a list copied from the host (one row is of 17 chunks), against a block that takes all chunks of a row."""
    M, nh, S = 300, 4, 4400
    q, k, v, _, _ = synth.attention_case(d, 8, 8, nh, d, S, dtype, 1, 1, device="cuda", fill="all")
    q = torch.randn(M, nh, d, generator=torch.Generator().manual_seed(d)).to(TDT[dtype]).cuda()
    rng = np.random.default_rng(d)
    slots, lens = rng.integers(0, 8, size=M).astype(np.int32), rng.integers(1, 1101, size=M).astype(np.int32)
    rows = fl.k_decode_attention(q, k, v, slots, lens)
    lone = fl.k_decode_attention_noalloc(q[:256].contiguous(), k, v, slots[:256], lens[:256], torch.empty_like(q[:256]))
    assert torch.equal(lone, rows[:256])
    lens[290] = S
    listed = fl.k_decode_attention(q, k, v, slots, lens)
    assert torch.equal(listed[:290], rows[:290]) and torch.equal(listed[291:], rows[291:])
    assert torch.equal(listed[290:291], fl.k_decode_attention(q[290:291].contiguous(), k, v, slots[290:291], lens[290:291]))


@pytest.mark.parametrize("dtype,d,nh,M,hi", [
    (synth.DT_BF16, 128, 4, 1, 257), (synth.DT_BF16, 128, 4, 64, 768), (synth.DT_BF16, 128, 4, 65, 768),      # three chunks, 256 and 260 blocks
    (synth.DT_BF16, 128, 4, 64, 769), (synth.DT_F16, 64, 4, 64, 1024), (synth.DT_F16, 64, 4, 64, 1025),       # four and five chunks of short rows
    (synth.DT_F32, 128, 4, 3, 700), (synth.DT_F32, 64, 4, 200, 512),
    (synth.DT_F16, 64, 4, 199, 256), (synth.DT_F16, 64, 4, 200, 256), (synth.DT_F16, 64, 4, 256, 256),        # one chunk, 796 to 1024 waves
    (synth.DT_BF16, 64, 16, 63, 2048), (synth.DT_BF16, 64, 16, 64, 2048), (synth.DT_BF16, 64, 16, 64, 2305),     # 1008 and 1024 blocks; nine
    (synth.DT_BF16, 64, 16, 64, 4096), (synth.DT_F16, 64, 20, 52, 4097), (synth.DT_BF16, 64, 4, 300, 600)])   # sixteen and seventeen; a list
def test_attention_has_the_same_bits_in_blocks_of_rows_of_chunks_and_of_heads(dtype, d, nh, M, hi):
    """A block takes a (row, head) with all its chunks, one head of a chunk, or four heads of it with the merge in a launch of its own (what
    the call that cannot allocate always does): either side of every edge between them, against the last."""
    Cn = min(M, 16)
    q, k, v, slots, lens = synth.attention_case(M + hi, Cn, Cn, nh, d, hi, dtype, 1, hi, device="cuda", fill="all")
    rng = np.random.default_rng(M)
    qd = torch.randn(M, nh, d, generator=torch.Generator().manual_seed(5)).to(TDT[dtype]).cuda()
    slots, lens = rng.integers(0, Cn, size=M).astype(np.int32), rng.integers(1, hi + 1, size=M).astype(np.int32)
    lens[0] = hi
    got = fl.k_decode_attention(qd, k, v, slots, lens)
    part = 40                                  # its scratch does not hold the partial results of many long rows
    assert torch.equal(got, fl.k_decode_attention(qd, k, v, slots, lens))
    for lo in range(0, M, part):
        ref = fl.k_decode_attention_noalloc(qd[lo:lo + part].contiguous(), k, v, slots[lo:lo + part], lens[lo:lo + part],
                                            torch.empty_like(qd[lo:lo + part]))
        assert torch.equal(got[lo:lo + part], ref), lo


@pytest.mark.parametrize("hi,merges", [(200, False), (600, False), (4097, True)])
def test_attention_of_a_list_copies_row_lengths_only_for_the_merge(hi, merges):
    """More than 256 rows: slot | len go to the head of the workspace where a merge launch reads them, and nowhere else."""
    M, nh, d = 300, 4, 64
    q, k, v, _, _ = synth.attention_case(hi, 4, 4, nh, d, hi, synth.DT_BF16, 1, 1, device="cuda", fill="all")
    q = torch.randn(M, nh, d, generator=torch.Generator().manual_seed(1)).to(torch.bfloat16).cuda()
    rng = np.random.default_rng(hi)
    slots, lens = rng.integers(0, 4, size=M).astype(np.int32), rng.integers(1, min(hi, 900) + 1, size=M).astype(np.int32)
    lens[7] = hi
    ws = fl.binding.AttentionWorkspace(M, nh, d, hi)
    ws.buf.fill_(0x5a)
    got = fl.k_decode_attention(q, k, v, slots, lens, workspace=ws)
    head = ws.buf[:8 * M].cpu().numpy()
    assert np.array_equal(head.view(np.int32), np.concatenate([slots, lens])) if merges else (head == 0x5a).all()
    for lo in range(0, M, 60):
        assert torch.equal(got[lo:lo + 60], fl.k_decode_attention(q[lo:lo + 60].contiguous(), k, v, slots[lo:lo + 60], lens[lo:lo + 60])), lo


@pytest.mark.parametrize("M,hi", [(6, 200), (6, 600), (300, 100), (300, 600)])
def test_attention_output_may_share_memory_with_the_queries(M, hi):
    """The output over q itself and over its neighbouring rows, with and without second chunks, by argument and by list."""
    dtype, nh, d = synth.DT_BF16, 4, 128
    q, k, v, slots, lens = synth.attention_case(M, M, M, nh, d, hi, dtype, 1, hi)
    kd, vd = k.cuda(), v.cuda()
    ref = fl.k_decode_attention(q.cuda(), kd, vd, slots, lens)
    room = torch.zeros((M + 1, nh, d), dtype=TDT[dtype], device="cuda")
    for q_at, out_at in ((0, 0), (0, 1), (1, 0)):
        qd, out = room[q_at:q_at + M], room[out_at:out_at + M]
        qd.copy_(q)
        assert torch.equal(fl.k_decode_attention(qd, kd, vd, slots, lens, out), ref), (q_at, out_at)
        if M <= 256:
            qd.copy_(q)
            assert torch.equal(fl.k_decode_attention_noalloc(qd, kd, vd, slots, lens, out), ref), (q_at, out_at)


def test_attention_benchmark_shape_sampled_pairs():
    """Config 2's shape (256 live, 32 heads, head_dim 128, lengths U{1..4096}, bf16): sampled (row, head) outputs."""
    dtype, M, Cn, nh, d, S = synth.DT_BF16, 256, 256, 32, 128, 4096
    print("attention full size", flush=True)
    q, k, v, slots, lens = synth.attention_case(2, M, Cn, nh, d, S, dtype, 1, S, device="cuda", fill="all")
    got = fl.k_decode_attention(q, k, v, slots, lens)
    rng = np.random.default_rng(0)
    rows = np.concatenate([rng.choice(M, size=10, replace=False), [int(np.argmax(lens)), int(np.argmin(lens))]])
    heads = rng.integers(0, nh, size=len(rows))
    # a compact host cache holding just the sampled (slot, head) planes
    kk = torch.stack([k[slots[r], h] for r, h in zip(rows, heads)]).unsqueeze(1).cpu().contiguous()
    vv = torch.stack([v[slots[r], h] for r, h in zip(rows, heads)]).unsqueeze(1).cpu().contiguous()
    qq = torch.stack([q[r, h] for r, h in zip(rows, heads)]).unsqueeze(1).cpu().contiguous()
    ref = orc.attention(dtype, qq, kk, vv, np.arange(len(rows)), lens[rows], [(i, 0) for i in range(len(rows))])
    g = torch.stack([got[r, h] for r, h in zip(rows, heads)]).cpu().double().numpy()
    scale = np.abs(ref).max(axis=1, keepdims=True)
    assert (np.abs(g - ref) / scale).max() <= ATT_TOL[dtype]
    del k, v
    torch.cuda.empty_cache()


def test_attention_rejects_bad_arguments():
    q, k, v, slots, lens = synth.attention_case(1, 2, 3, 4, 64, 32, synth.DT_BF16, 1, 32)
    bad = lens.copy()
    bad[0] = 33
    with pytest.raises(fl.FloverError):
        fl.k_decode_attention(q.cuda(), k.cuda(), v.cuda(), slots, bad)
    bad = slots.copy()
    bad[1] = 3
    with pytest.raises(fl.FloverError):
        fl.k_decode_attention(q.cuda(), k.cuda(), v.cuda(), bad, lens)
    out = fl.k_decode_attention(q.cuda()[:0].contiguous(), k.cuda(), v.cuda(), slots[:0], lens[:0])   # empty batch
    assert out.shape[0] == 0


# ---------------------------------------------------------------- memory shuffle copy

@pytest.mark.parametrize("dtype", [synth.DT_BF16, synth.DT_F32])
def test_compact_is_bit_exact(dtype):
    L, Cn, nh, S, d = 3, 10, 4, 300, 64
    g = torch.Generator().manual_seed(9)
    cache = torch.randn((L, 2, Cn, nh, S, d), generator=g).to(TDT[dtype])
    src, dst, ln = [7, 9, 0, 8], [2, 3, 5, 4], [300, 1, 129, 0]
    ref = cache.clone()
    orc.compact(ref, L, Cn, nh, S, d, cache.element_size(), src, dst, ln)
    dev = cache.cuda()
    fl.k_compact(dev, src, dst, ln)
    assert torch.equal(dev.cpu().view(torch.uint8), ref.view(torch.uint8))
    # rows >= len of the destination and all other slots stay untouched
    assert torch.equal(dev.cpu()[:, :, 3, :, 1:], cache[:, :, 3, :, 1:])
    assert torch.equal(dev.cpu()[:, :, 1], cache[:, :, 1])


@pytest.mark.parametrize("n", [1, 64, 65])
def test_compact_moves_by_argument_and_by_copy(n):
    L, Cn, nh, S, d = 1, 140, 4, 24, 64
    cache = torch.randn((L, 2, Cn, nh, S, d), generator=torch.Generator().manual_seed(n)).to(torch.bfloat16)
    rng = np.random.default_rng(n)
    perm = rng.permutation(Cn)
    src, dst, ln = perm[:n].tolist(), perm[n:2 * n].tolist(), rng.integers(0, S + 1, size=n).tolist()
    ref = cache.clone()
    for a, b, m in zip(src, dst, ln):
        ref[:, :, b, :, :m] = cache[:, :, a, :, :m]
    dev = cache.cuda()
    fl.k_compact(dev, src, dst, ln)
    assert torch.equal(dev.cpu().view(torch.uint8), ref.view(torch.uint8))


def test_compact_rejects_overlapping_sets_and_empty_list():
    cache = torch.zeros((1, 2, 4, 4, 8, 64), dtype=torch.bfloat16, device="cuda")
    with pytest.raises(fl.FloverError):
        fl.k_compact(cache, [0, 1], [1, 2], [4, 4])
    with pytest.raises(fl.FloverError):
        fl.k_compact(cache, [0], [5], [4])
    fl.k_compact(cache, [], [], [])


def test_compact_benchmark_shape():
    """Config 2's cache (1 layer, 256 slots, 32 heads, 4096 x 128 bf16 = 16 GiB): 26 moves, checked by equality with
    the sources' snapshots and by checksums of every untouched slot."""
    print("compact full size", flush=True)
    L, Cn, nh, S, d = 1, 256, 32, 4096, 128
    cache = torch.empty((L, 2, Cn, nh, S, d), dtype=torch.bfloat16, device="cuda")
    gen = torch.Generator(device="cuda").manual_seed(4)
    for c in range(Cn):
        cache[0, :, c].copy_(torch.randn((2, nh, S, d), generator=gen, device="cuda"))
    rng = np.random.default_rng(4)
    perm = rng.permutation(Cn)
    src, dst = perm[:26].tolist(), perm[26:52].tolist()
    ln = rng.integers(1, S + 1, size=26).tolist()
    ln[0], ln[1] = S, 1
    before = [cache[:, :, s, :, :n].clone() for s, n in zip(src, ln)]
    tails = [cache[:, :, t, :, n:].clone() for t, n in zip(dst, ln)]
    sums = cache.view(torch.int16).to(torch.int32).sum(dim=(0, 1, 3, 4, 5))
    fl.k_compact(cache, src, dst, ln)
    for i, (s, t, n) in enumerate(zip(src, dst, ln)):
        assert torch.equal(cache[:, :, t, :, :n], before[i])
        assert torch.equal(cache[:, :, t, :, n:], tails[i])
    after = cache.view(torch.int16).to(torch.int32).sum(dim=(0, 1, 3, 4, 5))
    untouched = np.setdiff1d(np.arange(Cn), dst)
    assert torch.equal(after[untouched], sums[untouched])
    del cache
    torch.cuda.empty_cache()


def test_copy_probe_copies():
    src = torch.arange(1 << 20, dtype=torch.int32, device="cuda")
    dst = torch.zeros_like(src)
    fl.k_copy_probe(dst, src)
    torch.cuda.synchronize()
    assert torch.equal(dst, src)


@pytest.mark.parametrize("dtype,M,F,K", [(synth.DT_BF16, 129, 1376, 512), (synth.DT_F16, 515, 1376, 512), (synth.DT_BF16, 1000, 1376, 512),
                                         (synth.DT_F16, 260, 4096, 1536), (synth.DT_BF16, 300, 320, 3072), (synth.DT_F16, 530, 4064, 3072)])
def test_gated_windows_of_more_than_128_rows(dtype, M, F, K):
    """Rows of a fused iteration with narrow gate|up matrices: every block above 128 rows, rows on and off the 16-byte grid, with the room
    that flover_k_gated_workspace_bytes names, the room of two slices and no less; the bits of calls of at most 128 rows."""
    import paper_2305_13484_amd as fl
    lib = fl.load_library()
    g = torch.Generator(device="cuda").manual_seed(M + F)
    x = torch.randn((M, K), generator=g, device="cuda").to(TDT[dtype])
    w = [(torch.randn((F, K), generator=g, device="cuda") * 0.05).to(TDT[dtype]) for _ in range(2)]
    gw = fl.binding.GatedWeight(*w)
    ref = torch.cat([fl.binding.k_gated_mlp(x[m:m + 100].contiguous(), gw) for m in range(0, M, 100)])
    xd = x.double()
    exact = torch.nn.functional.silu(xd @ w[0].double().T) * (xd @ w[1].double().T)
    assert float((ref.double() - exact).norm() / exact.norm()) <= (6e-3 if dtype == synth.DT_BF16 else 8e-4)
    n = C.c_uint64()
    assert lib.flover_k_gated_workspace_bytes(dtype, M, F, K, C.byref(n)) == 0
    two = 2 * M * 2 * F * 4
    assert n.value >= two
    for at in (0, 1):
        rows = _at_element(x, at)
        for room in (int(n.value), two, two - 1):
            ws = torch.full((int(n.value) + 256,), 7, dtype=torch.uint8, device="cuda")
            out = torch.full((M * F + 64,), 3.0, dtype=x.dtype, device="cuda")
            rc = lib.flover_k_gated_mlp(dtype, rows.data_ptr(), gw.buf.data_ptr(), M, F, K, 0, out.data_ptr(), ws.data_ptr(), room,
                                        torch.cuda.current_stream().cuda_stream)
            assert rc == (0 if room >= two else -3)
            torch.cuda.synchronize()
            if rc == 0:
                assert torch.equal(out[:M * F].view(M, F), ref), (at, room)
                assert bool((ws[room:] == 7).all()) and bool((out[M * F:] == 3.0).all())


@pytest.mark.parametrize("dtype", [synth.DT_BF16, synth.DT_F16])
@pytest.mark.parametrize("N,K", [(1617, 608), (3071, 1024), (7000, 2560), (64, 512)])
def test_gemm_sums_in_one_launch_have_the_bits_of_two(dtype, N, K):
    """Four slices of K, the last one shorter at 608, rows that end inside a group of four columns: one launch up to the row counts where it
    is the shorter way and two above, rows on and off the 16-byte grid, y at any float.  A row's bits do not depend on the call; the bound
    is that of the other GEMM tests."""
    import paper_2305_13484_amd as fl
    lib = fl.load_library()
    assert fl.binding.k_gemm_plan(dtype, N, K)[0] == 4
    g = torch.Generator(device="cuda").manual_seed(N)
    x = torch.randn((65, K), generator=g, device="cuda").to(TDT[dtype])
    W = (torch.randn((N, K), generator=g, device="cuda") * 0.05).to(TDT[dtype])
    tw = fl.binding.TiledWeight(W)
    full = fl.k_gemm(x, tw)
    xd, Wd = x.double(), W.double()
    assert torch.all((full.double() - xd @ Wd.T).abs() <= 4e-6 * (xd.abs() @ Wd.abs().T) + 1e-30)
    n = C.c_uint64()
    assert lib.flover_k_gemm_workspace_bytes(dtype, 65, N, K, C.byref(n)) == 0
    ws = torch.empty(int(n.value), dtype=torch.uint8, device="cuda")
    for M in sorted({1, 16, 17, 33, 60000 // K, 60000 // K + 1, 64} & set(range(1, 65))):
        for at in (0, 1):
            rows = _at_element(x[:M], at)
            for y_at in range(4):
                y = torch.full((M * N + 8,), 3.0, device="cuda")
                assert lib.flover_k_gemm(dtype, rows.data_ptr(), tw.buf.data_ptr(), M, N, K, y[y_at:].data_ptr(), ws.data_ptr(), ws.numel(),
                                         torch.cuda.current_stream().cuda_stream) == 0
                torch.cuda.synchronize()
                assert torch.equal(y[y_at:y_at + M * N].view(M, N), full[:M]), (M, at, y_at)
                assert bool((y[:y_at] == 3.0).all()) and bool((y[y_at + M * N:] == 3.0).all())
