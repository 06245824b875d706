"""flover_k_decode_attention_noalloc (the entry point for callers that cannot allocate) against
flover_k_decode_attention on the same inputs, through the C ABI: same kernels, so the outputs must be equal bit for
bit; two calls in a row on the library's one scratch array, the second with a smaller input."""
import ctypes as C

import numpy as np
import pytest
import torch

import flover_synth as synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fl():
    assert torch.cuda.is_available(), "these tests need the MI355X"
    import paper_2305_13484_amd as m
    m.load_library()
    return m


@pytest.mark.parametrize("dtype,d", [(synth.DT_BF16, 128), (synth.DT_F16, 64), (synth.DT_F32, 128)])
def test_noalloc_attention_equals_the_workspace_entry_point_twice_in_a_row(fl, dtype, d):
    print("noalloc attention", dtype, d, flush=True)
    Cn, nh, S = 40, 8, 700
    # first call: 37 rows, lengths across the 256-position chunk boundaries; second call: 5 rows, short
    for M, lo, hi, seed in ((37, 1, S, 5), (5, 1, 90, 6)):
        q, k, v, slots, lens = synth.attention_case(seed + d, M, Cn, nh, d, S, dtype, lo, hi)
        if M > 6:
            lens[:6] = [1, 2, 255, 256, 257, S]
        qd, kd, vd = q.cuda(), k.cuda(), v.cuda()
        ref = fl.k_decode_attention(qd, kd, vd, slots, lens)
        out = torch.full_like(ref, float("nan"))
        got = fl.k_decode_attention_noalloc(qd, kd, vd, slots, lens, out)
        torch.cuda.synchronize()
        assert torch.isfinite(got.float()).all()
        assert torch.equal(got.view(torch.uint8), ref.view(torch.uint8)), (M, dtype, d)


def test_noalloc_attention_limits_and_bad_arguments(fl):
    dtype, d, nh = synth.DT_BF16, 128, 32
    # more rows than one call serves
    q, k, v, slots, lens = synth.attention_case(1, 257, 4, 4, 64, 16, dtype, 1, 16)
    slots = np.arange(257, dtype=np.int32) % 4
    out = torch.empty_like(q, device="cuda")
    with pytest.raises(fl.FloverError, match="at most 256 rows"):
        fl.k_decode_attention_noalloc(q.cuda(), k.cuda(), v.cuda(), slots, lens, out)
    # a workspace beyond the built-in scratch: 256 rows x 16 chunks x 32 heads x (128 + 2) floats = 68 MB
    S, M = 4096, 256
    q = torch.zeros((M, nh, d), dtype=torch.bfloat16, device="cuda")
    kv = torch.zeros((1, nh, S, d), dtype=torch.bfloat16, device="cuda")
    with pytest.raises(fl.FloverError, match="exceeds the built-in scratch"):
        fl.k_decode_attention_noalloc(q, kv, kv, np.zeros(M, np.int32), np.full(M, S, np.int32), torch.empty_like(q))
    # the same checks as the workspace entry point
    q, k, v, slots, lens = synth.attention_case(1, 2, 3, 4, 64, 32, dtype, 1, 32)
    bad = lens.copy()
    bad[0] = 33
    with pytest.raises(fl.FloverError):
        fl.k_decode_attention_noalloc(q.cuda(), k.cuda(), v.cuda(), slots, bad, torch.empty_like(q, device="cuda"))
    out = fl.k_decode_attention_noalloc(q.cuda()[:0].contiguous(), k.cuda(), v.cuda(), slots[:0], lens[:0],
                                        torch.empty_like(q[:0], device="cuda"))
    assert out.shape[0] == 0
    # and it still works after the refused calls
    qd, kd, vd = q.cuda(), k.cuda(), v.cuda()
    ref = fl.k_decode_attention(qd, kd, vd, slots, lens)
    got = fl.k_decode_attention_noalloc(qd, kd, vd, slots, lens, torch.empty_like(ref))
    assert torch.equal(got, ref)


class _KernelNode(C.Structure):              # hipKernelNodeParams
    _fields_ = [("block", C.c_uint32 * 3), ("extra", C.c_void_p), ("func", C.c_void_p), ("grid", C.c_uint32 * 3), ("params", C.c_void_p),
                ("lds", C.c_uint32)]


def _captured_grids(call):
    """Grids of the kernels that `call` enqueues on the current stream, in order; any other node fails the test."""
    path = next(line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64" in line)
    hip = C.CDLL(path)
    stream, graph, n = C.c_void_p(torch.cuda.current_stream().cuda_stream), C.c_void_p(), C.c_size_t()
    assert hip.hipStreamBeginCapture(stream, 1) == 0
    try:
        call()
    finally:
        rc = hip.hipStreamEndCapture(stream, C.byref(graph))
    assert rc == 0
    assert hip.hipGraphGetNodes(graph, None, C.byref(n)) == 0
    nodes = (C.c_void_p * n.value)()
    assert hip.hipGraphGetNodes(graph, nodes, C.byref(n)) == 0
    grids = []
    for node in nodes:
        p = _KernelNode()
        assert hip.hipGraphKernelNodeGetParams(C.c_void_p(node), C.byref(p)) == 0
        grids.append(tuple(p.grid))
    assert hip.hipGraphDestroy(graph) == 0
    return grids


@pytest.mark.parametrize("M,hi", [(1, 256), (1, 700), (9, 256), (48, 700), (200, 1500)])
def test_noalloc_attention_launches_one_block_row_per_chunk(fl, M, hi):
    """The streaming kernel's grid holds the rows' chunks of 256 positions and nothing else, and where no row has a second
    one it is the only launch: no block without work and no launch that only prepares another."""
    nh, d = 8, 64
    q, k, v, slots, lens = synth.attention_case(M, M, M, nh, d, hi, synth.DT_BF16, 1, hi)
    qd, kd, vd = q.cuda(), k.cuda(), v.cuda()
    out = torch.empty_like(qd)
    ref = fl.k_decode_attention_noalloc(qd, kd, vd, slots, lens, out).clone()
    with torch.cuda.stream(torch.cuda.Stream()):
        grids = _captured_grids(lambda: fl.k_decode_attention_noalloc(qd, kd, vd, slots, lens, out))
    chunks = int(((lens + 255) // 256).sum())
    assert grids[0] == (chunks, nh // 4, 1)
    assert len(grids) == (1 if chunks == M else 2)
    assert torch.equal(fl.k_decode_attention_noalloc(qd, kd, vd, slots, lens, out), ref)


@pytest.mark.parametrize("M,nh,long,rest,one_launch", [
    (64, 16, [4096], 100, False), (64, 16, [2048], 256, False),                  # 5.9 chunks a unit for 16, 4.9 for 8
    (64, 16, [1024, 600], 256, True), (64, 16, [1152, 600], 256, False),         # 69 chunks, 4.3 a unit, for 4 and for 5
    (64, 16, [769] * 64, 256, True), (128, 16, [2048], 100, True)])              # alike; 8.9 for 8
def test_a_block_takes_a_whole_row_only_while_the_longest_ends_with_the_rest(fl, M, nh, long, rest, one_launch):
    """1024 and more (row, head) blocks: one launch while the longest row has at most a compute unit's share of all chunks, else its chunks
    go to units of their own and a merge follows; the same bits in both."""
    d = 64
    rng = np.random.default_rng(M + len(long))
    q, k, v, slots, lens = synth.attention_case(M + len(long), M, M, nh, d, max(long), synth.DT_BF16, 1, rest, device="cuda", fill="all")
    lens[rng.permutation(M)[:len(long)]] = long
    out, ws = torch.empty_like(q), fl.binding.AttentionWorkspace(M, nh, d, max(long))
    got = fl.k_decode_attention(q, k, v, slots, lens, out, ws).clone()
    with torch.cuda.stream(torch.cuda.Stream()):
        grids = _captured_grids(lambda: fl.k_decode_attention(q, k, v, slots, lens, out, ws))
    assert (int(((lens + 255) // 256).sum()) * nh >= (max(long) + 255) // 256 * 256) == one_launch
    assert len(grids) == (1 if one_launch else 2)
    for lo in range(0, M, 32):                     # two launches, whatever the lengths
        ref = fl.k_decode_attention_noalloc(q[lo:lo + 32].contiguous(), k, v, slots[lo:lo + 32], lens[lo:lo + 32],
                                            torch.empty_like(q[lo:lo + 32]))
        assert torch.equal(got[lo:lo + 32], ref), lo


@pytest.mark.parametrize("dtype,d,nh,chunks,one_wave", [
    (synth.DT_F16, 64, 16, [1] * 60, True), (synth.DT_F32, 64, 4, [1] * 256, True),                             # one chunk per row: 960, 1024 waves
    (synth.DT_F16, 64, 4, [4] * 47 + [8], True), (synth.DT_F16, 64, 4, [4] * 47 + [9], False),                  # 784 and 788 waves
    (synth.DT_F16, 128, 16, [4] * 16, False), (synth.DT_F16, 128, 16, [4] * 15 + [5], True),                    # 1024 and 1040
    (synth.DT_F16, 64, 16, [8] * 23, True), (synth.DT_F16, 64, 16, [8] * 22 + [9], False),                      # 2944 and 2960, of eight and of nine chunks
    (synth.DT_F16, 64, 16, [9] * 16, True), (synth.DT_F16, 64, 12, [11] * 17 + [10], False),                    # 2304 and 2364: a last round of 1.3 times
    (synth.DT_F32, 128, 4, [9] * 82, True), (synth.DT_BF16, 128, 4, [9] * 82, False),                           # 2952 waves, rows of 512 and of 256 bytes
    (synth.DT_F16, 64, 8, [17] * 22, False)])
def test_attention_blocks_of_one_wave_and_of_four_either_side_of_every_line(fl, dtype, d, nh, chunks, one_wave):
    """The streaming kernel's grid is (heads, chunks) where a block is one wave, (chunks, heads / 4) where it has four; the same bits."""
    M, most = len(chunks), max(chunks)
    rng = np.random.default_rng(M)
    Cn = min(M, 12)
    q, k, v, _, _ = synth.attention_case(M + most, Cn, Cn, nh, d, 256 * most, dtype, 1, 1, device="cuda", fill="all")
    q = torch.randn(M, nh, d, generator=torch.Generator().manual_seed(M)).to(q.dtype).cuda()
    slots = rng.integers(0, Cn, size=M).astype(np.int32)
    lens = (256 * np.array(chunks) - rng.integers(0, 256, size=M)).astype(np.int32)
    out, ws = torch.empty_like(q), fl.binding.AttentionWorkspace(M, nh, d, 256 * most)
    got = fl.k_decode_attention(q, k, v, slots, lens, out, ws).clone()
    with torch.cuda.stream(torch.cuda.Stream()):
        grids = _captured_grids(lambda: fl.k_decode_attention(q, k, v, slots, lens, out, ws))
    assert grids[0] == ((nh, sum(chunks), 1) if one_wave else (sum(chunks), nh // 4, 1))
    assert len(grids) == (1 if most == 1 else 2)
    for lo in range(0, M, 20):                     # blocks of four, whatever the chunks
        ref = fl.k_decode_attention_noalloc(q[lo:lo + 20].contiguous(), k, v, slots[lo:lo + 20], lens[lo:lo + 20],
                                            torch.empty_like(q[lo:lo + 20]))
        assert torch.equal(got[lo:lo + 20], ref), lo
