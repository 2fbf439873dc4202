"""GPU parity of the streaming kernels on contexts that are too long to be rebuilt on the fly, for what the other files test at
lengths that decode_direct.hip now takes: rotary keys with gathered rows and with either pair layout, the scatter's resolution
check, ragged and empty sequences in chunks, reproducibility, the static scratch and capture.  Every test asserts its form."""
import numpy as np
import pytest
import torch

import oracle
import paper_2412_11741_amd as csr
from tests import parity
from tests.test_gpu_decode import TOL_F16_OUT, TOL_F32_OUT, _case, _check, _chunked_case, _run, _u16
from tests import test_gpu_decode_rope as rope

pytestmark = pytest.mark.gpu


def _table(B, Hkv, T, pairs, f32=False):
    assert parity.decode_form(B, Hkv, T, pairs, f32) == "table"


@pytest.mark.parametrize("Hq,N,sK,sV,snV,layout,T", [
    # rows gathered from device memory
    (1, 768, 8, 8, 1, 0, 33001), (1, 4096, 8, 8, 1, 1, 33001), (1, 1024, 16, 16, 1, 0, 17001), (1, 1024, 4, 4, 1, 1, 66001),
    (1, 8192, 8, 24, 1, 1, 17001), (1, 640, 12, 6, 1, 0, 30001),
    (2, 1024, 8, 4, 1, 0, 44001), (2, 768, 16, 4, 2, 1, 22501), (2, 1024, 4, 16, 1, 1, 27001),
    (4, 4096, 8, 8, 1, 1, 33001), (4, 640, 4, 6, 1, 0, 53001), (4, 1024, 16, 24, 1, 0, 14001), (8, 1024, 12, 4, 1, 1, 33001),
    # the dictionary in LDS: interleaved pairs, and value codes that are not requested as a whole
    (1, 256, 8, 8, 1, 1, 33001), (2, 512, 16, 8, 1, 1, 22001), (4, 256, 8, 4, 2, 1, 33001), (8, 128, 12, 3, 1, 1, 36001),
    (3, 384, 4, 16, 1, 1, 27001), (1, 256, 8, 24, 1, 0, 17001), (4, 256, 8, 32, 1, 1, 14001), (2, 256, 4, 12, 2, 0, 19001),
])
def test_rotary_keys(Hq, N, sK, sV, snV, layout, T):
    _table(2, 1, T // 2, sK + snV * sV)
    args = rope._case(81, 2, Hq, 1, T // 2, N, sK, sV, snV)
    lens = np.array([T // 2, T // 5], dtype=np.int32)
    out = rope._run(args, 10000.0, layout, 11, seq_lens=lens)
    ref = oracle.decode_attn_rope(*args, 10000.0, layout, 11, seq_lens=lens)
    rope._check(out, ref, f"streaming rope Hq{Hq} N{N} s{sK}/{snV}x{sV} layout {layout}")


@pytest.mark.parametrize("G,dtype", [(1, "f32"), (1, "f16"), (4, "f16")])
def test_an_outlier_coefficient_in_the_sample_and_a_diffuse_tail(G, dtype):
    # one sampled value coefficient far above the typical one, nearly all of the attention mass on a flat tail of tokens
    # far below the maximum score: the tail's adds are tiny against a unit fitted to the outlier, which the resolution check
    # of the 32-bit scatter has to catch
    T, N, s = (16400 if dtype == "f32" else 33000), 4096, 8
    _table(1, 1, T, 2 * s, dtype == "f32")
    q, DK, idxK, coefK, DV, idxV, coefV = _case(82, 1, G, 1, T, N, s, s, dtype=dtype, itype="i32" if dtype == "f32" else "i16")
    q[:] = q[:, :1]
    coefK[...] = 0
    dot = float(q[0, 0].astype(np.float64) @ DK[0, int(idxK[0, 0, 0, 0]) & 0xffff].astype(np.float64)) / np.sqrt(128.0)
    coefK[0, 0, 0, 0] = 9.0 / (np.sign(dot) * max(abs(dot), 1e-3))      # token 0 leads by a score of 9
    coefV[0, 0, 5, 3] = 2.0 ** 14 * 3.0
    out = _run(q, DK, idxK, coefK, DV, idxV, coefV, out_dtype=torch.float32)
    wide = (lambda a: a) if dtype == "f32" else _u16
    _check(out, oracle.decode_attn(q, DK, wide(idxK), coefK, DV, wide(idxV), coefV), TOL_F32_OUT, f"outlier, diffuse tail {G} {dtype}")


@pytest.mark.parametrize("Hq,snK,sK,snV,sV,T", [(1, 1, 8, 2, 4, 15000), (4, 2, 4, 2, 8, 11000), (2, 8, 4, 4, 8, 4200), (4, 4, 8, 8, 4, 4200)])
def test_ragged_and_empty_sequences_in_chunks(Hq, snK, sK, snV, sV, T):
    _table(4, 1, T, snK * sK + snV * sV)
    q, DK, iK, cK, DV, iV, cV = _chunked_case(83, 4, Hq, 1, T, 256, snK, sK, snV, sV)
    keys = (DK, iK, cK) if snK > 1 else (DK[:, 0], np.ascontiguousarray(iK[:, :, :, 0]), np.ascontiguousarray(cK[:, :, :, 0]))
    lens = np.array([T, 0, 1, T // 2 + 1], dtype=np.int32)
    out = _run(q, *keys, DV, iV, cV, seq_lens=lens)
    ref = np.zeros(q.shape)
    for b in (0, 2, 3):
        n = lens[b]
        ref[b:b + 1] = oracle.decode_attn_chunked(q[b:b + 1], DK, _u16(iK[b:b + 1, :, :n]), cK[b:b + 1, :, :n], DV, _u16(iV[b:b + 1, :, :n]), cV[b:b + 1, :, :n])
    assert np.all(out[1] == 0)
    _check(out[[0, 2, 3]], ref[[0, 2, 3]], TOL_F16_OUT, f"ragged chunks {Hq} {snK} {snV}")


@pytest.mark.parametrize("Hq,s,base", [(4, 8, 0.0), (1, 16, 0.0), (2, 8, 10000.0)])
def test_same_bits_again_on_the_static_scratch_and_in_a_captured_call(Hq, s, base):
    B, Hkv, T, N = 2, 2, 8700, 256
    _table(B, Hkv, T, 2 * s)
    args = [torch.from_numpy(a).cuda() for a in rope._case(84, B, Hq * Hkv, Hkv, T, N, s, s)]
    lens = torch.tensor([T, T // 3], dtype=torch.int32, device="cuda")
    more = dict(seq_lens=lens, rope_base=base, rope_pos0=5 if base else 0)
    q, out = args[0], torch.empty_like(args[0])
    desc = csr.decode_desc(q, args[1], args[2], args[3], args[5], rope_base=base, rope_pos0=more["rope_pos0"])
    ws = torch.empty(csr.csr_decode_workspace_bytes(desc), dtype=torch.uint8, device="cuda")

    def call():
        return csr.csr_decode_attn(*args, out=out, workspace=ws, **more)
    want = call().clone()
    assert want.abs().sum() > 0 and torch.equal(call(), want)
    static = torch.zeros_like(out)
    csr.csr_decode_attn_static(*args, static, **more)
    assert torch.equal(static, want)
    graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        with torch.cuda.graph(graph, stream=side):
            call()
    torch.cuda.current_stream().wait_stream(side)
    for seed in (1, 2, 3):
        q.copy_(torch.randn(q.shape, generator=torch.Generator().manual_seed(seed)).half())
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        got = out.clone()
        out.zero_()
        assert torch.equal(call(), got) and not torch.equal(got, want)
