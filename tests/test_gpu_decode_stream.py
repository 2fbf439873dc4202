"""GPU parity: the score-table path (contexts too long to be rebuilt on the fly) for every code size that the streaming kernel
requests as a whole - 4, 6, 8 and 16 pairs, whole-vector and chunked - by query heads per workgroup (1, 2, 4) and rounds per
chunk, with lengths that end inside a round, and for codes whose sizes differ (loaded where they are used)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2412_11741_amd as csr
from tests.test_gpu_decode import TOL_F16_OUT, _case, _check, _chunked_case, _run, _u16
from tests import test_gpu_decode_rope as rope

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,Hq,Hkv,T,N,sK,sV", [
    (33, 2, 2, 1025, 256, 4, 4),        # a round and one token
    (2, 2, 2, 16500, 300, 4, 4),
    (1, 2, 1, 70001, 512, 4, 4),
    (1, 4, 1, 70001, 512, 4, 4),        # four heads
    (1, 8, 1, 530000, 128, 4, 4),       # four heads, more tokens than one pass of 16-wave chunks over the chip
    (3, 3, 3, 5000, 512, 6, 6),
    (1, 2, 1, 44001, 1000, 6, 6),
    (1, 4, 1, 44001, 512, 6, 6),
    (1, 4, 1, 17001, 512, 16, 16),      # halves of a code
    (1, 6, 1, 20001, 256, 16, 16),
    (1, 4, 1, 530000, 128, 16, 16),
    (1, 4, 1, 36001, 512, 8, 12),       # codes of different sizes
])
def test_whole_codes(B, Hq, Hkv, T, N, sK, sV):
    args = _case(71, B, Hq, Hkv, T, N, sK, sV)
    lens = np.full(B, T, dtype=np.int32)
    lens[-1] -= T // 3 if B > 1 else 0
    ref = oracle.decode_attn(*args[:2], *(a if i % 3 else _u16(a) for i, a in enumerate(args[2:])), seq_lens=lens)
    _check(_run(*args, seq_lens=lens), ref, TOL_F16_OUT, f"stream {B} {Hq} {Hkv} {T} {sK} {sV}")


@pytest.mark.parametrize("Hq,snK,sK,snV,sV,T", [
    (1, 1, 4, 2, 2, 70001), (2, 1, 6, 2, 3, 45001), (4, 1, 8, 2, 4, 36001), (4, 1, 16, 2, 8, 18001), (2, 2, 4, 4, 2, 36001),
    (4, 4, 4, 1, 16, 18001), (1, 2, 3, 2, 3, 45001), (4, 2, 4, 2, 3, 45001),
])
def test_chunked_codes(Hq, snK, sK, snV, sV, T):
    q, DK, iK, cK, DV, iV, cV = _chunked_case(72, 1, Hq, 1, T, 256, snK, sK, snV, sV)
    keys = (DK, iK, cK) if snK > 1 else (DK[:, 0], np.ascontiguousarray(iK[:, :, :, 0]), np.ascontiguousarray(cK[:, :, :, 0]))
    vals = (DV, iV, cV) if snV > 1 else (DV[:, 0], np.ascontiguousarray(iV[:, :, :, 0]), np.ascontiguousarray(cV[:, :, :, 0]))
    ref = oracle.decode_attn_chunked(q, DK, _u16(iK), cK, DV, _u16(iV), cV)
    _check(_run(q, *keys, *vals), ref, TOL_F16_OUT, f"stream chunks {Hq} {snK} {sK} {snV} {sV}")


@pytest.mark.parametrize("Hq,N,sK,snV,sV,T", [
    (1, 256, 4, 2, 2, 70001), (1, 256, 8, 2, 4, 36001), (2, 512, 16, 1, 16, 18001), (4, 256, 8, 1, 4, 44001), (4, 256, 8, 2, 8, 22001),
    (1, 256, 8, 2, 3, 40001),
])
def test_values_of_rotary_keys(Hq, N, sK, snV, sV, T):
    args = rope._case(73, 1, Hq, 1, T, N, sK, sV, snV=snV)
    rope._check(rope._run(args, 10000.0, 0, 3), oracle.decode_attn_rope(*args, 10000.0, 0, 3), f"stream rope {Hq} {sK} {snV} {sV}")


def test_both_halves_of_a_code_are_sampled():
    # values in two chunks of 8 pairs, one with coefficients 1024 times the other's: the scatter's unit, chosen from a sample of
    # the coefficients, must not depend on which half of the code the large ones are in.  The two calls are each other's
    # mirror image, so the bits are equal - unless one of them has had to repeat its scatter in 64 bits
    Hq, T, N, s = 4, 20000, 256, 8
    q, DK, iK, cK, DV, iV, cV = _chunked_case(74, 1, Hq, 1, T, N, 1, 16, 2, s)
    cV[:, :, :, 1] = (cV[:, :, :, 1].astype(np.float32) / 1024).astype(np.float16)
    keys = (DK[:, 0], np.ascontiguousarray(iK[:, :, :, 0]), np.ascontiguousarray(cK[:, :, :, 0]))
    one = _run(q, *keys, DV, iV, cV, out_dtype=torch.float32)
    two = _run(q, *keys, *(np.ascontiguousarray(np.flip(a, ax)) for a, ax in ((DV, 1), (iV, 3), (cV, 3))), out_dtype=torch.float32)
    assert np.array_equal(one, np.concatenate([two[..., 64:], two[..., :64]], axis=-1))


@pytest.mark.parametrize("B,Hkv,G,T,N,s,rope_base", [
    (13, 8, 4, 60000, 256, 4, 0.0),       # 8-wave shape, four chunks of the plan
    (6, 32, 1, 40000, 128, 4, 0.0),       # 16-wave shape, one query head
    (13, 8, 2, 40000, 128, 4, 0.0),       # two query heads
    (7, 16, 1, 40000, 128, 5, 0.0),       # codes that are not requested as a whole: one kernel, with and without the cut
    (64, 1, 4, 50000, 128, 4, 0.0),       # as many sequences as a wave has lanes
    (65, 1, 4, 50000, 128, 4, 0.0),       # one more: the plan's chunks
    (9, 8, 4, 16000, 128, 4, 10000.0),    # rotary keys, a group
    (13, 8, 2, 18000, 128, 4, 10000.0),   # rotary keys, two query heads
    (5, 32, 1, 12000, 64, 4, 10000.0),    # rotary keys, one query head
])
def test_long_sequences_are_cut_by_their_own_lengths(B, Hkv, G, T, N, s, rope_base):
    # lengths of 0, 1, the edges of the plan's chunks and rounds, out of range on both sides; sampled pairs against the oracle
    d = 128
    gen = torch.Generator(device="cuda")
    gen.manual_seed(75)
    unit = lambda *sh: (lambda a: (a / a.norm(dim=-1, keepdim=True)).half())(torch.randn(*sh, device="cuda", generator=gen))
    idx = lambda: torch.randint(0, N, (B, Hkv, T, s), device="cuda", generator=gen, dtype=torch.int32).to(torch.int16)
    coef = lambda: (torch.randn(B, Hkv, T, s, device="cuda", generator=gen) * 3).half()
    q, DK, DV = torch.randn(B, Hkv * G, d, device="cuda", generator=gen).half(), unit(Hkv, N, d), unit(Hkv, N, d)
    ik, ck, iv, cv = idx(), coef(), idx(), coef()
    edges = [T, 0, 1, T // 4, T // 4 + 1, T // 2, -5, T + 70000, T - 1, 512, 1025, 4097, 3 * T // 4]
    lens = np.array([edges[(7 * b) % len(edges)] for b in range(B)], dtype=np.int32)
    out = csr.csr_decode_attn(q, DK, ik, ck, DV, iv, cv, seq_lens=torch.from_numpy(lens).cuda(), out_dtype=torch.float16,
                              rope_base=rope_base)
    torch.cuda.synchronize()
    valid = np.clip(lens, 0, T)
    n = lambda t: t.cpu().numpy()
    for b in range(min(B, 13)):
        if valid[b] == 0:
            assert not n(out[b]).any()
            continue
        h = (3 * b) % Hkv
        one = [n(a) for a in (q[b:b + 1, h * G:(h + 1) * G], DK[h:h + 1], ik[b:b + 1, h:h + 1], ck[b:b + 1, h:h + 1], DV[h:h + 1],
                              iv[b:b + 1, h:h + 1], cv[b:b + 1, h:h + 1])]
        ref = oracle.decode_attn_rope(*one, rope_base, 0, 0, seq_lens=valid[b:b + 1]) if rope_base else \
            oracle.decode_attn(*one, seq_lens=valid[b:b + 1])
        _check(n(out[b:b + 1, h * G:(h + 1) * G]), ref, TOL_F16_OUT, f"cut by length {B} {Hkv} {G} {T}: sequence {b}, {lens[b]} tokens")
    # and the lengths of every sequence full: the same as no lengths at all
    full = csr.csr_decode_attn(q, DK, ik, ck, DV, iv, cv, seq_lens=torch.full((B,), T, dtype=torch.int32, device="cuda"), rope_base=rope_base)
    none = csr.csr_decode_attn(q, DK, ik, ck, DV, iv, cv, rope_base=rope_base)
    assert torch.allclose(full.float(), none.float(), rtol=2e-3, atol=2e-3)
