"""GPU parity: the score-table path (contexts too long to be rebuilt on the fly) for every code size that the streaming kernel
requests as a whole - 4, 6, 8 and 16 pairs, whole-vector and chunked - by query heads per workgroup (1, 2, 4) and rounds per
chunk, with lengths that end inside a round, and for codes whose sizes differ (loaded where they are used)."""
import numpy as np
import pytest
import torch

import oracle
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
