"""GPU parity: attention over short contexts, where the cached tokens are rebuilt on the fly (decode_direct.hip), at the edges
of its teams and chunks; and the score-table path's own checks at contexts above that form's limit."""
import numpy as np
import pytest
import torch

import oracle
import paper_2412_11741_amd as csr
from paper_2412_11741_amd import binding, synth
from tests.test_gpu_decode import TOL_F16_OUT, TOL_F32_OUT, _case, _check, _chunked_case, _run, _u16
from tests import test_gpu_decode_rope as rope

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,Hq,Hkv,T,N,sK,sV,dtype", [
    (1, 1, 1, 1, 32, 1, 1, "f16"),        # one token, one pair
    (2, 6, 2, 15, 100, 3, 5, "f16"),      # fewer tokens than teams, odd codes, three query heads
    (1, 5, 1, 17, 300, 6, 2, "f16"),      # one token past a round, five query heads, codes read in words
    (3, 16, 2, 333, 512, 8, 16, "f16"),   # eight query heads, a second block of value pairs
    (2, 4, 2, 700, 1024, 32, 12, "f16"),  # the longest codes
    (40, 2, 2, 16, 256, 8, 8, "f16"),     # one chunk per sequence: no second launch
    (1, 2, 1, 6000, 512, 4, 4, "f32"),    # fp32 throughout, many chunks
    (2, 7, 1, 90, 96, 7, 9, "f32"),
])
def test_short_contexts(B, Hq, Hkv, T, N, sK, sV, dtype):
    args = _case(61, B, Hq, Hkv, T, N, sK, sV, dtype=dtype, itype="i16" if dtype == "f16" else "i32")
    lens = np.full(B, T, dtype=np.int32)
    if B > 1:
        lens[0], lens[-1] = 0, max(1, T // 2)
    out = _run(*args, seq_lens=lens)
    ref = oracle.decode_attn(*args[:2], *(a if i % 3 else _u16(a) if dtype == "f16" else a for i, a in enumerate(args[2:])), seq_lens=lens)
    assert B == 1 or np.all(out[0] == 0)
    _check(out[lens > 0], ref[lens > 0], TOL_F16_OUT if dtype == "f16" else TOL_F32_OUT, f"direct {B} {Hq} {Hkv} {T}")


@pytest.mark.parametrize("chunks", [2, 16, 17, 64, 65, 128, 129, 256, 257, 513, 1024])
def test_the_combine_of_any_number_of_chunks(chunks):
    # one head: chunks of 16 tokens; the shorter sequence leaves its last chunks without tokens, never written
    T = 16 * chunks - 5
    B, Hq = (2, 2) if chunks <= 256 else (1, 1)   # two query heads: at most 256 chunks for each of two sequences; one: 1024
    args = _case(65, B, Hq, 1, T, 256, 2, 2)
    lens = np.full(B, T, dtype=np.int32)
    lens[-1] = 16 * (chunks // 2) + 1
    if chunks >= 16:   # the scratch is what so many partial outputs and their weights take
        t = [torch.from_numpy(a) for a in args]
        up = lambda n: (n + 255) // 256 * 256  # noqa: E731
        assert csr.csr_decode_workspace_bytes(csr.decode_desc(t[0], t[1], t[2], t[3], t[5])) == up(B * Hq * chunks * 512) + up(B * Hq * chunks * 8)
    ref = oracle.decode_attn(*args[:2], *(a if i % 3 else _u16(a) for i, a in enumerate(args[2:])), seq_lens=lens)
    _check(_run(*args, seq_lens=lens), ref, TOL_F16_OUT, f"combine of {chunks} chunks")


@pytest.mark.parametrize("snK,sK,snV,sV", [(1, 8, 2, 4), (2, 4, 4, 2), (8, 2, 8, 3)])
def test_short_contexts_in_chunks(snK, sK, snV, sV):
    q, DK, iK, cK, DV, iV, cV = _chunked_case(62, 2, 4, 2, 150, 256, snK, sK, snV, sV)
    whole = (DK, iK, cK) if snK > 1 else (DK[:, 0], np.ascontiguousarray(iK[:, :, :, 0]), np.ascontiguousarray(cK[:, :, :, 0]))
    out = _run(q, *whole, DV, iV, cV)
    _check(out, oracle.decode_attn_chunked(q, DK, _u16(iK), cK, DV, _u16(iV), cV), TOL_F16_OUT, f"direct chunks {snK} {snV}")


@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("Hq,T,pos0", [(2, 33, 0), (8, 500, 100000)])
def test_short_contexts_with_rotary_keys(layout, Hq, T, pos0):
    args = rope._case(63, 2, Hq, 2, T, 256, 8, 4, snV=2)
    rope._check(rope._run(args, 10000.0, layout, pos0), oracle.decode_attn_rope(*args, 10000.0, layout, pos0), f"direct rope {layout} {Hq}")


@pytest.mark.parametrize("what", ["hot", "growing", "tiny", "f32", "odd", "rope"])
def test_the_score_table_path_above_the_limit(what):
    # the scatter's unit, its checks and the wide form (see test_gpu_decode.py), and code widths of the streaming kernel
    B, Hq, Hkv, T, N, s = 2, 4, 1, 36000, 512, 8
    if what == "odd":
        args = list(_case(64, B, Hq, Hkv, T, 1000, 6, 10))
    elif what == "rope":
        args = rope._case(64, B, Hq, Hkv, T, 256, 8, 6)
        return rope._check(rope._run(args, 10000.0, 0, 5), oracle.decode_attn_rope(*args, 10000.0, 0, 5), "rope above the limit")
    else:
        f32 = what == "f32"
        args = list(_case(64, B, Hq, Hkv, T, N, s, s, dtype="f32" if f32 else "f16", itype="i32" if f32 else "i16"))
    if what == "hot":
        args[3][...], args[5][...], args[6][...] = 0, 3, np.float16(60000.0)
    elif what == "growing":
        args[6][:, :, :1024] = 0
        args[6][:, :, 1024:] *= np.float16(512.0)
    elif what == "tiny":
        args[6][...] = (args[6].astype(np.float32) * 2.0 ** -20).astype(np.float16)
    out = _run(*args, out_dtype=torch.float32)
    _check(out, oracle.decode_attn(*args), TOL_F32_OUT, f"table path, {what}")


def test_a_workspace_of_the_score_table_form_is_enough():
    # one sized for a longer context on a small dictionary holds the table and the histograms, not the short form's partial sums
    B, Hq, Hkv, T, N, s = 1, 4, 1, 2000, 64, 4
    args = _case(65, B, Hq, Hkv, T, N, s, s)

    def scratch(tokens):
        return binding.csr_decode_workspace_bytes(binding.DecodeDesc(
            B=B, Hq=Hq, Hkv=Hkv, T=tokens, d=128, N=N, sK=s, sV=s, q_dtype=1, dict_dtype=1, coef_dtype=1, idx_dtype=1, out_dtype=1))
    longer = 70000   # 560000 gathered rows
    assert scratch(longer) < scratch(T)
    out = csr.csr_decode_attn(*(torch.from_numpy(a).cuda() for a in args), workspace=torch.empty(scratch(longer), dtype=torch.uint8, device="cuda"))
    ref = oracle.decode_attn(*args[:2], *(a if i % 3 else _u16(a) for i, a in enumerate(args[2:])))
    _check(out.cpu().numpy(), ref, TOL_F16_OUT, "table form for lack of scratch")


@pytest.mark.parametrize("B,G,Hkv,T,snK", [
    (1, 1, 2, 40, 1),      # several chunks
    (1, 3, 1, 40, 2),      # keys in chunks, a query group
    (40, 1, 32, 16, 1),    # one chunk: no second launch
])
def test_a_score_of_minus_infinity_has_weight_zero(B, G, Hkv, T, snK):
    # an overflowed key coefficient against the query's sign: the token drops out, as with a coefficient of -6e4
    # (whose weight, exp(-6e4 * 0.1), is zero in any precision); a sequence of such tokens only gives zero
    N, s = 256, 4
    q, DK, iK, cK, DV, iV, cV = _chunked_case(66, B, Hkv * G, Hkv, T, N, snK, s, 1, 4)
    groups = q.reshape(B, Hkv, G, -1)
    groups[:] = groups[:, :, :1] * np.arange(1, G + 1, dtype=np.float16)[:, None]
    far = cK.copy()
    dc = 128 // snK
    for b in range(B):
        for h in range(Hkv):
            dots = DK[h, 0].astype(np.float64) @ q[b, h * G, :dc].astype(np.float64)
            n = int(np.abs(dots).argmax())
            assert abs(dots[n]) / np.sqrt(128) > 0.1
            for t in (range(T) if b == B - 1 and B > 1 else (0, T // 2, T - 1)):
                iK[b, h, t, 0, 1] = n
                cK[b, h, t, 0, 1] = -np.inf * np.sign(dots[n])
                far[b, h, t, 0, 1] = -6e4 * np.sign(dots[n])

    def plain(*codes):
        return [a if snK > 1 else np.ascontiguousarray(a[:, :, :, 0]) for a in codes]
    DKx, DVx, vals = (DK if snK > 1 else DK[:, 0]), DV[:, 0], [np.ascontiguousarray(a[:, :, :, 0]) for a in (iV, cV)]
    out = _run(q, DKx, *plain(iK, cK), DVx, *vals)
    some = slice(0, B - 1 if B > 1 else 1)
    if snK > 1:
        ref = oracle.decode_attn_chunked(q, DK, _u16(iK), far, DV, _u16(iV), cV)
    else:
        ref = oracle.decode_attn(q, DKx, *(_u16(a) if i == 0 else a for i, a in enumerate(plain(iK, far))), DVx, _u16(vals[0]), vals[1])
    _check(out[some], ref[some], TOL_F16_OUT, f"minus infinity {B} {G} {Hkv} {snK}")
    assert B == 1 or np.all(out[-1] == 0)


@pytest.mark.parametrize("what", ["f16", "f32", "rope"])
def test_an_index_outside_the_dictionary_reads_inside_it(what):
    # one sequence's codes hold stale indices: the call ends, they count as the last atom, the other sequences do not notice
    B, Hq, Hkv, T, N = 3, 4, 2, 77, 256
    if what == "rope":
        args, bad = list(rope._case(67, B, Hq, Hkv, T, N, 12, 4)), np.array([256, 40000, 65535], dtype=np.uint16).view(np.int16)
    else:
        args = list(_case(67, B, Hq, Hkv, T, N, 8, 12, dtype=what, itype="i16" if what == "f16" else "i32"))
        bad = np.array([256, 40000, 65535], dtype=np.uint16).view(np.int16) if what == "f16" else np.array([256, -1, 2 ** 30], dtype=np.int32)

    def run(a):
        return rope._run(a, 10000.0, 0, 5) if what == "rope" else _run(*a)
    clean = run(args)
    stale, last = [a.copy() for a in args], [a.copy() for a in args]
    for side in (2, 5):
        stale[side][1, :, ::7, -1] = np.resize(bad, stale[side][1, :, ::7, -1].shape)
        last[side][1, :, ::7, -1] = N - 1
    out = run(stale)
    assert np.array_equal(out[[0, 2]], clean[[0, 2]]) and not np.array_equal(out[1], clean[1])
    assert np.array_equal(out, run(last))
