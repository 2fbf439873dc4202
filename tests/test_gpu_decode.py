"""GPU parity: csr_decode_attn (through the C ABI) against the oracle's dense-reconstruction attention."""
import numpy as np
import pytest
import torch

import oracle
import paper_2412_11741_amd as csr
from paper_2412_11741_amd import synth
from tests import parity

pytestmark = pytest.mark.gpu

# Relative L2 error per (sequence, query head).  Inputs are identical bits on both sides; the GPU
# accumulates in fp32 (score sums of <= 32 terms, histogram sums over T tokens, 2 N-term dot
# products), which stays near 1e-5; fp16 output adds a 2^-11 rounding per element (~3e-4).
TOL_F32_OUT = 1e-3
TOL_F16_OUT = 2e-3


def _run(q, DK, idxK, coefK, DV, idxV, coefV, scale=0.0, seq_lens=None, out_dtype=None):
    g = lambda a: torch.from_numpy(a).cuda()
    sl = None if seq_lens is None else torch.from_numpy(np.asarray(seq_lens, dtype=np.int32)).cuda()
    out = csr.csr_decode_attn(g(q), g(DK), g(idxK), g(coefK), g(DV), g(idxV), g(coefV), scale=scale,
                              seq_lens=sl, out_dtype=out_dtype)
    torch.cuda.synchronize()
    return out.cpu().numpy()


def _check(out, ref, tol, what=""):
    rel, mx = parity.assert_decode_close(out, ref, tol, what)
    print(f"[decode parity] {what} max rel L2 {rel.max():.2e}, max element error / peak {mx:.2e}")


def _case(seed, B, Hq, Hkv, T, N, sK, sV, dtype="f16", itype="i16"):
    d = 128
    q = synth.queries(seed, B, Hq, d, dtype)
    DK = synth.dictionary(seed, "dict_k", Hkv, N, d, dtype)
    DV = synth.dictionary(seed, "dict_v", Hkv, N, d, dtype)
    idxK, coefK = synth.random_codes(seed, 0, B, Hkv, T, sK, N, dtype, itype)
    idxV, coefV = synth.random_codes(seed, 1, B, Hkv, T, sV, N, dtype, itype)
    return q, DK, idxK, coefK, DV, idxV, coefV


def test_tiny_config_on_the_oracles_own_codes_fp32():
    w = synth.WORKLOADS["tiny"]
    DK = synth.dictionary(0, "dict_k", 1, w.n_atoms, w.d, "f32")
    DV = synth.dictionary(0, "dict_v", 1, w.n_atoms, w.d, "f32")
    XK = synth.vectors(0, "keys", 1, w.tokens, w.d, "f32", outliers=w.key_outliers)
    XV = synth.vectors(0, "values", 1, w.tokens, w.d, "f32")
    iK, cK = oracle.mp_encode(XK[0], DK[0], w.s)
    iV, cV = oracle.mp_encode(XV[0], DV[0], w.s)
    idxK, idxV = iK[None, None].astype(np.int32), iV[None, None].astype(np.int32)
    coefK, coefV = cK[None, None].astype(np.float32), cV[None, None].astype(np.float32)
    q = synth.queries(0, 1, 1, w.d, "f32")
    out = _run(q, DK, idxK, coefK, DV, idxV, coefV)
    ref = oracle.decode_attn(q, DK, idxK, coefK, DV, idxV, coefV)
    _check(out, ref, TOL_F32_OUT, "tiny")
    # the codes approximate the dense cache: attention on codes is close to attention on X itself
    dense = oracle.decode_attn(q, np.eye(w.d)[None], np.tile(np.arange(w.d, dtype=np.int32), (1, 1, w.tokens, 1)),
                               XK[None].astype(np.float64), np.eye(w.d)[None],
                               np.tile(np.arange(w.d, dtype=np.int32), (1, 1, w.tokens, 1)), XV[None].astype(np.float64))
    assert np.linalg.norm(ref - dense) < np.linalg.norm(dense)      # loose: sanity only


@pytest.mark.parametrize("B,Hq,Hkv,T,N,sK,sV", [
    (3, 8, 2, 3000, 4096, 8, 8),      # GQA group 4, ragged T, several chunks
    (2, 4, 4, 1025, 8192, 16, 16),    # MHA, N = 8192, one token past a block step
    (2, 4, 2, 2500, 4096, 8, 4),      # group 2, value codes shorter than key codes (s = 4)
    (1, 8, 1, 5000, 2048, 8, 8),      # group 8 = two slices of 4
    (2, 6, 2, 700, 1000, 5, 3),       # group 3, odd pair counts, N not a multiple of 64
    (1, 1, 1, 1, 64, 1, 1),           # one token, one pair
    (70, 2, 1, 300, 512, 8, 8),       # more sequences than one query tile
])
def test_fp16_codes_shapes(B, Hq, Hkv, T, N, sK, sV):
    args = _case(10, B, Hq, Hkv, T, N, sK, sV)
    out = _run(*args)
    ref = oracle.decode_attn(*args)
    _check(out, ref, TOL_F16_OUT, f"B{B} Hq{Hq} Hkv{Hkv} T{T} N{N} s{sK}/{sV}")


def test_fp32_everything_int32_indices_and_explicit_scale():
    args = _case(11, 2, 4, 2, 1500, 1024, 8, 8, "f32", "i32")
    out = _run(*args, scale=0.05)
    ref = oracle.decode_attn(*args, scale=0.05)
    _check(out, ref, TOL_F32_OUT, "fp32/int32")


def test_fp16_inputs_fp32_output():
    args = _case(12, 2, 8, 2, 2000, 4096, 8, 8)
    out = _run(*args, out_dtype=torch.float32)
    assert out.dtype == np.float32
    _check(out, oracle.decode_attn(*args), TOL_F32_OUT, "f16 in / f32 out")


def test_sequence_lengths_including_empty_and_full():
    B, T = 5, 2600
    args = _case(13, B, 4, 2, T, 2048, 8, 8)
    lens = np.array([T, 0, 1, 1024, 2047], dtype=np.int32)
    out = _run(*args, seq_lens=lens)
    ref = oracle.decode_attn(*args, seq_lens=lens)
    assert np.all(out[1] == 0)
    _check(out, ref, TOL_F16_OUT, "seq_lens")


def test_zero_tokens_give_zero_output():
    args = _case(14, 2, 4, 2, 0, 256, 8, 8)
    out = _run(*args)
    assert out.shape == (2, 4, 128) and np.all(out == 0)


def test_repeated_atoms_inside_codes_and_hot_atoms():
    # All tokens hit the same few atoms: worst case for the LDS histogram atomics.
    B, Hq, Hkv, T, N, s = 1, 4, 1, 4096, 256, 8
    q, DK, idxK, coefK, DV, idxV, coefV = _case(15, B, Hq, Hkv, T, N, s, s)
    idxK[..., 1] = idxK[..., 0]
    idxV[...] = (idxV.view(np.uint16) % 3).astype(np.uint16).view(np.int16)
    out = _run(q, DK, idxK, coefK, DV, idxV, coefV)
    _check(out, oracle.decode_attn(q, DK, idxK, coefK, DV, idxV, coefV), TOL_F16_OUT, "hot atoms")


def test_large_scores_stay_finite_and_running_max_rescaling_is_exact():
    # Scores grow along the sequence, so the running maximum moves in every block step.
    B, Hq, Hkv, T, N, s = 1, 2, 1, 6000, 512, 8
    q, DK, idxK, coefK, DV, idxV, coefV = _case(16, B, Hq, Hkv, T, N, s, s, "f32", "i32")
    ramp = np.linspace(0.1, 4.0, T, dtype=np.float32)[None, None, :, None]
    coefK = (np.abs(coefK) * ramp).astype(np.float32)
    out = _run(q, DK, idxK, coefK, DV, idxV, coefV, scale=3.0)
    ref = oracle.decode_attn(q, DK, idxK, coefK, DV, idxV, coefV, scale=3.0)
    _check(out, ref, TOL_F32_OUT, "ramp")


def test_long_context_shape_sampled_pairs():
    # Long-context configuration (N = 8192, s = 16, T = 32768, batch 4), 4 of its 32 KV heads;
    # every (sequence, head) output is checked against the oracle.
    w = synth.WORKLOADS["long_context"]
    args = _case(17, w.batch, 4, 4, w.tokens, w.n_atoms, w.s, w.s)
    out = _run(*args)
    _check(out, oracle.decode_attn(*args), TOL_F16_OUT, "long context x4 heads")


def test_gqa_llama3_shape_sampled_pairs():
    # GQA configuration (8 KV heads x group 4, T = 131072, batch 8) cut to 2 sequences x 2 KV heads.
    w = synth.WORKLOADS["gqa_llama3_8b"]
    args = _case(18, 2, 8, 2, w.tokens, w.n_atoms, w.s, w.s)
    out = _run(*args)
    _check(out, oracle.decode_attn(*args), TOL_F16_OUT, "gqa x2x2")


def test_llama7b_layer_full_decode_all_heads():
    # The benchmark's decode call: 32 KV heads = 32 query heads, 4096 cached tokens, N = 4096, s = 8, batch 1.
    w = synth.WORKLOADS["llama7b_layer"]
    args = _case(19, w.batch, w.hq, w.hkv, w.tokens, w.n_atoms, w.s, w.s)
    out = _run(*args)
    _check(out, oracle.decode_attn(*args), TOL_F16_OUT, "llama7b layer, all heads")


def _full_launch_sampled(name, picks):
    """The whole configuration in one call (the launch bench.py times), random codes drawn on the GPU;
    the oracle recomputes the sampled (sequence, KV head) pairs from the bits copied back."""
    w = synth.WORKLOADS[name]
    B, Hkv, Hq, T, N, d, s = w.batch, w.hkv, w.hq, w.tokens, w.n_atoms, w.d, w.s
    G = Hq // Hkv
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(20)
    unit = lambda *sh: (lambda a: (a / a.norm(dim=-1, keepdim=True)).half())(torch.randn(*sh, device=dev, generator=gen))
    idx = lambda: torch.randint(0, N, (B, Hkv, T, s), device=dev, generator=gen, dtype=torch.int32).to(torch.int16)
    coef = lambda: (torch.randn(B, Hkv, T, s, device=dev, generator=gen) * 3).half()
    q, DK, DV = torch.randn(B, Hq, d, device=dev, generator=gen).half(), unit(Hkv, N, d), unit(Hkv, N, d)
    ik, ck, iv, cv = idx(), coef(), idx(), coef()
    out = csr.csr_decode_attn(q, DK, ik, ck, DV, iv, cv)
    torch.cuda.synchronize()
    assert torch.isfinite(out.float()).all()
    h_ = lambda t: t.cpu().numpy()
    for b, h in picks:
        ref = oracle.decode_attn(h_(q[b:b + 1, h * G:(h + 1) * G]), h_(DK[h:h + 1]), h_(ik[b:b + 1, h:h + 1]),
                                 h_(ck[b:b + 1, h:h + 1]), h_(DV[h:h + 1]), h_(iv[b:b + 1, h:h + 1]),
                                 h_(cv[b:b + 1, h:h + 1]))
        _check(h_(out[b:b + 1, h * G:(h + 1) * G]), ref, TOL_F16_OUT, f"{name} full launch, sequence {b} KV head {h}")


def test_long_context_full_launch_sampled():
    _full_launch_sampled("long_context", [(0, 0), (3, 31), (2, 17)])


def test_gqa_llama3_full_launch_sampled():
    _full_launch_sampled("gqa_llama3_8b", [(0, 0), (7, 7), (4, 3)])


def test_four_query_heads_long_context_shape_ragged_lengths_and_a_hot_atom():
    # 8 sequences x 8 KV heads x 4 query heads with more than 32768 cached tokens run the streaming kernel's
    # 8-wave shape (32 rounds of 512 tokens per chunk).  Ragged lengths cut chunks at every kind of boundary; in
    # sequence 4 every value pair sits on one atom with the largest fp16 coefficients, which the 32-bit histogram
    # cannot hold (the scatter has to notice and repeat itself in the wide form).  Codes are drawn on the GPU; the
    # oracle recomputes sampled (sequence, KV head) pairs from the bits copied back.
    B, Hkv, G, T, N, d, s = 8, 8, 4, 36000, 4096, 128, 8
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(27)
    unit = lambda *sh: (lambda a: (a / a.norm(dim=-1, keepdim=True)).half())(torch.randn(*sh, device=dev, generator=gen))
    idx = lambda: torch.randint(0, N, (B, Hkv, T, s), device=dev, generator=gen, dtype=torch.int32).to(torch.int16)
    coef = lambda: (torch.randn(B, Hkv, T, s, device=dev, generator=gen) * 3).half()
    q, DK, DV = torch.randn(B, Hkv * G, d, device=dev, generator=gen).half(), unit(Hkv, N, d), unit(Hkv, N, d)
    ik, ck, iv, cv = idx(), coef(), idx(), coef()
    ck[4] = 0
    iv[4] = 7
    cv[4] = 60000.0
    lens = np.array([T, 1, 0, 20000, T - 1, 32769, 16385, T], dtype=np.int32)
    sl = torch.from_numpy(lens).to(dev)
    out = csr.csr_decode_attn(q, DK, ik, ck, DV, iv, cv, seq_lens=sl, out_dtype=torch.float32)
    torch.cuda.synchronize()
    assert torch.isfinite(out).all() and torch.all(out[2] == 0)
    h_ = lambda t: t.cpu().numpy()
    for b, h in [(0, 0), (4, 3), (5, 7), (1, 2), (6, 1), (3, 5), (7, 7)]:
        ref = oracle.decode_attn(h_(q[b:b + 1, h * G:(h + 1) * G]), h_(DK[h:h + 1]), h_(ik[b:b + 1, h:h + 1]),
                                 h_(ck[b:b + 1, h:h + 1]), h_(DV[h:h + 1]), h_(iv[b:b + 1, h:h + 1]),
                                 h_(cv[b:b + 1, h:h + 1]), seq_lens=lens[b:b + 1])
        _check(h_(out[b:b + 1, h * G:(h + 1) * G]), ref, TOL_F32_OUT, f"long four-head shape, sequence {b} KV head {h}")


@pytest.mark.parametrize("B,Hq,Hkv,T,N", [
    (4, 4, 1, 20000, 256),     # 16 pairs per KV head, 20 chunks: batches of 8 chunk histograms with a tail of 4
    (17, 2, 2, 3000, 128),     # 17 pairs: one block of pairs with 15 empty rows, a single 128-atom slice
    (33, 1, 1, 1500, 384),     # 33 pairs: a second block with one pair
    (9, 8, 2, 2600, 1024),     # 36 pairs per KV head from groups of four query heads
])
def test_many_pairs_per_kv_head_take_the_matrix_core_product(B, Hq, Hkv, T, N):
    # With 16 or more (sequence, query head) pairs per KV head the D_V product runs on the matrix cores in fp32;
    # some sequences are empty or short (their chunks have weight zero and histograms that were never written).
    args = _case(28, B, Hq, Hkv, T, N, 8, 8)
    lens = np.full(B, T, dtype=np.int32)
    lens[1] = 0
    lens[2] = 1
    lens[B - 1] = T // 2 + 3
    out = _run(*args, seq_lens=lens, out_dtype=torch.float32)
    assert np.all(out[1] == 0)
    _check(out, oracle.decode_attn(*args, seq_lens=lens), TOL_F32_OUT, f"matrix-core D_V product, {B * Hq // Hkv} pairs per KV head")


@pytest.mark.parametrize("B,Hq,Hkv,T,N", [
    (2, 1, 1, 17000, 130),     # 2 pairs per KV head, 17 chunks; two atoms in the last slice
    (1, 3, 1, 33000, 100),     # 3: more than eight chunks a lane's turn, a slice that is not full
    (5, 1, 1, 8000, 1000),     # 5: two launches' worth of four
    (8, 8, 8, 1100, 4096),     # 8
    (3, 20, 4, 3000, 257),     # 15, five query heads per KV head
    (1, 4, 1, 130000, 64),     # 127 chunks: two a lane in the last sum
    (17, 1, 1, 2100, 200),     # 16 pairs and more, where the atoms are no whole slices for the matrix cores: 17, two launches' worth of eight and one
    (11, 12, 4, 1500, 320),    # 33, three query heads per KV head
    (16, 8, 1, 1100, 1000),    # 128
])
def test_few_pairs_per_kv_head_take_the_product_from_registers(B, Hq, Hkv, T, N):
    args = _case(33, B, Hq, Hkv, T, N, 8, 8)
    lens = None if B == 1 else np.resize([T, 0, T // 2, 1, T - 1, 1025, 64, T // 3], B).clip(0, T).astype(np.int32)
    out = _run(*args, seq_lens=lens, out_dtype=torch.float32)
    _check(out, oracle.decode_attn(*args, seq_lens=lens), TOL_F32_OUT, f"{B * Hq // Hkv} pairs per KV head")
    assert lens is None or not out[1].any()


def test_decode_is_bit_reproducible():
    # Histogram sums are integer, partial outputs are added in a fixed order: same inputs, same bits.
    args = _case(22, 2, 8, 2, 5000, 4096, 8, 8)
    a, b = _run(*args), _run(*args)
    assert np.array_equal(a.view(np.uint16), b.view(np.uint16))


def test_sequence_longer_than_the_supported_maximum_is_refused():
    q = torch.zeros(1, 1, 128, dtype=torch.float16, device="cuda")
    D = torch.zeros(1, 64, 128, dtype=torch.float16, device="cuda")
    T = (1 << 20) + 1
    idx = torch.zeros(1, 1, T, 1, dtype=torch.int16, device="cuda")
    coef = torch.zeros(1, 1, T, 1, dtype=torch.float16, device="cuda")
    with pytest.raises(csr.CsrError) as e:
        csr.csr_decode_attn(q, D, idx, coef, D, idx, coef)
    assert "2^20" in str(e.value)


@pytest.mark.parametrize("scale", [2.0 ** -20, 2.0 ** 13])
def test_value_coefficient_scale_does_not_change_relative_accuracy(scale):
    # The histogram's fixed-point unit follows the data: tiny and huge value coefficients keep the accuracy.
    q, DK, idxK, coefK, DV, idxV, coefV = _case(23, 2, 8, 2, 3000, 4096, 8, 8)
    coefV = (coefV.astype(np.float32) * np.float32(scale)).astype(np.float16)
    out = _run(q, DK, idxK, coefK, DV, idxV, coefV, out_dtype=torch.float32)
    _check(out, oracle.decode_attn(q, DK, idxK, coefK, DV, idxV, coefV), TOL_F32_OUT, f"value coefficients x {scale:g}")


def test_hot_atom_with_largest_fp16_coefficients_does_not_overflow():
    # Flat softmax (all key coefficients zero), every value pair on the same atom with |c| = 60000.
    B, Hq, Hkv, T, N, s = 1, 2, 1, 16384, 256, 8
    q, DK, idxK, coefK, DV, idxV, coefV = _case(24, B, Hq, Hkv, T, N, s, s)
    coefK[...] = 0
    idxV[...] = 3
    coefV[...] = np.float16(60000.0)
    out = _run(q, DK, idxK, coefK, DV, idxV, coefV, out_dtype=torch.float32)
    _check(out, oracle.decode_attn(q, DK, idxK, coefK, DV, idxV, coefV), TOL_F32_OUT, "hot atom, largest coefficients")


@pytest.mark.parametrize("dtype", ["f16", "f32"])
def test_value_coefficients_that_grow_far_beyond_the_sampled_ones(dtype):
    # The histogram unit is chosen from the value coefficients of a chunk's first 1024 tokens.  Here those are zero
    # (then tiny), and the later tokens carry coefficients 2^20 times larger (fp32 storage: 2^40): the 32-bit
    # scatter must notice that its unit does not fit and the result must still be right.
    B, Hq, Hkv, T, N, s = 1, 4, 1, 6000, 512, 8
    q, DK, idxK, coefK, DV, idxV, coefV = _case(25, B, Hq, Hkv, T, N, s, s, dtype=dtype, itype="i16" if dtype == "f16" else "i32")
    big = 2.0 ** 40 if dtype == "f32" else 2.0 ** 9
    for head_scale in (0.0, 2.0 ** -11):
        cv = coefV.astype(np.float64)
        cv[:, :, :1024] *= head_scale
        cv[:, :, 1024:] *= big
        cv = cv.astype(coefV.dtype)
        out = _run(q, DK, idxK, coefK, DV, idxV, cv, out_dtype=torch.float32)
        _check(out, oracle.decode_attn(q, DK, idxK, coefK, DV, idxV, cv), TOL_F32_OUT, f"growing coefficients ({dtype}, x{head_scale})")


def test_an_outlier_coefficient_in_the_sample_and_a_diffuse_tail():
    # One sampled value coefficient is 2^14 times the typical one while nearly all of the attention mass sits on a
    # flat tail of tokens far below the maximum score: the adds of the tail are tiny against a unit fitted to the
    # outlier, which the resolution check of the 32-bit scatter has to catch.  (This context counts as a short one, which has
    # no scatter; test_gpu_decode_forms.py asks the same of the streaming kernel.)
    B, Hq, Hkv, T, N, s = 1, 1, 1, 16384, 4096, 8
    q, DK, idxK, coefK, DV, idxV, coefV = _case(26, B, Hq, Hkv, T, N, s, s, dtype="f32", itype="i32")
    coefK[...] = 0
    coefK[0, 0, 0, 0] = 9.0 / max(abs(float(q[0, 0] @ DK[0, idxK[0, 0, 0, 0]])) / np.sqrt(128.0), 1e-3)
    coefK[0, 0, 0, 0] *= np.sign(float(q[0, 0] @ DK[0, idxK[0, 0, 0, 0]]))      # token 0 leads by a score of 9
    coefV[0, 0, 5, 3] = 2.0 ** 14 * 3.0
    out = _run(q, DK, idxK, coefK, DV, idxV, coefV, out_dtype=torch.float32)
    _check(out, oracle.decode_attn(q, DK, idxK, coefK, DV, idxV, coefV), TOL_F32_OUT, "outlier in the sample, diffuse tail")


# --- chunked codes (s_n of Section "NeuralDict"; the experiments store values with s = 4, s_n = 2) ---------

def _chunked_case(seed, B, Hq, Hkv, T, N, snK, sK, snV, sV):
    d = 128
    q = synth.queries(seed, B, Hq, d, "f16")
    DK = synth.dictionary(seed, "dict_k", Hkv * snK, N, d // snK, "f16").reshape(Hkv, snK, N, d // snK)
    DV = synth.dictionary(seed, "dict_v", Hkv * snV, N, d // snV, "f16").reshape(Hkv, snV, N, d // snV)
    idxK, coefK = synth.random_codes(seed, 0, B, Hkv, T, snK * sK, N, "f16", "i16")
    idxV, coefV = synth.random_codes(seed, 1, B, Hkv, T, snV * sV, N, "f16", "i16")
    r = lambda a, sn, s: np.ascontiguousarray(a.reshape(B, Hkv, T, sn, s))
    return q, DK, r(idxK, snK, sK), r(coefK, snK, sK), DV, r(idxV, snV, sV), r(coefV, snV, sV)


def _u16(idx):
    return idx.view(np.uint16).astype(np.int64)


@pytest.mark.parametrize("B,Hq,Hkv,T,N,snK,sK,snV,sV", [
    (1, 2, 2, 700, 256, 1, 8, 2, 4),      # CSR-8 of the experiments: keys whole, values in two chunks
    (2, 4, 4, 2500, 1024, 1, 16, 2, 8),   # CSR-16, several token chunks with a ragged tail
    (1, 8, 2, 1300, 512, 2, 4, 2, 4),     # both chunked, query groups of 4
    (3, 2, 1, 333, 128, 4, 2, 8, 1),      # many chunks, odd vector widths of the code loads
    (1, 1, 1, 1, 128, 8, 4, 4, 8),        # a single token, the most pairs per token
    (1, 4, 2, 5000, 2048, 2, 3, 4, 5),    # pair counts that are not a multiple of 4
])
def test_chunked_codes_against_the_concatenated_reconstruction(B, Hq, Hkv, T, N, snK, sK, snV, sV):
    q, DK, iK, cK, DV, iV, cV = _chunked_case(21, B, Hq, Hkv, T, N, snK, sK, snV, sV)
    DKo = DK if snK > 1 else DK[:, 0]
    iKo, cKo = (iK, cK) if snK > 1 else (iK[:, :, :, 0], cK[:, :, :, 0])
    out = _run(q, DKo, iKo, cKo, DV, iV, cV)
    ref = oracle.decode_attn_chunked(q, DK, _u16(iK), cK, DV, _u16(iV), cV)
    _check(out, ref, TOL_F16_OUT, f"chunked snK={snK} sK={sK} snV={snV} sV={sV} T={T} N={N}")


def test_chunked_codes_with_sequence_lengths():
    B, T = 4, 3000
    q, DK, iK, cK, DV, iV, cV = _chunked_case(22, B, 4, 2, T, 512, 2, 4, 2, 4)
    lens = [0, 1, 1024, T]
    out = _run(q, DK, iK, cK, DV, iV, cV, seq_lens=lens)
    ref = oracle.decode_attn_chunked(q, DK, _u16(iK), cK, DV, _u16(iV), cV, seq_lens=lens)
    assert np.all(out[0] == 0)
    _check(out[1:], ref[1:], TOL_F16_OUT, "chunked with seq_lens")


def test_one_chunk_given_as_five_dimensional_codes_is_the_plain_path_bit_for_bit():
    q, DK, iK, cK, DV, iV, cV = _case(23, 2, 4, 2, 1500, 512, 8, 4)
    a = _run(q, DK, iK, cK, DV, iV, cV)
    b = _run(q, DK[:, None], iK[:, :, :, None], cK[:, :, :, None], DV[:, None], iV[:, :, :, None], cV[:, :, :, None])
    assert np.array_equal(a.view(np.uint16), b.view(np.uint16))


def test_end_to_end_in_the_experiments_layout_keys_whole_values_in_two_chunks():
    # csr_encode output feeds csr_decode_attn unchanged: keys s = 8 whole, values s = 4 in each of two chunks
    Hkv, G, T, N, d = 2, 2, 1500, 1024, 128
    XK = synth.vectors(24, "keys", Hkv, T, d, "f16", outliers=8)
    XV = synth.vectors(24, "values", Hkv, T, d, "f16")
    DK = synth.dictionary(24, "dict_k", Hkv, N, d, "f16")
    DV = synth.dictionary(24, "dict_v", Hkv * 2, N, d // 2, "f16").reshape(Hkv, 2, N, d // 2)
    q = synth.queries(24, 1, Hkv * G, d, "f16")
    g = lambda a: torch.from_numpy(a).cuda()
    iK, cK = csr.csr_encode(g(XK), g(DK), 8)
    iV, cV = csr.csr_encode(g(XV), g(DV), 4)
    assert iV.shape == (Hkv, T, 2, 4)
    out = csr.csr_decode_attn(g(q), g(DK), iK[None], cK[None], g(DV), iV[None], cV[None])
    torch.cuda.synchronize()
    iKh, cKh, iVh, cVh = (t.cpu().numpy()[None] for t in (iK, cK, iV, cV))
    ref = oracle.decode_attn_chunked(q, DK[:, None], _u16(iKh)[:, :, :, None], cKh[:, :, :, None], DV, _u16(iVh), cVh)
    _check(out.cpu().numpy(), ref, TOL_F16_OUT, "encode -> decode, CSR-8 layout")


def test_decoding_steps_append_codes_in_place_and_attend_over_the_grown_cache():
    # prefill T0 tokens, then three decoding steps: every step encodes one new key and value per
    # (sequence, head) straight into row `len` of the code cache and attends over len + 1 tokens
    B, Hkv, G, T0, T_max, N, d, s = 2, 2, 2, 300, 320, 512, 128, 8
    DK = synth.dictionary(25, "dict_k", Hkv, N, d, "f16")
    DV = synth.dictionary(25, "dict_v", Hkv, N, d, "f16")
    XK = synth.vectors(25, "keys", B * Hkv, T_max, d, "f16", outliers=8)
    XV = synth.vectors(25, "values", B * Hkv, T_max, d, "f16")
    g = lambda a: torch.from_numpy(a).cuda()
    XKg, XVg, DKg, DVg = g(XK), g(XV), g(DK), g(DV)
    cache = {n: torch.zeros((B * Hkv, T_max, s), dtype=dt, device="cuda")
             for n, dt in (("iK", torch.int16), ("cK", torch.float16), ("iV", torch.int16), ("cV", torch.float16))}
    csr.csr_encode(XKg[:, :T0], DKg, s, idx=cache["iK"][:, :T0], coef=cache["cK"][:, :T0])
    csr.csr_encode(XVg[:, :T0], DVg, s, idx=cache["iV"][:, :T0], coef=cache["cV"][:, :T0])
    v = lambda t: t.view(B, Hkv, T_max, s)
    for step in range(3):
        pos = T0 + step
        q = synth.queries(25 + step, B, Hkv * G, d, "f16")
        csr.csr_encode(XKg[:, pos:pos + 1], DKg, s, idx=cache["iK"][:, pos:pos + 1], coef=cache["cK"][:, pos:pos + 1])
        csr.csr_encode(XVg[:, pos:pos + 1], DVg, s, idx=cache["iV"][:, pos:pos + 1], coef=cache["cV"][:, pos:pos + 1])
        lens = torch.full((B,), pos + 1, dtype=torch.int32, device="cuda")
        out = csr.csr_decode_attn(g(q), DKg, v(cache["iK"]), v(cache["cK"]), DVg, v(cache["iV"]), v(cache["cV"]),
                                  seq_lens=lens)
        torch.cuda.synchronize()
        h = {n: v(t).cpu().numpy() for n, t in cache.items()}
        ref = oracle.decode_attn(q, DK, h["iK"], h["cK"], DV, h["iV"], h["cV"], seq_lens=[pos + 1] * B)
        _check(out.cpu().numpy(), ref, TOL_F16_OUT, f"decoding step {step}")
    # the appended rows are what encoding the whole sequence at once gives (the encoders may part at ties only)
    i_all, _ = csr.csr_encode(XKg[:, :T0 + 3], DKg, s, algo=csr.CSR_ENCODE_MFMA)
    torch.cuda.synchronize()
    same = (i_all[:, T0:] == cache["iK"][:, T0:T0 + 3]).all(dim=-1).float().mean().item()
    assert same >= 0.75, same
    assert (cache["iK"][:, T0 + 3:] == 0).all()          # rows past the last appended one were never written


def test_chunked_values_full_layer_all_heads():
    # bench.py's chunked_step decode call: 32 heads, 4096 tokens, keys s = 8 whole, values s = 4 in two chunks
    w = synth.WORKLOADS["llama7b_layer"]
    q, DK, iK, cK, DV, iV, cV = _chunked_case(26, w.batch, w.hq, w.hkv, w.tokens, w.n_atoms, 1, 8, 2, 4)
    out = _run(q, DK[:, 0], iK[:, :, :, 0], cK[:, :, :, 0], DV, iV, cV)
    ref = oracle.decode_attn_chunked(q, DK, _u16(iK), cK, DV, _u16(iV), cV)
    _check(out, ref, TOL_F16_OUT, "llama7b layer, values in two chunks, all heads")


@pytest.mark.parametrize("rope_base,gram", [(0.0, False), (10000.0, False), (0.0, True)])
def test_a_decoding_step_can_be_captured_in_a_graph_and_replayed(rope_base, gram):
    # (rope_base set: the keys count as coded before the rotary embedding;
    # gram: the append takes the dictionaries' Gram matrices - its two launches instead of the split encoder's)
    # append (split encoder: one launch behind the one that clears its slots) + attention (a short context: two launches; the
    # streaming kernels' capture is in test_gpu_decode_forms.py) recorded once, replayed on new data;
    # every replay must equal the eager result of the same inputs bit for bit (nothing allocates, nothing is cleared
    # by a memset node, every kernel argument is fixed at capture time)
    B, Hkv, G, T_max, N, d, s, pos = 2, 2, 2, 256, 512, 128, 8, 200
    DK = torch.from_numpy(synth.dictionary(27, "dict_k", Hkv, N, d, "f16")).cuda()
    DV = torch.from_numpy(synth.dictionary(27, "dict_v", Hkv, N, d, "f16")).cuda()
    iK0, cK0 = synth.random_codes(27, 0, B, Hkv, T_max, s, N, "f16", "i16")
    iV0, cV0 = synth.random_codes(27, 1, B, Hkv, T_max, s, N, "f16", "i16")
    g = lambda a: torch.from_numpy(a).cuda()
    mk_cache = lambda: [g(a).view(B * Hkv, T_max, s) for a in (iK0, cK0, iV0, cV0)]
    xk, xv = (torch.zeros((B * Hkv, 1, d), dtype=torch.float16, device="cuda") for _ in range(2))
    q = torch.zeros((B, Hkv * G, d), dtype=torch.float16, device="cuda")
    out = torch.zeros_like(q)
    lens = torch.full((B,), pos + 1, dtype=torch.int32, device="cuda")
    iK, cK, iV, cV = mk_cache()
    edesc = csr.encode_desc(xk, DK, s, torch.float16, torch.int16, code_stride_h=T_max * s)
    wsE = torch.empty(max(csr.csr_encode_workspace_bytes(edesc), 1 << 20), dtype=torch.uint8, device="cuda")
    gk = dict(gram=csr.csr_gram_build(DK)) if gram else {}
    gv = dict(gram=csr.csr_gram_build(DV)) if gram else {}
    v4 = lambda t: t.view(B, Hkv, T_max, s)
    wsD = torch.empty(max(csr.csr_decode_workspace_bytes(csr.decode_desc(q, DK, v4(iK), v4(cK), v4(iV), rope_base=rope_base)), 256),
                      dtype=torch.uint8, device="cuda")

    def step():
        csr.csr_encode(xk, DK, s, idx=iK[:, pos:pos + 1], coef=cK[:, pos:pos + 1], workspace=wsE, **gk)
        csr.csr_encode(xv, DV, s, idx=iV[:, pos:pos + 1], coef=cV[:, pos:pos + 1], workspace=wsE, **gv)
        csr.csr_decode_attn(q, DK, v4(iK), v4(cK), DV, v4(iV), v4(cV), seq_lens=lens, out=out, workspace=wsD,
                            rope_base=rope_base, rope_pos0=7 if rope_base else 0)

    def load(seed):
        xk.copy_(g(synth.vectors(seed, "keys", B * Hkv, 1, d, "f16", outliers=8)))
        xv.copy_(g(synth.vectors(seed, "values", B * Hkv, 1, d, "f16")))
        q.copy_(g(synth.queries(seed, B, Hkv * G, d, "f16")))

    load(100)
    step()                                   # eager once: per-device set-up happens outside the capture
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        with torch.cuda.graph(graph, stream=side):
            step()
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    for seed in (101, 102, 103):
        load(seed)
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        got = (out.clone(), iK[:, pos].clone(), cK[:, pos].clone(), iV[:, pos].clone(), cV[:, pos].clone())
        out.zero_()
        iK[:, pos].zero_(); cK[:, pos].zero_(); iV[:, pos].zero_(); cV[:, pos].zero_()
        step()                               # the program's own eager work between the replays
        torch.cuda.synchronize()
        want = (out, iK[:, pos], cK[:, pos], iV[:, pos], cV[:, pos])
        for a, b in zip(got, want):
            assert torch.equal(a, b), seed
        assert torch.isfinite(out.float()).all() and out.abs().sum() > 0
