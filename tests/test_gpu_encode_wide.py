"""GPU parity: the encoder that splits the atoms over a workgroup's waves (encode_wide.hip), what CSR_ENCODE_AUTO runs for
fp32 inputs and for fp16 launches that do not fill the chip otherwise."""
import numpy as np
import pytest
import torch

import oracle
import paper_2412_11741_amd as csr
from paper_2412_11741_amd import binding, synth
from tests import parity
from tests.test_gpu_encode import _assert_ok, _compare

pytestmark = pytest.mark.gpu


def _encode(X, D, s, **kw):
    idx, coef = csr.csr_encode(torch.from_numpy(X).cuda(), torch.from_numpy(D).cuda(), s, algo=csr.CSR_ENCODE_WIDE, **kw)
    torch.cuda.synchronize()
    return idx.cpu().numpy(), coef.cpu().numpy()


@pytest.mark.parametrize("dtype", ["f32", "f16"])
@pytest.mark.parametrize("d,N,T,H,s", [
    (128, 1024, 700, 2, 8),    # two passes of vectors would not fill the chip: one pass, ragged last workgroup
    (128, 31, 33, 1, 4),       # fewer atoms than a tile, two workgroups
    (128, 1, 1, 1, 2),         # one atom, one vector
    (128, 257, 65, 3, 6),      # one atom in a tile of its own, waves without tiles
    (128, 4099, 40, 1, 5),     # odd atom count over 16 or 17 tiles a wave
    (64, 1000, 150, 2, 8),     # teams of eight lanes, two lists each
    (32, 600, 300, 2, 8),      # teams of four lanes, four lists each
    (128, 256, 9000, 2, 3),    # two passes of vectors per workgroup
    (64, 160, 17000, 2, 3),
])
def test_shapes_against_the_oracle(dtype, d, N, T, H, s):
    D = synth.dictionary(5, "dict_k", H, N, d, dtype)
    X = synth.vectors(5, "keys", H, T, d, dtype, outliers=4)
    X[0, 0] = 0.0                                  # a zero residual emits (0, 0)
    if dtype == "f16":
        X[-1, T // 2] = 3.0 * D[-1, N // 2]        # a residual that collapses after one step
    idx, coef = _encode(X, D, s)
    rows = None if T <= 1000 else np.r_[0:40, T // 2 - 20:T // 2 + 20, T - 40:T]
    _assert_ok(_compare(X, D, s, idx, coef, rows=rows))
    if T > 1:
        assert not idx[0, 0].any() and not coef[0, 0].any()


@pytest.mark.parametrize("dtype,scale", [("f32", 1e-20), ("f32", 1e15), ("f16", 1.0)])
def test_equal_atoms_and_extreme_scales(dtype, scale):
    # every atom three times: the best group, other groups and whole lists are undecided; the lowest atom has to win
    base = synth.dictionary(6, "dict_k", 1, 96, 128, dtype)
    D = np.concatenate([base] * 3, axis=1)
    X = (synth.vectors(6, "values", 1, 50, 128, dtype).astype(np.float64) * scale).astype(base.dtype)
    idx, coef = _encode(X, D, 4)
    _assert_ok(_compare(X, D, 4, idx, coef))
    assert idx.max() < 96


def test_shared_dictionaries_in_place_chunks_and_errors():
    B, Hkv, T, N, s, sn = 3, 2, 70, 160, 4, 2
    D = np.stack([synth.dictionary(7 + c, "dict_v", Hkv, N, 64, "f16") for c in range(sn)], axis=1)
    X = synth.vectors(7, "values", B * Hkv, T, 128, "f16")
    Xg, Dg = torch.from_numpy(X).cuda(), torch.from_numpy(D).cuda()
    icache = torch.zeros(B * Hkv, T + 9, sn, s, dtype=torch.int16, device="cuda")
    ccache = torch.zeros(B * Hkv, T + 9, sn, s, dtype=torch.float16, device="cuda")
    err = torch.empty(B * Hkv, T, sn, device="cuda")
    csr.csr_encode(Xg, Dg, s, algo=csr.CSR_ENCODE_WIDE, idx=icache[:, 5:5 + T], coef=ccache[:, 5:5 + T], res_norm2=err)
    for c in range(sn):
        Xc, Dc = np.ascontiguousarray(X[:, :, 64 * c:64 * c + 64]), np.tile(D[:, c], (B, 1, 1))
        _assert_ok(_compare(Xc, Dc, s, icache[:, 5:5 + T, c].cpu().numpy(), ccache[:, 5:5 + T, c].cpu().numpy()))
    rebuilt = csr.csr_reconstruct(Dg, icache[:, 5:5 + T], ccache[:, 5:5 + T], out_dtype=torch.float32)
    exact = ((Xg.float() - rebuilt).view(B * Hkv, T, sn, 64) ** 2).sum(-1)
    assert torch.allclose(err, exact, rtol=5e-3, atol=1e-3)
    assert not icache[:, :5].any() and not ccache[:, 5 + T:].any()


@pytest.mark.parametrize("algo,dtype,d,N,T,H", [
    ("valu", "f32", 128, 1024, 3000, 2), ("valu", "f32", 64, 500, 2000, 2), ("valu", "f32", 32, 1024, 2000, 2),
    ("valu", "f16", 128, 1000, 2000, 2), ("mfma", "f16", 128, 2048, 9000, 2), ("mfma", "f16", 64, 2048, 9000, 2),
    ("resident", "f16", 128, 256, 9000, 2), ("resident", "f16", 128, 512, 3000, 2), ("resident", "f16", 64, 1024, 9000, 2),
])
@pytest.mark.parametrize("closed", [False, True])
def test_same_bits_as_the_encoder_of_the_larger_launches(algo, dtype, d, N, T, H, closed):
    # CSR_ENCODE_AUTO chooses between the two by the launch's size: the codes must not depend on it, down to ties
    algo = {"valu": csr.CSR_ENCODE_VALU, "mfma": csr.CSR_ENCODE_MFMA, "resident": csr.CSR_ENCODE_RESIDENT}[algo]
    X = torch.from_numpy(synth.vectors(8, "keys", H, T, d, dtype, outliers=4)).cuda()
    D = torch.from_numpy(synth.dictionary(8, "dict_k", H, N, d, dtype)).cuda()
    iw, cw = csr.csr_encode(X, D, 8, algo=csr.CSR_ENCODE_WIDE, closed_loop=closed)
    ie, ce = csr.csr_encode(X, D, 8, algo=algo, closed_loop=closed)
    assert torch.equal(iw, ie) and torch.equal(cw, ce)


@pytest.mark.parametrize("algo,dtype,d,N,T,H", [   # the passes per workgroup that the rule takes: 3, 4, 5, 6
    ("valu", "f32", 128, 100, 9000, 2), ("valu", "f32", 128, 70, 16000, 2), ("valu", "f16", 64, 33, 20000, 2),
    ("mfma", "f16", 128, 544, 16000, 2), ("mfma", "f16", 128, 544, 20001, 2), ("mfma", "f16", 128, 608, 24500, 2),
    ("mfma", "f16", 128, 544, 2450, 16), ("mfma", "f16", 64, 1056, 20001, 2),
])
def test_same_bits_with_several_passes_per_workgroup(algo, dtype, d, N, T, H):
    algo = {"valu": csr.CSR_ENCODE_VALU, "mfma": csr.CSR_ENCODE_MFMA}[algo]
    X = torch.from_numpy(synth.vectors(9, "keys", H, T, d, dtype, outliers=4)).cuda()
    D = torch.from_numpy(synth.dictionary(9, "dict_k", H, N, d, dtype)).cuda()
    iw, cw = csr.csr_encode(X, D, 4, algo=csr.CSR_ENCODE_WIDE)
    ie, ce = csr.csr_encode(X, D, 4, algo=algo)
    assert torch.equal(iw, ie) and torch.equal(cw, ce)


@pytest.mark.parametrize("s", [1, 2, 3, 6])   # one pair: no dictionary is held, two: those without tiles in LDS
@pytest.mark.parametrize("algo,dtype,d,N,T,H", [   # the dictionary on the CU: its last tiles in LDS, waves without one there, one atom too many
    ("valu", "f32", 128, 513, 40, 2), ("valu", "f32", 128, 769, 33, 3), ("valu", "f32", 128, 1023, 1000, 2), ("valu", "f32", 128, 1025, 100, 2),
    ("valu", "f32", 64, 1537, 100, 2), ("valu", "f32", 64, 2047, 700, 2), ("valu", "f32", 32, 3073, 150, 2), ("valu", "f32", 32, 4096, 300, 1),
    ("valu", "f16", 128, 1000, 100, 2), ("mfma", "f16", 128, 800, 300, 2), ("mfma", "f16", 128, 1024, 1001, 4), ("mfma", "f16", 128, 1056, 300, 2),
    ("mfma", "f16", 64, 1568, 300, 2), ("mfma", "f16", 64, 2048, 1001, 2),
])
def test_same_bits_with_the_dictionary_on_the_cu(algo, dtype, d, N, T, H, s):
    algo = {"valu": csr.CSR_ENCODE_VALU, "mfma": csr.CSR_ENCODE_MFMA}[algo]
    X = torch.from_numpy(synth.vectors(12, "keys", H, T, d, dtype, outliers=4)).cuda()
    D = torch.from_numpy(synth.dictionary(12, "dict_k", H, N, d, dtype)).cuda()
    iw, cw = csr.csr_encode(X, D, s, algo=csr.CSR_ENCODE_WIDE)
    ie, ce = csr.csr_encode(X, D, s, algo=algo)
    assert torch.equal(iw, ie) and torch.equal(cw, ce)


@pytest.mark.parametrize("N,d,T,H", [   # blocks per wave that the resident encoder's rule takes: 1, 2, 3, 4
    (64, 128, 30001, 2), (96, 128, 60007, 2), (64, 128, 90001, 2), (32, 128, 131000, 2), (96, 64, 130001, 2), (1024, 64, 40001, 2),
])
def test_resident_encoder_with_one_to_four_blocks_per_wave(N, d, T, H):
    X = torch.from_numpy(synth.vectors(11, "keys", H, T, d, "f16", outliers=4)).cuda()
    D = torch.from_numpy(synth.dictionary(11, "dict_k", H, N, d, "f16")).cuda()
    ir, cr = csr.csr_encode(X, D, 2, algo=csr.CSR_ENCODE_RESIDENT)
    iw, cw = csr.csr_encode(X, D, 2, algo=csr.CSR_ENCODE_WIDE)
    assert torch.equal(ir, iw) and torch.equal(cr, cw)


@pytest.mark.parametrize("N,d", [(32, 128), (96, 128), (256, 128), (512, 128), (32, 64), (160, 64), (1024, 64)])   # one tile, odd and even numbers of them
@pytest.mark.parametrize("gain", [1.0, 1.6])   # 1.6: Eq.4 lengthens the residual
def test_resident_encoder_where_the_residual_collapses_or_grows(N, d, gain):
    # |hi|^2 stands for |R|^2 but near the lines where the residual is scaled again: vectors on either side of them
    T, s = 600, 7
    rng = np.random.default_rng(13)
    D = (synth.dictionary(13, "dict_k", 1, N, d, "f16").astype(np.float32) * gain)
    D[0, :min(N, d) // 2] = gain * np.eye(d, dtype=np.float32)[:min(N, d) // 2]       # unit vectors: residuals of exactly zero, and of one subnormal
    D = D.astype(np.float16)
    X = rng.standard_normal((1, T, d)).astype(np.float32)
    X[0, 0] = 0.0
    near = D[0, rng.integers(0, N, T // 2)].astype(np.float32)
    X[0, 1:1 + T // 2] = near * 3.0 + rng.standard_normal((T // 2, d)) * 10.0 ** rng.uniform(-6, 0, (T // 2, 1))
    X[0, -2] = 0.0
    X[0, -2, 0], X[0, -2, 1] = 65504.0, 6e-8
    X = X.astype(np.float16)
    Xg, Dg = torch.from_numpy(X).cuda(), torch.from_numpy(D).cuda()
    er, ew = torch.empty(1, T, device="cuda"), torch.empty(1, T, device="cuda")
    ir, cr = csr.csr_encode(Xg, Dg, s, algo=csr.CSR_ENCODE_RESIDENT, res_norm2=er)
    iw, cw = csr.csr_encode(Xg, Dg, s, algo=csr.CSR_ENCODE_WIDE, res_norm2=ew)
    assert torch.equal(ir, iw) and torch.equal(cr, cw)
    assert torch.allclose(er, ew, rtol=2e-5, atol=0.0)   # the same terms in another order: 128 roundings of 2^-24
    # (the wide encoder shares helpers with this one: both against the oracle)
    ic, cc = ir.cpu().numpy(), cr.cpu().numpy()
    _assert_ok(_compare(X, D, s, ic, cc))
    io, co = oracle.mp_encode(X[0], D[0], s)
    same = (parity._as_index(ic[0]) == io).all(axis=1)   # (ties may be resolved either way)
    X64, D64 = X[0].astype(np.float64), D[0].astype(np.float64)
    left = ((X64 - np.einsum("ts,tsk->tk", co, D64[io])) ** 2).sum(axis=1)
    # An iteration's coefficient is a sum of 64 products a lane in two chains of pairs, and the residual's own rounding: less than 64 roundings of
    # 2^-24 of |R| |d|.  That moves the residual by |d| times as much; a later step stretches what is there, R and its error, by at most
    # |d|^2 - 1 where that is above 1.
    stretch = max(1.0, gain ** 2 - 1.0)
    off = s * 2.0 ** -18 * gain ** 2 * stretch ** s * np.linalg.norm(X64, axis=1)
    assert (np.abs(er[0].cpu().numpy() - left) <= 2.0 * np.sqrt(left) * off + off ** 2 + 2e-5 * left)[same].all()


@pytest.mark.parametrize("B,Hkv,T,N,sn", [
    (1, 2, 70000, 544, 1),     # one generation of the prefill encoder's workgroups, 4464 vectors of each dictionary left over
    (5, 3, 9001, 544, 1),      # sequences that share three dictionaries: the line lies inside one of them
    (1, 8, 10300, 1056, 2),    # chunks of 64 dimensions
])
def test_a_launch_shared_by_two_encoders_has_the_codes_of_one(B, Hkv, T, N, sn):
    D = torch.from_numpy(synth.dictionary(10, "dict_k", Hkv * sn, N, 128 // sn, "f16")).cuda()
    if sn > 1:
        D = D.view(Hkv, sn, N, 128 // sn)
    X = torch.from_numpy(synth.vectors(10, "keys", B * Hkv, T, 128, "f16", outliers=4)).cuda()
    shape = (B * Hkv, T) + ((sn,) if sn > 1 else ())
    ea, em = (torch.full(shape, -1.0, device="cuda") for _ in range(2))
    ia, ca = csr.csr_encode(X, D, 4, res_norm2=ea)
    im, cm = csr.csr_encode(X, D, 4, algo=csr.CSR_ENCODE_MFMA, res_norm2=em)
    assert torch.equal(ia, im) and torch.equal(ca, cm)
    assert torch.allclose(ea, em, rtol=1e-5, atol=1e-4)   # the squares are added in another order
    # with scratch for the prefill encoder alone it takes all vectors
    ws = torch.empty(256 * 64, dtype=torch.uint8, device="cuda")
    iw, cw = csr.csr_encode(X, D, 4, workspace=ws)
    assert torch.equal(iw, im) and torch.equal(cw, cm)


@pytest.mark.parametrize("dtype", ["f32", "f16"])
def test_a_workspace_too_small_for_this_encoder_keeps_the_other_one(dtype):
    # sized for more vectors (fp16), or none, where the vector ALU needs none: accepted, with the same codes
    T, N, s, f16 = 300, 1024, 4, int(dtype == "f16")
    D = torch.from_numpy(synth.dictionary(9, "dict_k", 1, N, 128, dtype)).cuda()
    X = torch.from_numpy(synth.vectors(9, "keys", 1, T, 128, dtype, outliers=4)).cuda()

    def scratch(algo, tokens):
        return binding.csr_encode_workspace_bytes(binding.EncodeDesc(
            H=1, T=tokens, d=128, N=N, s=s, x_dtype=f16, dict_dtype=f16, coef_dtype=f16, idx_dtype=f16, x_stride_h=tokens * 128,
            x_stride_t=128, algo=algo))
    small = scratch(csr.CSR_ENCODE_MFMA, 120000) if f16 else scratch(csr.CSR_ENCODE_VALU, T)
    assert small < scratch(csr.CSR_ENCODE_AUTO, T)
    one = csr.csr_encode(X, D, s, workspace=torch.empty(small, dtype=torch.uint8, device="cuda"))
    two = csr.csr_encode(X, D, s)
    assert torch.equal(one[0], two[0]) and torch.equal(one[1], two[1])


def test_an_output_that_does_not_fit_leaves_nothing_behind():
    # the atom numbers fit the device memory that is left, the coefficients do not: the call fails and gives the first back
    H, T, s = 1, 1 << 20, 32
    X = torch.zeros(H, T, 128, dtype=torch.float16, device="cuda")
    D = torch.ones(H, 32, 128, dtype=torch.float16, device="cuda")
    ws = torch.empty(1 << 20, dtype=torch.uint8, device="cuda")
    torch.cuda.empty_cache()
    room = torch.cuda.memory_reserved() + (96 << 20)            # idx takes 64 MB, coef 128 MB
    torch.cuda.set_per_process_memory_fraction(room / torch.cuda.mem_get_info()[1])
    try:
        before = torch.cuda.memory_allocated()
        for _ in range(2):
            try:
                csr.csr_encode(X, D, s, coef_dtype=torch.float32, workspace=ws)
                pytest.fail("the limit has no effect")
            except torch.OutOfMemoryError:
                pass
        assert torch.cuda.memory_allocated() == before
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
        torch.cuda.empty_cache()
