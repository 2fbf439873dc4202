"""GPU parity: csr_reconstruct (Eq.12, through the C ABI) against the oracle's dense rebuild."""
import numpy as np
import pytest
import torch

import oracle
import paper_2412_11741_amd as csr
from paper_2412_11741_amd import synth

pytestmark = pytest.mark.gpu


def _ref(D, idx, coef):
    """Per block and chunk: oracle.reconstruct, chunks side by side.  D [H', (sn,) N, dc], codes [H, T, (sn,) s]."""
    if D.ndim == 3:
        D, idx, coef = D[:, None], idx[:, :, None], coef[:, :, None]
    H, T, sn, s = idx.shape
    u = idx.view(np.uint16).astype(np.int32) if idx.dtype == np.int16 else idx
    return np.stack([np.concatenate([oracle.reconstruct(u[h, :, c], coef[h, :, c], D[h % D.shape[0], c])
                                     for c in range(sn)], axis=1) for h in range(H)])


def _check(out, ref, D, coef, storage):
    # fp32 accumulation of s products: a few 2^-24 of sum |c| |d| per element; fp16 output adds one rounding
    mag = np.abs(coef.astype(np.float64)).reshape(coef.shape[0], coef.shape[1], -1).sum(-1)[..., None] * np.abs(D.astype(np.float64)).max()
    tol = 4 * 2.0 ** -24 * mag + (2.0 ** -11 * np.abs(ref) + 6e-8 if storage == "f16" else 0.0)
    err = np.abs(out.astype(np.float64) - ref)
    assert np.all(err <= tol), (err.max(), (err / np.maximum(tol, 1e-300)).max())


@pytest.mark.parametrize("H,T,N,d,sn,s,dicts,dtype,itype", [
    (3, 777, 1024, 128, 1, 8, 3, "f16", "i16"),
    (4, 300, 512, 128, 2, 4, 2, "f16", "i16"),       # values in two chunks, blocks sharing dictionaries
    (2, 65, 96, 64, 1, 5, 2, "f32", "i32"),
    (1, 1, 4096, 128, 1, 32, 1, "f16", "i16"),
    (2, 40, 256, 256, 4, 3, 1, "f16", "i32"),
])
def test_reconstruct_matches_the_dense_rebuild(H, T, N, d, sn, s, dicts, dtype, itype):
    dc = d // sn
    D = synth.dictionary(51, "dict_v", dicts * sn, N, dc, dtype).reshape(dicts, sn, N, dc)
    idx, coef = synth.random_codes(51, 0, 1, H, T, sn * s, N, dtype, itype)
    idx, coef = idx[0].reshape(H, T, sn, s), coef[0].reshape(H, T, sn, s)
    if sn == 1:
        D, idx, coef = D[:, 0], idx[:, :, 0], coef[:, :, 0]
    g = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    out = csr.csr_reconstruct(g(D), g(idx), g(coef))
    out32 = csr.csr_reconstruct(g(D), g(idx), g(coef), out_dtype=torch.float32)
    torch.cuda.synchronize()
    ref = _ref(D, idx, coef)
    _check(out.cpu().numpy(), ref, D, coef, dtype)
    _check(out32.cpu().numpy(), ref, D, coef, "f32")


def test_reconstruct_of_the_encoders_codes_shrinks_the_error_and_reads_codes_in_place():
    # encode into a cache of codes, rebuild from a window of that cache into a strided output
    H, T_max, T, N, d, s = 4, 200, 150, 1024, 128, 8
    D = synth.dictionary(52, "dict_k", H, N, d, "f16")
    X = synth.vectors(52, "keys", H, T, d, "f16", outliers=8)
    Dg, Xg = torch.from_numpy(D).cuda(), torch.from_numpy(X).cuda()
    ci = torch.zeros((H, T_max, s), dtype=torch.int16, device="cuda")
    cc = torch.zeros((H, T_max, s), dtype=torch.float16, device="cuda")
    csr.csr_encode(Xg, Dg, s, idx=ci[:, 10:10 + T], coef=cc[:, 10:10 + T])
    wide = torch.full((H, T, 2 * d), 9.0, dtype=torch.float16, device="cuda")
    csr.csr_reconstruct(Dg, ci[:, 10:10 + T], cc[:, 10:10 + T], out=wide[:, :, d:])
    torch.cuda.synchronize()
    assert (wide[:, :, :d] == 9.0).all()
    rec = wide[:, :, d:].cpu().numpy()
    ref = _ref(D, ci[:, 10:10 + T].cpu().numpy(), cc[:, 10:10 + T].cpu().numpy())
    _check(rec, ref, D, cc[:, 10:10 + T].cpu().numpy(), "f16")
    x = X.astype(np.float64)
    assert np.all(((x - ref) ** 2).sum(-1) < (x ** 2).sum(-1))      # Eq.4 removes energy at every step


@pytest.mark.parametrize("out_dtype", [torch.float16, torch.float32])
@pytest.mark.parametrize("s", [1, 2, 3, 4, 5, 6, 7])
def test_short_codes_at_any_alignment(s, out_dtype):
    # a short code is read as a whole where it is aligned; the same pairs off a word, one at a time, and padded to eight with
    # zero coefficients, as two 16-byte vectors: the sums have one order, so the bits are equal
    H, T, N, d, sn = 2, 131, 320, 128, 2
    gen = torch.Generator().manual_seed(70 + s)
    D = torch.randn(H, sn, N, d // sn, generator=gen).half().cuda()
    idx = torch.randint(0, N, (H, T, sn, s), generator=gen).short()
    idx[0, 0], idx[-1, -1] = 0, N - 1
    coef = torch.randn(H, T, sn, s, generator=gen).half()

    def off_a_word(t):
        buf = torch.empty(t.numel() + 1, dtype=t.dtype, device="cuda")
        return buf[1:].view(t.shape).copy_(t)

    def padded(t):
        return torch.nn.functional.pad(t, (0, 8 - s)).cuda()
    one = csr.csr_reconstruct(D, idx.cuda(), coef.cuda(), out_dtype=out_dtype)
    assert torch.equal(one, csr.csr_reconstruct(D, off_a_word(idx), off_a_word(coef), out_dtype=out_dtype))
    assert torch.equal(one, csr.csr_reconstruct(D, padded(idx), padded(coef), out_dtype=out_dtype))
    rows = torch.gather(D.cpu().double().unsqueeze(1).expand(H, T, sn, N, d // sn), 3,
                        idx.long().unsqueeze(-1).expand(H, T, sn, s, d // sn))
    terms = rows * coef.double().unsqueeze(-1)
    ref, size = terms.sum(3).view(H, T, d), terms.abs().sum(3).view(H, T, d)
    # s fp32 multiply-adds, then one rounding to the output type
    bound = size * s * 2.0 ** -23 + (ref.abs() * 2.0 ** -11 + 2.0 ** -25 if out_dtype == torch.float16 else 0.0)
    assert ((one.cpu().double() - ref).abs() <= bound).all()


@pytest.mark.parametrize("dict_dtype,out_dtype", [(torch.float16, torch.float16), (torch.float16, torch.float32), (torch.float32, torch.float16)])
@pytest.mark.parametrize("s", [2, 4, 6, 8, 10, 16, 24, 32])
def test_whole_vectors_share_their_code_over_a_row_of_lanes(s, dict_dtype, out_dtype):
    # codes that start at a 32-bit word are handed round in a row of 16 lanes; off a word every lane reads its pairs one by one:
    # the sums have one order, so the bits are equal.  131 tokens: the last workgroup is partly filled.
    N, gen = 320, torch.Generator().manual_seed(90 + s)
    for H, T, d, sn, dicts in [(1, 1, 128, 1, 1), (4, 131, 128, 1, 2), (2, 131, 256, 1, 2), (2, 35, 384, 1, 1), (2, 35, 256, 2, 2)]:
        D = torch.randn(dicts, sn, N, d // sn, generator=gen).to(dict_dtype)
        idx = torch.randint(0, N, (H, T + 3, sn, s), generator=gen).short()
        coef = torch.randn(H, T + 3, sn, s, generator=gen).half()
        idx[0, 0], idx[-1, T - 1] = 0, N - 1
        if sn == 1:
            D, idx, coef = D[:, 0], idx[:, :, 0], coef[:, :, 0]
        D, idx, coef = D.cuda(), idx.cuda(), coef.cuda()

        def off_a_word(t):
            buf = torch.empty(t.numel() + 1, dtype=t.dtype, device="cuda")
            return buf[1:].view(t.shape).copy_(t)
        one = csr.csr_reconstruct(D, idx[:, :T], coef[:, :T], out_dtype=out_dtype)   # a window of a longer cache
        two = csr.csr_reconstruct(D, off_a_word(idx)[:, :T], off_a_word(coef)[:, :T], out_dtype=out_dtype)
        assert torch.equal(one, two), (H, T, d, sn)
        Dc, ic, cc = (x if sn > 1 else x.unsqueeze(-3 if x is D else -2) for x in (D, idx, coef))
        blocks = Dc.cpu().double()[torch.arange(H) % dicts]                               # [H, sn, N, dc]
        rows = torch.stack([torch.stack([blocks[h, c][ic[h, :T, c].cpu().long()] for c in range(sn)], 1) for h in range(H)])
        terms = rows * cc[:, :T].cpu().double().unsqueeze(-1)                             # [H, T, sn, s, dc]
        ref, size = terms.sum(3).view(H, T, d), terms.abs().sum(3).view(H, T, d)
        bound = size * s * 2.0 ** -23 + (ref.abs() * 2.0 ** -11 + 2.0 ** -25 if out_dtype == torch.float16 else 0.0)
        assert ((one.cpu().double() - ref).abs() <= bound).all(), (H, T, d, sn)


@pytest.mark.parametrize("dtype,s,per_block", [(torch.float16, 8, 4096), (torch.float16, 5, 4096), (torch.float16, 16, 4096), (torch.float32, 6, 2048)])
@pytest.mark.parametrize("more", [-1, 0, 1])   # tokens of the last block: one less than 4 MB of output, as many, one more
def test_outputs_around_the_line_of_the_non_temporal_stores(dtype, s, per_block, more):
    H, N, gen = 4, 200, torch.Generator(device="cuda").manual_seed(17)
    T = per_block + more
    D = torch.randn(H, N, 128, device="cuda", generator=gen).to(dtype)
    idx = torch.randint(0, N, (H, T, s), device="cuda", generator=gen).short()
    coef = torch.randn(H, T, s, device="cuda", generator=gen).half()
    whole = torch.full((H, T + 1, 128), 7.0, device="cuda", dtype=dtype)   # a row of each block that is not written
    csr.csr_reconstruct(D, idx, coef, out=whole[:, :T])
    parts = torch.cat([csr.csr_reconstruct(D[h:h + 1], idx[h:h + 1], coef[h:h + 1]) for h in range(H)])   # below the line
    assert torch.equal(whole[:, :T], parts.to(dtype)) and (whole[:, T] == 7.0).all()
