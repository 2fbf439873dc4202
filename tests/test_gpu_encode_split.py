"""GPU parity: the few-vectors encoder's slices - several workgroups share a dictionary and exchange their candidates - at
the edges of its split (tests of its options and storage types are with the other encoders')."""
import ctypes

import numpy as np
import pytest
import torch

import paper_2412_11741_amd as csr
from paper_2412_11741_amd import binding, synth
from tests.test_gpu_encode import _assert_ok, _compare

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dicts,M,N,d,s", [
    (8, 1, 4160, 128, 6),      # 130 tiles on 16 slices of 9: the last slice is empty
    (3, 31, 544, 128, 4),      # 17 tiles on 2 slices, a block of vectors with one column missing
    (2, 33, 800, 128, 4),      # 25 tiles on 3 slices, a second block with one vector
    (16, 128, 1024, 64, 4),    # the most vectors; two slots per lane
    (5, 64, 64, 128, 3),       # fewer tiles than waves, no exchange
    (40, 2, 2048, 128, 4),     # dictionaries dealt to the XCDs: 5 each, 6 slices
    (1, 7, 65536, 128, 3),     # tiles beyond the registers are read again in every iteration
    (300, 1, 256, 128, 3),     # more dictionaries than CUs
    (4, 16, 1056, 128, 4),     # the most vectors whose hi and lo share a pass, 33 tiles on 4 slices
    (4, 17, 1056, 128, 4),     # one more
    (32, 15, 8192, 128, 3),    # four tiles a wave in registers
    (6, 16, 320, 64, 4),       # chunks
])
def test_slices_of_a_dictionary_agree(dicts, M, N, d, s):
    D = synth.dictionary(91, "dict_k", dicts, N, d, "f16")
    X = synth.vectors(91, "keys", dicts, M, d, "f16", outliers=4)
    X[-1, -1] = 0.0
    idx, coef = csr.csr_encode(torch.from_numpy(X).cuda(), torch.from_numpy(D).cuda(), s, algo=csr.CSR_ENCODE_SPLIT)
    again = csr.csr_encode(torch.from_numpy(X).cuda(), torch.from_numpy(D).cuda(), s, algo=csr.CSR_ENCODE_SPLIT)
    assert torch.equal(idx, again[0]) and torch.equal(coef, again[1])
    heads = sorted({0, dicts // 2, dicts - 1})
    _assert_ok(_compare(X, D, s, idx.cpu().numpy().view(np.uint16).astype(np.int32), coef.cpu().numpy(), heads=heads))
    assert not idx[-1, -1].any() and not coef[-1, -1].any()


@pytest.mark.parametrize("dicts,M,N,d,s,sn", [
    (8, 1, 4160, 128, 6, 1),    # 16 slices, the last one empty
    (2, 33, 800, 128, 4, 1),    # 3 slices, a second block of vectors
    (3, 128, 1024, 64, 5, 2),   # the most vectors in chunks: two slots per lane, several groups of vectors per wave
    (4, 31, 2048, 64, 32, 1),   # 8 slices, the longest code
])
@pytest.mark.parametrize("closed", [0, csr.CSR_FLAG_CLOSED_LOOP])
def test_codes_do_not_depend_on_who_computed_them(dicts, M, N, d, s, sn, closed):
    # with CSR_FLAG_NO_WAIT every workgroup takes every other one for absent: the missing candidates are computed by the wave
    # that wants them.  The sums are the same, so are the bits
    D = torch.from_numpy(synth.dictionary(92, "dict_k", dicts * sn, N, d, "f16")).cuda()
    D = D.view(dicts, sn, N, d) if sn > 1 else D
    X = torch.from_numpy(synth.vectors(92, "keys", dicts, M, d * sn, "f16", outliers=4)).cuda()
    X[-1, -1] = 0.0
    got = []
    for flags in (closed, closed | csr.CSR_FLAG_NO_WAIT):
        desc = binding.encode_desc(X, D, s, torch.float16, torch.int16, csr.CSR_ENCODE_SPLIT, flags=flags)
        idx = torch.empty(dicts, M, sn, s, dtype=torch.int16, device="cuda")
        coef, err = torch.empty(idx.shape, dtype=torch.float16, device="cuda"), torch.empty(dicts, M, sn, device="cuda")
        desc.res_norm2 = err.data_ptr()
        ws = torch.empty(binding.csr_encode_workspace_bytes(desc), dtype=torch.uint8, device="cuda")
        assert ws.numel() > 0                    # several workgroups share a dictionary
        binding._check(binding.lib().csr_encode(ctypes.byref(desc), *(ctypes.c_void_p(t.data_ptr()) for t in (X, D, idx, coef, ws)),
                                                ws.numel(), binding._stream()))
        torch.cuda.synchronize()
        got.append((idx, coef, err))
    assert all(torch.equal(a, b) for a, b in zip(*got))


@pytest.mark.parametrize("d,N,s", [(128, 4096, 8), (64, 2048, 8), (128, 320, 3)])
def test_sixteen_vectors_are_coded_as_in_a_launch_of_seventeen(d, N, s):
    # with at most 16 vectors hi . d and lo . d are sums of their own, with more one chain: 2 d products either way, whose rounding
    # errors have a standard deviation of sqrt(2 d) 2^-25 |R| |d| = 4.8e-7 |R| at most.  Four of them for a coefficient, and atoms agree
    # wherever the two largest correlations are further apart than both launches' errors
    dicts, bound = 6, 4 * (2 * d) ** 0.5 * 2.0 ** -25
    D = torch.from_numpy(synth.dictionary(95, "dict_k", dicts, N, d, "f16")).cuda()
    X = torch.from_numpy(synth.vectors(95, "keys", dicts, 17, d, "f16", outliers=4)).cuda()
    (i16, c16), (i17, c17) = ([t[:, :16] for t in csr.csr_encode(X[:, :M].contiguous(), D, s, algo=csr.CSR_ENCODE_SPLIT, coef_dtype=torch.float32)]
                              for M in (16, 17))
    i16, i17 = i16.long() & 0xffff, i17.long() & 0xffff
    D64, R = D.double(), X[:, :16].double()
    sure = torch.ones(dicts, 16, dtype=torch.bool, device="cuda")
    for g in range(s):
        first, second = (R @ D64.transpose(1, 2).contiguous()).abs().topk(2, dim=-1).values.unbind(-1)
        error = bound * R.norm(dim=-1)
        sure &= first - second > 2 * error
        atom = D64.gather(1, i16[:, :, g, None].expand(-1, -1, d))
        exact = (R * atom).sum(-1)
        assert torch.equal(i16[:, :, g][sure], i17[:, :, g][sure])
        for c in (c16, c17):
            assert ((c[:, :, g].double() - exact).abs() <= error)[sure].all()
        R = R - exact[..., None] * atom
    assert sure.float().mean() > 0.9
