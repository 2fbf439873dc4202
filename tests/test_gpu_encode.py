"""GPU parity: csr_encode (through the C ABI) against the CPU oracle on the same seeded inputs."""
import numpy as np
import pytest
import torch

import oracle
import paper_2412_11741_amd as csr
from paper_2412_11741_amd import synth
from tests import parity

pytestmark = pytest.mark.gpu

# Coefficient tolerance: 1e-3 * |c|, or, where that is larger, 2^-23 |x| (one fp32 ulp of the input's norm)
# plus one storage ulp for fp16 coefficients (tests/parity.py states the rule and why).  fp32 storage: fp32
# dot products of 128 terms against fp64 (well under 1e-5).  fp16 storage adds one rounding to 11 bits
# (2^-11 = 4.9e-4); the oracle value is rounded the same way before comparing, and 1e-3 covers a one-ulp
# flip at a rounding boundary.  On the benchmark configurations the absolute clause must never be needed:
# their tests pass no_floor=True, which asserts that no index and no coefficient was accepted by it.
TOL = 1e-3

ALGOS = {"valu": csr.CSR_ENCODE_VALU, "mfma": csr.CSR_ENCODE_MFMA, "split": csr.CSR_ENCODE_SPLIT,
         "resident": csr.CSR_ENCODE_RESIDENT}
SPLIT_MAX = 128   # vectors per dictionary the split encoder takes


def _gpu_encode(X, D, s, algo, coef_dtype=None, idx_dtype=None):
    Xg, Dg = torch.from_numpy(X).cuda(), torch.from_numpy(D).cuda()
    idx, coef = csr.csr_encode(Xg, Dg, s, coef_dtype=coef_dtype, idx_dtype=idx_dtype, algo=algo)
    torch.cuda.synchronize()
    return idx.cpu().numpy(), coef.cpu().numpy()


def _compare(X, D, s, idx_g, coef_g, heads=None, rows=None):
    """Oracle on (a subset of) the vectors; returns the merged report."""
    H = X.shape[0]
    reports = []
    for h in (range(H) if heads is None else heads):
        r = slice(None) if rows is None else rows
        Xh = X[h][r]
        idx_o, coef_o, diag = oracle.mp_encode(Xh, D[h], s, diagnostics=True)
        with np.errstate(over="ignore"):
            coef_o_st = coef_o.astype(coef_g.dtype).astype(np.float64)  # storage rounding, RNE; infinite beyond the largest value
        rep = parity.check_encode(Xh, D[h], idx_g[h][r], coef_g[h][r], idx_o, coef_o_st, diag, TOL,
                                  coef_storage="f16" if coef_g.dtype == np.float16 else "f32", coef_o_exact=coef_o)
        reports.append(rep)
    return reports


def _assert_ok(reports, no_floor=False):
    for rep in reports:
        assert rep.ok, rep.summary() + "\n" + "\n".join(rep.failures)
    total = sum(r.steps for r in reports)
    exact = sum(r.exact_steps for r in reports)
    ties = sum(r.tie_vectors for r in reports)
    floor_ties = sum(r.floor_ties for r in reports)
    floor_coefs = sum(r.floor_coefs for r in reports)
    print(f"[encode parity] {sum(r.vectors for r in reports)} vectors, {exact}/{total} steps identical, "
          f"{ties} tie-diverged vectors ({ties - floor_ties} within 1e-6 relative, {floor_ties} by the absolute floor), "
          f"{floor_coefs} coefficients by the absolute floor, max coef err {max(r.max_coef_err for r in reports):.2e}",
          flush=True)
    # ties within 1e-6 are rare events: if more than a handful of vectors diverge, something is off
    assert ties <= max(2, total // 20000)
    if no_floor:
        assert floor_ties == 0 and floor_coefs == 0, (floor_ties, floor_coefs)


def test_tiny_config_fp32_full():
    w = synth.WORKLOADS["tiny"]
    D = synth.dictionary(0, "dict_k", 1, w.n_atoms, w.d, "f32")
    X = synth.vectors(0, "keys", 1, w.tokens, w.d, "f32", outliers=w.key_outliers)
    idx, coef = _gpu_encode(X, D, w.s, csr.CSR_ENCODE_VALU)
    assert idx.dtype == np.int32 and coef.dtype == np.float32 and idx.shape == (1, 4096, 8)
    _assert_ok(_compare(X, D, w.s, idx, coef), no_floor=True)


@pytest.mark.parametrize("algo", ["valu", "mfma"])
def test_fp16_ragged_tail_several_heads(algo):
    H, T, N, d, s = 3, 777, 1024, 128, 8
    D = synth.dictionary(1, "dict_k", H, N, d, "f16")
    X = synth.vectors(1, "keys", H, T, d, "f16", outliers=8)
    idx, coef = _gpu_encode(X, D, s, ALGOS[algo])
    assert idx.dtype == np.int16 and coef.dtype == np.float16
    _assert_ok(_compare(X, D, s, idx, coef))


def test_valu_atom_count_not_a_multiple_of_anything():
    H, T, N, d, s = 2, 130, 1000 + 3, 128, 6
    D = synth.dictionary(2, "dict_v", H, N, d, "f16")
    X = synth.vectors(2, "values", H, T, d, "f16")
    idx, coef = _gpu_encode(X, D, s, csr.CSR_ENCODE_VALU)
    _assert_ok(_compare(X, D, s, idx, coef))


@pytest.mark.parametrize("d", [32, 64])
@pytest.mark.parametrize("dtype", ["f16", "f32"])
def test_valu_smaller_head_chunks(d, dtype):
    H, T, N, s = 2, 200, 256, 4
    D = synth.dictionary(3, "dict_v", H, N, d, dtype)
    X = synth.vectors(3, "values", H, T, d, dtype)
    idx, coef = _gpu_encode(X, D, s, csr.CSR_ENCODE_VALU)
    _assert_ok(_compare(X, D, s, idx, coef))


@pytest.mark.parametrize("algo", ["valu", "mfma", "split", "resident"])
@pytest.mark.parametrize("s", [1, 16, 32])
def test_iteration_counts(algo, s):
    H, T, N, d = 1, 192 if algo != "split" else 70, 512, 128
    D = synth.dictionary(4, "dict_k", H, N, d, "f16")
    X = synth.vectors(4, "keys", H, T, d, "f16", outliers=8)
    idx, coef = _gpu_encode(X, D, s, ALGOS[algo])
    _assert_ok(_compare(X, D, s, idx, coef))


@pytest.mark.parametrize("algo", ["valu", "mfma", "split", "resident"])
def test_orthonormal_dictionary_recovers_top_s_coordinates(algo):
    # Identity atoms (padded with a second, rotated orthonormal basis so N is a multiple of 32 x 8):
    # with the identity alone the codes are the s largest |x_k| in order.
    d, s, T = 128, 8, 256 if algo != "split" else SPLIT_MAX
    D = np.eye(d, dtype=np.float16)[None]
    X = synth.vectors(5, "keys", 1, T, d, "f16", outliers=4)
    # make magnitudes distinct so the order is unique
    X = (X.astype(np.float32) + np.linspace(0, 0.01, d, dtype=np.float32)).astype(np.float16)
    idx, coef = _gpu_encode(X, D, s, ALGOS[algo])
    order = np.argsort(-np.abs(X[0].astype(np.float64)), axis=1, kind="stable")[:, :s]
    assert np.array_equal(idx[0].view(np.uint16).astype(np.int64), order)
    assert np.array_equal(coef[0], np.take_along_axis(X[0], order, axis=1))


@pytest.mark.parametrize("algo", ["valu", "mfma", "split", "resident"])
def test_degenerate_inputs_zero_vectors_scaled_atoms_single_vector(algo):
    H, N, d, s = 1, 256, 128, 4
    D = synth.dictionary(6, "dict_k", H, N, d, "f16")
    X = np.zeros((1, 3, d), dtype=np.float16)
    X[0, 1] = D[0, 77] * np.float16(2.0)
    X[0, 2] = -D[0, 5]
    idx, coef = _gpu_encode(X, D, s, ALGOS[algo])
    assert np.all(idx[0, 0] == 0) and np.all(coef[0, 0] == 0) and not np.any(np.isnan(coef.astype(np.float32)))
    assert idx[0, 1, 0] == 77 and abs(float(coef[0, 1, 0]) - 2.0) < 4e-3
    assert idx[0, 2, 0] == 5 and abs(float(coef[0, 2, 0]) + 1.0) < 2e-3
    _assert_ok(_compare(X, D, s, idx, coef))
    # T = 1
    idx1, coef1 = _gpu_encode(X[:, 1:2], D, s, ALGOS[algo])
    assert np.array_equal(idx1[0, 0], idx[0, 1]) and np.array_equal(coef1[0, 0], coef[0, 1])


def test_empty_problem_is_a_noop():
    D = torch.zeros(2, 64, 128, dtype=torch.float16, device="cuda")
    X = torch.zeros(2, 0, 128, dtype=torch.float16, device="cuda")
    idx, coef = csr.csr_encode(X, D, 4)
    assert idx.shape == (2, 0, 4) and coef.shape == (2, 0, 4)


@pytest.mark.parametrize("algo", ["valu", "mfma"])
def test_strided_input_and_storage_types_do_not_change_indices(algo):
    H, T, N, d, s = 2, 100, 512, 128, 8
    D = synth.dictionary(7, "dict_k", H, N, d, "f16")
    X = synth.vectors(7, "keys", H, T, d, "f16", outliers=8)
    Dg = torch.from_numpy(D).cuda()
    wide = torch.zeros(H, T, 2 * d, dtype=torch.float16, device="cuda")   # e.g. K and V interleaved
    wide[:, :, :d] = torch.from_numpy(X).cuda()
    i16, c16 = csr.csr_encode(wide[:, :, :d], Dg, s, algo=ALGOS[algo])
    i32, c32 = csr.csr_encode(torch.from_numpy(X).cuda(), Dg, s, coef_dtype=torch.float32,
                              idx_dtype=torch.int32, algo=ALGOS[algo])
    torch.cuda.synchronize()
    # open loop: the residual uses the unrounded coefficient, so storage precision cannot move indices
    assert np.array_equal(i16.cpu().numpy().view(np.uint16).astype(np.int32), i32.cpu().numpy())
    assert np.array_equal(c16.cpu().numpy(), c32.cpu().numpy().astype(np.float16))
    _assert_ok(_compare(X, D, s, i32.cpu().numpy(), c32.cpu().numpy()))


@pytest.mark.parametrize("algo", ["valu", "mfma"])
def test_llama7b_layer_shape_subset(algo):
    # 4 of the 64 dictionaries (2 key heads with outlier channels, 2 value heads), 512 tokens each.
    w = synth.WORKLOADS["llama7b_layer"]
    T = 512
    DK = synth.dictionary(0, "dict_k", 2, w.n_atoms, w.d, "f16")
    DV = synth.dictionary(0, "dict_v", 2, w.n_atoms, w.d, "f16")
    XK = synth.vectors(0, "keys", 2, T, w.d, "f16", outliers=w.key_outliers)
    XV = synth.vectors(0, "values", 2, T, w.d, "f16")
    D, X = np.concatenate([DK, DV]), np.concatenate([XK, XV])
    idx, coef = _gpu_encode(X, D, w.s, ALGOS[algo])
    _assert_ok(_compare(X, D, w.s, idx, coef), no_floor=True)


@pytest.mark.parametrize("algo", ["valu", "mfma"])
def test_llama7b_layer_full_size_sampled(algo):
    # The benchmark's launch: 64 dictionaries x 4096 vectors in one call; the oracle checks a sample
    # of 24 vectors from every dictionary (ragged positions, first and last rows included).
    w = synth.WORKLOADS["llama7b_layer"]
    DK = synth.dictionary(0, "dict_k", w.hkv, w.n_atoms, w.d, "f16")
    DV = synth.dictionary(0, "dict_v", w.hkv, w.n_atoms, w.d, "f16")
    XK = synth.vectors(0, "keys", w.hkv, w.tokens, w.d, "f16", outliers=w.key_outliers)
    XV = synth.vectors(0, "values", w.hkv, w.tokens, w.d, "f16")
    D, X = np.concatenate([DK, DV]), np.concatenate([XK, XV])
    idx, coef = _gpu_encode(X, D, w.s, ALGOS[algo])
    rows = np.unique(np.concatenate([[0, 63, 64, w.tokens - 1],
                                     synth.stream(0, "misc", 1).integers(0, w.tokens, 20)]))
    _assert_ok(_compare(X, D, w.s, idx, coef, rows=rows), no_floor=True)
    # every index in range
    assert int(idx.view(np.uint16).max()) < w.n_atoms


def test_llama7b_layer_every_vector_of_the_benchmark_launch():
    # The benchmark's launch again, and this time the oracle encodes ALL 262144 vectors (about 20 s of host time on
    # the GPU machine's cores), so that the encoder's rare decision paths - two or three candidate groups resolved
    # exactly, and the evaluate-every-atom fallback when a lane's fourth tracked group is still a candidate - are
    # compared wherever this data takes them (Eq.3 decided at fp32 precision).
    w = synth.WORKLOADS["llama7b_layer"]
    DK = synth.dictionary(0, "dict_k", w.hkv, w.n_atoms, w.d, "f16")
    DV = synth.dictionary(0, "dict_v", w.hkv, w.n_atoms, w.d, "f16")
    XK = synth.vectors(0, "keys", w.hkv, w.tokens, w.d, "f16", outliers=w.key_outliers)
    XV = synth.vectors(0, "values", w.hkv, w.tokens, w.d, "f16")
    D, X = np.concatenate([DK, DV]), np.concatenate([XK, XV])
    idx, coef = _gpu_encode(X, D, w.s, csr.CSR_ENCODE_AUTO)
    reports = []
    for h in range(X.shape[0]):
        reports += _compare(X, D, w.s, idx, coef, heads=[h])
        if h % 8 == 7:
            print(f"[encode parity] dictionaries 0..{h} compared", flush=True)
    _assert_ok(reports, no_floor=True)
    assert sum(r.vectors for r in reports) == 2 * w.hkv * w.tokens


def test_long_context_shape_subset_mfma():
    # Long-context configuration: N = 8192 atoms, s = 16 iterations; 2 dictionaries x 1024 vectors.
    w = synth.WORKLOADS["long_context"]
    D = np.concatenate([synth.dictionary(0, "dict_k", 1, w.n_atoms, w.d, "f16"),
                        synth.dictionary(0, "dict_v", 1, w.n_atoms, w.d, "f16")])
    X = np.concatenate([synth.vectors(0, "keys", 1, 1024, w.d, "f16", outliers=w.key_outliers),
                        synth.vectors(0, "values", 1, 1024, w.d, "f16")])
    idx, coef = _gpu_encode(X, D, w.s, csr.CSR_ENCODE_MFMA)
    _assert_ok(_compare(X, D, w.s, idx, coef, rows=slice(0, 1024, 3)), no_floor=True)


def _sampled_rows_of_a_resident_launch(X, D, idx, coef, s, dicts, blocks, rows, no_floor=True):
    """X [H, T, d], idx / coef [H, T, s] on the GPU, D [dicts, N, d]: copies the sampled (block, row) entries back and
    compares them with the oracle, block h on dictionary h % dicts."""
    rt = torch.from_numpy(np.asarray(rows)).to(X.device)
    bt = torch.from_numpy(np.asarray(blocks)).to(X.device)
    Xs = X[bt][:, rt].cpu().numpy()
    idx_s, coef_s = idx[bt][:, rt].cpu().numpy(), coef[bt][:, rt].cpu().numpy()
    Dh = D.cpu().numpy()
    Db = np.stack([Dh[h % dicts] for h in blocks])
    _assert_ok(_compare(Xs, Db, s, idx_s, coef_s), no_floor=no_floor)


def _indices_in_range(idx, N):
    return int(idx.view(torch.uint8).view(torch.int16).to(torch.int32).bitwise_and(0xffff).max()) < N


def test_long_context_full_launch_sampled():
    # The long-context configuration at its full shape, in one call: 4 sequences x 32 heads x {K, V} = 256 blocks of
    # 32768 vectors on 64 dictionaries of 8192 atoms, s = 16 (8.4 M vectors, the 8-wave workgroups, 128 tiles per
    # sweep).  The oracle checks sampled rows of sampled blocks: first and last rows, both sides of tile and
    # workgroup boundaries, first and last block of a dictionary.
    w = synth.WORKLOADS["long_context"]
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(31)
    dicts, H, T = 2 * w.hkv, 2 * w.hkv * w.batch, w.tokens
    D = torch.randn(dicts, w.n_atoms, w.d, device=dev, generator=gen)
    D = (D / D.norm(dim=-1, keepdim=True)).half()
    X = torch.empty(H, T, w.d, device=dev, dtype=torch.float16)
    for h in range(H):                              # block h: sequence h // 64, dictionary h % 64 (keys first)
        x = torch.randn(T, w.d, device=dev, generator=gen)
        if h % dicts < w.hkv:
            x[:, :w.key_outliers] *= 10
        X[h] = x.half()
    print(f"[long_context] encoding {H * T} vectors", flush=True)
    idx, coef = csr.csr_encode(X, D, w.s)
    torch.cuda.synchronize()
    assert _indices_in_range(idx, w.n_atoms)
    rows = np.unique(np.concatenate([[0, 63, 64, 511, 512, T - 513, T - 512, T - 1],
                                     synth.stream(0, "misc", 5).integers(0, T, 4)]))
    blocks = [0, 1, 31, 32, 63, 64, 127, 128, 200, 255]
    _sampled_rows_of_a_resident_launch(X, D, idx, coef, w.s, dicts, blocks, rows)


def test_gqa_full_launch_shared_dictionaries_sampled():
    # The grouped-query configuration at its full shape, keys and values in one call: 8 sequences x 8 KV heads x
    # {K, V} = 128 blocks of 131072 vectors on 16 shared dictionaries (1 M vectors per dictionary, 16.8 M vectors,
    # 4.3 GB of input: vector numbers and byte offsets beyond 2^31).
    w = synth.WORKLOADS["gqa_llama3_8b"]
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(32)
    dicts, H, T = 2 * w.hkv, 2 * w.hkv * w.batch, w.tokens
    D = torch.randn(dicts, w.n_atoms, w.d, device=dev, generator=gen)
    D = (D / D.norm(dim=-1, keepdim=True)).half()
    X = torch.empty(H, T, w.d, device=dev, dtype=torch.float16)
    for h in range(H):
        x = torch.randn(T, w.d, device=dev, generator=gen)
        if h % dicts < w.hkv:
            x[:, :w.key_outliers] *= 10
        X[h] = x.half()
    assert X.numel() * 2 >= 2 ** 32
    print(f"[gqa] encoding {H * T} vectors", flush=True)
    idx, coef = csr.csr_encode(X, D, w.s)
    torch.cuda.synchronize()
    assert _indices_in_range(idx, w.n_atoms)
    rows = np.unique(np.concatenate([[0, 63, 64, 511, 512, T - 513, T - 512, T - 1],
                                     synth.stream(0, "misc", 6).integers(0, T, 8)]))
    blocks = [0, 7, 8, 15, 16, 63, 64, 65, 100, 112, 127]      # 64 and up start beyond 2^31 bytes of input
    _sampled_rows_of_a_resident_launch(X, D, idx, coef, w.s, dicts, blocks, rows)


def test_prefill_stress_one_layer_launch_sampled():
    # One layer of the prefill stress configuration in one call: 16 dictionaries (8 KV heads x K, V),
    # 16 sequences x 8192 tokens each; the oracle checks 12 sampled vectors per dictionary.
    w = synth.WORKLOADS["prefill_stress"]
    T = w.batch * w.tokens
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(21)
    H = 2 * w.hkv
    D = torch.randn(H, w.n_atoms, w.d, device=dev, generator=gen)
    D = (D / D.norm(dim=-1, keepdim=True)).half()
    X = torch.randn(H, T, w.d, device=dev, generator=gen)
    X[:w.hkv, :, :w.key_outliers] *= 10
    X = X.half()
    idx, coef = csr.csr_encode(X, D, w.s, algo=csr.CSR_ENCODE_MFMA)
    torch.cuda.synchronize()
    assert int(idx.view(torch.uint8).view(torch.int16).to(torch.int32).bitwise_and(0xffff).max()) < w.n_atoms
    rows = np.unique(np.concatenate([[0, 255, 256, T - 1], synth.stream(0, "misc", 2).integers(0, T, 8)]))
    rt = torch.from_numpy(rows).to(dev)
    Xs, Dh = X[:, rt].cpu().numpy(), D.cpu().numpy()
    idx_s, coef_s = idx[:, rt].cpu().numpy(), coef[:, rt].cpu().numpy()
    _assert_ok(_compare(Xs, Dh, w.s, idx_s, coef_s), no_floor=True)


@pytest.mark.parametrize("N", [32, 96, 160, 2080])
def test_mfma_atom_counts_that_leave_partial_stages(N):
    # N is a multiple of the 32-atom tile but not of the 64-atom LDS stage or of the three-buffer ring.
    H, T, d, s = 2, 300, 128, 6
    D = synth.dictionary(8, "dict_k", H, N, d, "f16")
    X = synth.vectors(8, "keys", H, T, d, "f16", outliers=8)
    idx, coef = _gpu_encode(X, D, s, csr.CSR_ENCODE_MFMA)
    _assert_ok(_compare(X, D, s, idx, coef))
    assert int(idx.view(np.uint16).max()) < N


def test_mfma_results_do_not_depend_on_the_run():
    # The encoder has no atomics and no order-dependent reductions: two runs give the same bits.
    H, T, N, d, s = 2, 1000, 1024, 128, 8
    D = synth.dictionary(9, "dict_k", H, N, d, "f16")
    X = synth.vectors(9, "keys", H, T, d, "f16", outliers=8)
    a = _gpu_encode(X, D, s, csr.CSR_ENCODE_MFMA)
    b = _gpu_encode(X, D, s, csr.CSR_ENCODE_MFMA)
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])


def _adversarial_cases():
    rng = synth.stream(0, "misc", 3)
    N, d = 512, 128
    base = synth.dictionary(10, "dict_k", 1, N, d, "f16")[0].astype(np.float32)
    cases = {}
    # atoms far from unit norm (the screening bound scales with the largest atom norm)
    D = base.copy(); D[::7] *= 2.0; D[1::7] *= 0.25
    cases["atom norms 0.25 .. 2"] = (D, synth.vectors(10, "keys", 1, 200, d, "f16", outliers=8)[0])
    # duplicated atoms: exact ties in every iteration that picks one of them -> lowest index must win
    D = base.copy(); D[300:332] = D[10:42]
    X = synth.vectors(11, "keys", 1, 200, d, "f16", outliers=8)[0].astype(np.float32)
    X[:32] = D[10:42] * 3.0 + 0.01 * X[:32]
    cases["duplicated atoms"] = (D, X)
    # huge dynamic range inside one vector and across vectors (fp16 subnormals up to 3e4)
    X = synth.vectors(12, "values", 1, 200, d, "f16")[0].astype(np.float32)
    X *= np.exp(rng.uniform(-9.0, 2.0, size=X.shape)).astype(np.float32)
    X[:50] *= 3.0e3; X[50:100] *= 1.0e-4
    cases["dynamic range"] = (base, X)
    # vectors that are sparse combinations of atoms: the residual collapses after a few iterations
    X = np.zeros((200, d), dtype=np.float32)
    for t in range(200):
        k = rng.integers(1, 4)
        X[t] = (rng.standard_normal(k).astype(np.float32)[:, None] * base[rng.integers(0, N, k)]).sum(0)
    cases["sparse combinations of atoms"] = (base, X)
    # constant vectors and single-channel vectors
    X = np.zeros((64, d), dtype=np.float32); X[:32] = 1.5; X[32:, 5] = -7.0
    cases["constant and one-hot vectors"] = (base, X)
    return cases


@pytest.mark.parametrize("name", ["atom norms 0.25 .. 2", "duplicated atoms", "dynamic range",
                                  "sparse combinations of atoms", "constant and one-hot vectors"])
@pytest.mark.parametrize("algo", ["valu", "mfma", "split", "resident"])
def test_adversarial_inputs(algo, name):
    D, X = _adversarial_cases()[name]
    if algo == "split":
        X = X[:SPLIT_MAX]
    D16, X16 = D.astype(np.float16)[None], X.astype(np.float16)[None]
    s = 8
    idx, coef = _gpu_encode(X16, D16, s, ALGOS[algo])
    assert np.all(np.isfinite(coef.astype(np.float32)))
    reports = _compare(X16, D16, s, idx, coef)
    for rep in reports:
        assert rep.ok, name + ": " + rep.summary() + "\n" + "\n".join(rep.failures)
    print(f"[encode parity] {name} ({algo}): " + reports[0].summary())


# --- chunked vectors (the s_n of Section "NeuralDict"; the experiments store values with s = 4, s_n = 2) -----

def _compare_chunked(X, D, s, idx_g, coef_g):
    """X [H, T, d], D [H, sn, N, dc], codes [H, T, sn, s]: every chunk against the oracle's plain encoder."""
    H, sn, _, dc = D.shape
    reports = []
    for h in range(H):
        for c in range(sn):
            Xc = np.ascontiguousarray(X[h][:, c * dc:(c + 1) * dc])
            idx_o, coef_o, diag = oracle.mp_encode(Xc, D[h, c], s, diagnostics=True)
            coef_o_st = coef_o.astype(coef_g.dtype).astype(np.float64)
            reports.append(parity.check_encode(Xc, D[h, c], idx_g[h][:, c], coef_g[h][:, c], idx_o, coef_o_st, diag, TOL,
                                               coef_storage="f16" if coef_g.dtype == np.float16 else "f32",
                                               coef_o_exact=coef_o))
    return reports


@pytest.mark.parametrize("algo", ["valu", "mfma"])
@pytest.mark.parametrize("H,T,N,d,sn,s", [
    (2, 700, 1024, 128, 2, 4),     # the value cache of the experiments: two chunks of 64, four pairs each
    (1, 300, 4096, 128, 2, 8),
    (3, 257, 96, 128, 2, 3),       # a partial last stage of the dictionary (96 of 128 atoms), ragged tokens
    (2, 130, 512, 256, 2, 4),      # two chunks of 128
    (2, 100, 2080, 256, 4, 2),     # four chunks of 64
])
def test_chunked_vectors_every_chunk_on_its_own_dictionary(algo, H, T, N, d, sn, s):
    dc = d // sn
    D = synth.dictionary(31, "dict_v", H * sn, N, dc, "f16").reshape(H, sn, N, dc)
    X = synth.vectors(31, "values", H, T, d, "f16")
    idx, coef = _gpu_encode(X, D, s, ALGOS[algo])
    assert idx.shape == coef.shape == (H, T, sn, s)
    # the oracle's own chunked entry point has the same layout
    io, co = oracle.mp_encode_chunked(X[0], D[0], s)
    assert io.shape == idx[0].shape
    _assert_ok(_compare_chunked(X, D, s, idx.view(np.uint16).astype(np.int32), coef))


@pytest.mark.parametrize("H,T,N,d,sn,s", [
    (2, 700, 1024, 128, 4, 2),     # s_n = 4 of the dictionary-size tables of Section "NeuralDict": four chunks of 32
    (1, 300, 4096, 128, 4, 4),
    (3, 257, 96, 128, 4, 3),       # a partial dictionary stage (96 of 256 atoms), ragged tokens
    (2, 500, 320, 32, 1, 6),       # vectors of 32 dimensions, a stage and a quarter
    (64, 2100, 160, 128, 4, 2),    # 8-wave workgroups with a ragged last tile
])
def test_mfma_chunks_of_32_dimensions(H, T, N, d, sn, s):
    dc = d // sn
    D = synth.dictionary(34, "dict_v", H * sn, N, dc, "f16").reshape(H, sn, N, dc)
    X = synth.vectors(34, "values", H, T, d, "f16", outliers=2)
    Dg = torch.from_numpy(D if sn > 1 else D[:, 0]).cuda()
    idx, coef = csr.csr_encode(torch.from_numpy(X).cuda(), Dg, s, algo=csr.CSR_ENCODE_MFMA)
    ia, ca = csr.csr_encode(torch.from_numpy(X).cuda(), Dg, s)
    torch.cuda.synchronize()
    assert torch.equal(idx, ia) and torch.equal(coef, ca)          # what AUTO runs for these shapes
    idx, coef = idx.cpu().numpy().reshape(H, T, sn, s), coef.cpu().numpy().reshape(H, T, sn, s)
    heads = range(H) if H <= 3 else [0, 31, 63]
    _assert_ok(_compare_chunked(X[list(heads)], D[list(heads)], s, idx[list(heads)].view(np.uint16).astype(np.int32),
                                coef[list(heads)]))
    assert int(idx.view(np.uint16).max()) < N


@pytest.mark.parametrize("N", [32, 64, 160, 4096])
def test_mfma_vectors_of_64_dimensions(N):
    H, T, d, s = 2, 500, 64, 6
    D = synth.dictionary(32, "dict_k", H, N, d, "f16")
    X = synth.vectors(32, "keys", H, T, d, "f16", outliers=4)
    idx, coef = _gpu_encode(X, D, s, csr.CSR_ENCODE_MFMA)
    _assert_ok(_compare(X, D, s, idx.view(np.uint16).astype(np.int32), coef))


def test_chunked_mfma_and_valu_agree_and_strided_input():
    H, T, N, d, sn, s = 2, 400, 1024, 128, 2, 4
    D = synth.dictionary(33, "dict_v", H * sn, N, d // sn, "f16").reshape(H, sn, N, d // sn)
    X = synth.vectors(33, "values", H, T, d, "f16")
    wide = torch.zeros(H, T, 2 * d, dtype=torch.float16, device="cuda")
    wide[:, :, d:] = torch.from_numpy(X).cuda()
    Dg = torch.from_numpy(D).cuda()
    im, cm = csr.csr_encode(wide[:, :, d:], Dg, s, algo=csr.CSR_ENCODE_MFMA)
    iv, cv = csr.csr_encode(torch.from_numpy(X).cuda(), Dg, s, algo=csr.CSR_ENCODE_VALU)
    torch.cuda.synchronize()
    same = (im == iv).all(dim=-1).float().mean().item()
    assert same > 0.999          # the two encoders may part only at ties
    _assert_ok(_compare_chunked(X, D, s, im.cpu().numpy().view(np.uint16).astype(np.int32), cm.cpu().numpy()))


# --- few vectors per dictionary: the tokens of a decoding step (Section "KV Decomposition and Sparse Storage") ---

@pytest.mark.parametrize("H,T,N,d,sn,s,dicts", [
    (8, 1, 4096, 128, 1, 8, 8),       # one new token for each of 8 heads
    (16, 1, 4096, 128, 1, 8, 4),      # 4 sequences x 4 heads sharing the heads' dictionaries
    (3, 33, 1024, 128, 1, 6, 3),      # two blocks of 32 vectors, the second with one
    (2, 128, 512, 128, 1, 4, 2),      # the most vectors it takes
    (24, 5, 2080, 128, 1, 5, 2),      # 60 vectors per dictionary, 65 tiles over uneven slices
    (2, 7, 96, 128, 1, 8, 2),         # three tiles: fewer than waves
    (4, 2, 1024, 128, 2, 4, 2),       # values in two chunks of 64
    (6, 3, 256, 64, 1, 8, 3),         # 64-dimensional vectors
])
def test_split_encoder_parity(H, T, N, d, sn, s, dicts):
    dc = d // sn
    D = synth.dictionary(41, "dict_v", dicts * sn, N, dc, "f16").reshape(dicts, sn, N, dc)
    X = synth.vectors(41, "values", H, T, d, "f16", outliers=4)
    Dg = torch.from_numpy(D if sn > 1 else D[:, 0]).cuda()
    idx, coef = csr.csr_encode(torch.from_numpy(X).cuda(), Dg, s, algo=csr.CSR_ENCODE_SPLIT)
    torch.cuda.synchronize()
    idx, coef = idx.cpu().numpy().reshape(H, T, sn, s), coef.cpu().numpy().reshape(H, T, sn, s)
    D_blocks = np.stack([D[h % dicts] for h in range(H)])               # block h uses dictionary h % dicts
    _assert_ok(_compare_chunked(X, D_blocks, s, idx.view(np.uint16).astype(np.int32), coef))


def test_auto_picks_the_split_encoder_for_a_decoding_step_and_storage_types_do_not_move_indices():
    H, T, N, d, s = 8, 1, 1024, 128, 8
    D = synth.dictionary(42, "dict_k", H, N, d, "f16")
    X = synth.vectors(42, "keys", H, T, d, "f16", outliers=8)
    Xg, Dg = torch.from_numpy(X).cuda(), torch.from_numpy(D).cuda()
    ia, ca = csr.csr_encode(Xg, Dg, s)
    isp, csp = csr.csr_encode(Xg, Dg, s, algo=csr.CSR_ENCODE_SPLIT)
    i32, c32 = csr.csr_encode(Xg, Dg, s, algo=csr.CSR_ENCODE_SPLIT, coef_dtype=torch.float32, idx_dtype=torch.int32)
    im, cm = csr.csr_encode(Xg, Dg, s, algo=csr.CSR_ENCODE_MFMA)
    torch.cuda.synchronize()
    assert torch.equal(ia, isp) and torch.equal(ca, csp)                 # same kernel, same bits
    assert np.array_equal(isp.cpu().numpy().view(np.uint16).astype(np.int32), i32.cpu().numpy())
    assert np.array_equal(csp.cpu().numpy(), c32.cpu().numpy().astype(np.float16))
    assert (im == isp).all(dim=-1).float().mean().item() >= 0.75         # the encoders may part only at ties
    _assert_ok(_compare(X, D, s, i32.cpu().numpy(), c32.cpu().numpy()))


@pytest.mark.parametrize("algo", ["split", "mfma", "valu", "resident"])
def test_append_in_place_into_a_cache_of_codes(algo):
    # the codes of one new token per (sequence, head) land at row `pos` of a cache [blocks][T_max][s]
    B, Hkv, T_max, N, d, s, pos = 3, 4, 50, 512, 128, 8, 17
    D = synth.dictionary(43, "dict_k", Hkv, N, d, "f16")
    X = synth.vectors(43, "keys", B * Hkv, 1, d, "f16", outliers=8)
    Xg, Dg = torch.from_numpy(X).cuda(), torch.from_numpy(D).cuda()
    cache_i = torch.full((B * Hkv, T_max, s), -7, dtype=torch.int16, device="cuda")
    cache_c = torch.full((B * Hkv, T_max, s), 123.0, dtype=torch.float16, device="cuda")
    csr.csr_encode(Xg, Dg, s, algo=ALGOS[algo], idx=cache_i[:, pos:pos + 1], coef=cache_c[:, pos:pos + 1])
    i_ref, c_ref = csr.csr_encode(Xg, Dg, s, algo=ALGOS[algo])
    torch.cuda.synchronize()
    assert torch.equal(cache_i[:, pos:pos + 1], i_ref) and torch.equal(cache_c[:, pos:pos + 1], c_ref)
    keep = torch.ones(T_max, dtype=torch.bool, device="cuda"); keep[pos] = False
    assert (cache_i[:, keep] == -7).all() and (cache_c[:, keep] == 123.0).all()    # neighbours untouched
    D_blocks = np.stack([D[h % Hkv] for h in range(B * Hkv)])
    _assert_ok(_compare(X, D_blocks, s, i_ref.cpu().numpy(), c_ref.cpu().numpy()))


def test_split_results_do_not_depend_on_the_run():
    H, T, N, d, s = 16, 4, 4096, 128, 8
    D = synth.dictionary(44, "dict_k", H, N, d, "f16")
    X = synth.vectors(44, "keys", H, T, d, "f16", outliers=8)
    a = _gpu_encode(X, D, s, csr.CSR_ENCODE_SPLIT)
    b = _gpu_encode(X, D, s, csr.CSR_ENCODE_SPLIT)
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])


def test_chunked_values_full_size_sampled():
    # bench.py's chunked_step value launch: 32 heads x 4096 vectors, two chunks of 64, s = 4, N = 4096 per chunk
    w = synth.WORKLOADS["llama7b_layer"]
    sn, s = 2, 4
    D = synth.dictionary(0, "dict_v", w.hkv * sn, w.n_atoms, w.d // sn, "f16").reshape(w.hkv, sn, w.n_atoms, w.d // sn)
    X = synth.vectors(0, "values", w.hkv, w.tokens, w.d, "f16")
    idx, coef = _gpu_encode(X, D, s, csr.CSR_ENCODE_AUTO)
    assert idx.shape == (w.hkv, w.tokens, sn, s) and int(idx.view(np.uint16).max()) < w.n_atoms
    rows = np.unique(np.concatenate([[0, 255, 256, w.tokens - 1], synth.stream(0, "misc", 4).integers(0, w.tokens, 12)]))
    _assert_ok(_compare_chunked(X[:, rows], D, s, idx[:, rows].view(np.uint16).astype(np.int32), coef[:, rows]))


def test_decoding_step_full_size_one_token_for_every_head_of_a_layer():
    # bench.py's decode_step append: keys' and values' new vectors of 32 heads stacked, 64 dictionaries, one call
    w = synth.WORKLOADS["llama7b_layer"]
    D = np.concatenate([synth.dictionary(0, "dict_k", w.hkv, w.n_atoms, w.d, "f16"),
                        synth.dictionary(0, "dict_v", w.hkv, w.n_atoms, w.d, "f16")])
    X = np.concatenate([synth.vectors(1, "keys", w.hkv, 1, w.d, "f16", outliers=w.key_outliers),
                        synth.vectors(1, "values", w.hkv, 1, w.d, "f16")])
    idx, coef = _gpu_encode(X, D, w.s, csr.CSR_ENCODE_AUTO)
    _assert_ok(_compare(X, D, w.s, idx, coef))
    # a batch of 16 sequences sharing the 64 dictionaries: 16 vectors per dictionary
    B = 16
    Xb = np.concatenate([synth.vectors(2 + b, "values", 2 * w.hkv, 1, w.d, "f16") for b in range(B)])
    ib, cb = csr.csr_encode(torch.from_numpy(Xb).cuda(), torch.from_numpy(D).cuda(), w.s)
    torch.cuda.synchronize()
    blocks = [0, 63, 64, 500, B * 2 * w.hkv - 1]
    Db = np.stack([D[h % (2 * w.hkv)] for h in blocks])
    _assert_ok(_compare(Xb[blocks], Db, w.s, ib.cpu().numpy()[blocks], cb.cpu().numpy()[blocks]))


@pytest.mark.parametrize("algo", ["valu", "mfma", "split", "resident"])
@pytest.mark.parametrize("sn", [1, 2])
def test_residual_norm_output_is_the_reconstruction_error(algo, sn):
    # |R_{s+1}|^2 per vector (chunk): the vector's term of the dictionary-training loss of Section "NeuralDict"
    H, T, N, d, s = 3, 100, 512, 128, 6
    dc = d // sn
    D = synth.dictionary(61, "dict_v", H * sn, N, dc, "f16").reshape(H, sn, N, dc)
    X = synth.vectors(61, "values", H, T, d, "f16", outliers=4)
    X[0, 0] = 0                                                       # a zero vector leaves nothing
    X[1, 1, :dc] = (D[1, 0, 7].astype(np.float32) * 3).astype(np.float16)   # a multiple of an atom leaves ~nothing
    Dg = torch.from_numpy(D if sn > 1 else D[:, 0]).cuda()
    shape = (H, T, sn) if sn > 1 else (H, T)
    rn = torch.full(shape, -1.0, dtype=torch.float32, device="cuda")
    idx, coef = csr.csr_encode(torch.from_numpy(X).cuda(), Dg, s, algo=ALGOS[algo], coef_dtype=torch.float32,
                               idx_dtype=torch.int32, res_norm2=rn)
    torch.cuda.synchronize()
    rn = rn.cpu().numpy().reshape(H, T, sn)
    idx, coef = idx.cpu().numpy().reshape(H, T, sn, s), coef.cpu().numpy().reshape(H, T, sn, s)
    for h in range(H):
        for c in range(sn):
            Xc = X[h][:, c * dc:(c + 1) * dc].astype(np.float64)
            # what the GPU's own pairs leave (they may differ from the oracle's at ties): x - D r in float64
            err = ((Xc - oracle.reconstruct(idx[h, :, c], coef[h, :, c], D[h, c])) ** 2).sum(axis=1)
            x2 = (Xc ** 2).sum(axis=1)
            assert np.all(np.abs(rn[h, :, c] - err) <= 1e-4 * err + 1e-6 * x2), (algo, h, c, np.abs(rn[h, :, c] - err).max())
            _, _, diag = oracle.mp_encode(Xc, D[h, c], s, diagnostics=True)
            close = np.abs(rn[h, :, c] - diag["res_norm2"][:, s]) <= 1e-3 * x2
            assert close.mean() > 0.97                                 # the oracle's own path, except after ties
    assert rn[0, 0, 0] == 0.0 and rn[1, 1, 0] <= 1e-5 * float((X[1, 1, :dc].astype(np.float64) ** 2).sum())


# --- small dictionaries kept in LDS (the 256 - 512 atoms per head of the paper's experiments) -------------------

@pytest.mark.parametrize("H,T,N,d,sn,s,dicts", [
    (4, 1000, 256, 128, 1, 8, 4),      # the paper's 256 atoms per head
    (3, 777, 512, 128, 1, 8, 3),       # the largest dictionary of 128-dimensional atoms that fits
    (2, 513, 32, 128, 1, 4, 2),        # one tile; a second workgroup with a single vector
    (6, 300, 1024, 128, 2, 4, 3),      # values in two chunks of 64, 1024 atoms each; blocks sharing dictionaries
    (2, 2000, 96, 64, 1, 6, 2),        # 64-dimensional vectors, three tiles
])
def test_resident_encoder_parity(H, T, N, d, sn, s, dicts):
    dc = d // sn
    D = synth.dictionary(71, "dict_k", dicts * sn, N, dc, "f16").reshape(dicts, sn, N, dc)
    X = synth.vectors(71, "keys", H, T, d, "f16", outliers=8)
    Dg = torch.from_numpy(D if sn > 1 else D[:, 0]).cuda()
    idx, coef = csr.csr_encode(torch.from_numpy(X).cuda(), Dg, s, algo=csr.CSR_ENCODE_RESIDENT)
    ia, ca = csr.csr_encode(torch.from_numpy(X).cuda(), Dg, s)
    torch.cuda.synchronize()
    assert torch.equal(idx, ia) and torch.equal(coef, ca)             # what AUTO runs for these shapes
    idx, coef = idx.cpu().numpy().reshape(H, T, sn, s), coef.cpu().numpy().reshape(H, T, sn, s)
    D_blocks = np.stack([D[h % dicts] for h in range(H)])
    _assert_ok(_compare_chunked(X, D_blocks, s, idx.view(np.uint16).astype(np.int32), coef))


def test_resident_encoder_is_refused_for_dictionaries_beyond_the_lds():
    D = torch.zeros(1, 544, 128, dtype=torch.float16, device="cuda")
    X = torch.zeros(1, 200, 128, dtype=torch.float16, device="cuda")
    with pytest.raises(csr.CsrError, match="128 KB"):
        csr.csr_encode(X, D, 4, algo=csr.CSR_ENCODE_RESIDENT)


def test_dictionaries_beyond_sixteen_bit_indices():
    # 70016 atoms need 32-bit indices: the split encoder (few vectors) and the vector-ALU encoder (AUTO's choice for
    # many vectors, the matrix-core kernel stops at 65536 atoms) against the oracle
    N, d, s = 70016, 128, 3
    D = synth.dictionary(81, "dict_k", 1, N, d, "f16")
    X = synth.vectors(81, "keys", 1, 140, d, "f16", outliers=8)
    Dg = torch.from_numpy(D).cuda()
    for rows in (slice(0, 5), slice(0, 140)):
        idx, coef = csr.csr_encode(torch.from_numpy(X[:, rows]).cuda(), Dg, s, idx_dtype=torch.int32)
        torch.cuda.synchronize()
        assert idx.dtype == torch.int32 and int(idx.max()) < N
        _assert_ok(_compare(X[:, rows], D, s, idx.cpu().numpy(), coef.cpu().numpy()))
    with pytest.raises(csr.CsrError, match="16-bit"):
        csr.csr_encode(torch.from_numpy(X).cuda(), Dg, s, idx_dtype=torch.int16)


@pytest.mark.parametrize("algo", ["mfma", "valu", "resident"])
def test_blocks_that_share_a_dictionary_are_packed_into_tiles_together(algo):
    # 75 sequences x 4 heads with 3 new vectors each: 225 vectors per dictionary, spread over 75 blocks, written
    # in place into a cache of codes; every block must get exactly its own vectors' codes
    B, Hkv, T, T_max, N, d, s, pos = 75, 4, 3, 11, 512, 128, 5, 6
    D = synth.dictionary(91, "dict_k", Hkv, N, d, "f16")
    X = synth.vectors(91, "keys", B * Hkv, T, d, "f16", outliers=8)
    ci = torch.full((B * Hkv, T_max, s), -3, dtype=torch.int16, device="cuda")
    cc = torch.full((B * Hkv, T_max, s), 77.0, dtype=torch.float16, device="cuda")
    rn = torch.full((B * Hkv, T), -1.0, dtype=torch.float32, device="cuda")
    csr.csr_encode(torch.from_numpy(X).cuda(), torch.from_numpy(D).cuda(), s, algo=ALGOS[algo],
                   idx=ci[:, pos:pos + T], coef=cc[:, pos:pos + T], res_norm2=rn)
    torch.cuda.synchronize()
    keep = torch.ones(T_max, dtype=torch.bool, device="cuda"); keep[pos:pos + T] = False
    assert (ci[:, keep] == -3).all() and (cc[:, keep] == 77.0).all() and (rn >= 0).all()
    blocks = [0, 1, 5, 150, 151, 298, 299]
    Db = np.stack([D[h % Hkv] for h in blocks])
    _assert_ok(_compare(X[blocks], Db, s, ci[:, pos:pos + T].cpu().numpy()[blocks], cc[:, pos:pos + T].cpu().numpy()[blocks]))
    # and all blocks agree with a call that gives every block its own (repeated) dictionary
    i2, c2 = csr.csr_encode(torch.from_numpy(X).cuda(), torch.from_numpy(np.tile(D, (B, 1, 1))).cuda(), s, algo=ALGOS[algo])
    torch.cuda.synchronize()
    assert torch.equal(i2, ci[:, pos:pos + T]) and torch.equal(c2, cc[:, pos:pos + T])


def test_mfma_eight_wave_workgroups_with_a_ragged_last_tile():
    # 64 dictionaries x 2100 vectors: five 512-vector workgroups per dictionary (at least one per CU in all, so the
    # 8-wave configuration runs), the last with 52 vectors; 96 atoms leave a partial dictionary stage as well
    H, T, N, d, s = 64, 2100, 96, 128, 3
    D = synth.dictionary(95, "dict_k", H, N, d, "f16")
    X = synth.vectors(95, "keys", H, T, d, "f16", outliers=8)
    idx, coef = _gpu_encode(X, D, s, csr.CSR_ENCODE_MFMA)
    rows = np.array([0, 63, 64, 511, 512, 2047, 2048, 2049, 2098, 2099])
    _assert_ok(_compare(X, D, s, idx, coef, heads=[0, 1, 31, 62, 63], rows=rows))
    iv, cv = _gpu_encode(X, D, s, csr.CSR_ENCODE_VALU)
    same = (idx == iv).all(axis=-1).mean()
    assert same > 0.995, same          # all vectors, against the other encoder: they may part at ties only


# --- Eq.4 with the stored coefficient (CSR_FLAG_CLOSED_LOOP; Section "Analysis for CSR" stores fp16) -------------

def _compare_closed(X, D, s, idx_g, coef_g):
    reports = []
    for h in range(X.shape[0]):
        idx_o, coef_o, diag = oracle.mp_encode(X[h], D[h], s, diagnostics=True, closed_loop="f16")
        reports.append(parity.check_encode(X[h], D[h], idx_g[h], coef_g[h], idx_o, coef_o, diag, TOL, coef_storage="f16"))
    return reports


@pytest.mark.parametrize("algo", ["valu", "mfma", "split", "resident"])
def test_closed_loop_matches_the_oracles_closed_loop(algo):
    H, T, N, d, s = 2, 300 if algo != "split" else 100, 512, 128, 8
    D = synth.dictionary(101, "dict_k", H, N, d, "f16")
    X = synth.vectors(101, "keys", H, T, d, "f16", outliers=8)
    Xg, Dg = torch.from_numpy(X).cuda(), torch.from_numpy(D).cuda()
    rn = torch.empty(H, T, dtype=torch.float32, device="cuda")
    idx, coef = csr.csr_encode(Xg, Dg, s, algo=ALGOS[algo], closed_loop=True, res_norm2=rn)
    io, co = csr.csr_encode(Xg, Dg, s, algo=ALGOS[algo])
    torch.cuda.synchronize()
    idx, coef = idx.cpu().numpy(), coef.cpu().numpy()
    reports = _compare_closed(X, D, s, idx, coef)
    for rep in reports:
        assert rep.ok, rep.summary() + "\n" + "\n".join(rep.failures)
    print(f"[encode parity] closed loop ({algo}): " + reports[0].summary())
    # the two readings do part: later coefficients (and, now and then, atoms) change once the rounding of an early
    # coefficient stays in the residual
    assert (idx != io.cpu().numpy()).any() or (coef != co.cpu().numpy()).any()
    # and the reported residual norm is the error of the code AS STORED
    for h in range(H):
        err = ((X[h].astype(np.float64) - oracle.reconstruct(idx[h], coef[h], D[h])) ** 2).sum(axis=1)
        x2 = (X[h].astype(np.float64) ** 2).sum(axis=1)
        assert np.all(np.abs(rn[h].cpu().numpy() - err) <= 1e-4 * err + 1e-6 * x2)


@pytest.mark.parametrize("algo", ["valu", "mfma", "split", "resident"])
def test_closed_loop_third_pick_differs_from_the_open_loop_on_a_nearly_orthonormal_dictionary(algo):
    # identity atoms, the first turned by a small angle so that the first projection (1000 cos a + 0.1 sin a) is not
    # an fp16 value: the stored 1000.0 leaves +0.002 of the first atom in the closed-loop residual, which changes
    # the third pick (atom 1 with +0.00195 instead of atom 0 with -0.002: what the oracle's two readings give)
    d = 128
    D2 = np.eye(d, dtype=np.float16)[None].copy()
    a = 0.02
    D2[0, 0, 0], D2[0, 0, 1] = np.float16(np.cos(a)), np.float16(np.sin(a))
    X = np.zeros((1, 40, d), dtype=np.float16)
    X[0, :, 0] = np.float16(1000.0)
    X[0, :, 1] = np.float16(0.1)
    idx, coef = _gpu_encode_closed(X, D2, 3, ALGOS[algo])
    io, co, diag = oracle.mp_encode(X[0], D2[0], 3, diagnostics=True, closed_loop="f16")
    rep = parity.check_encode(X[0], D2[0], idx[0], coef[0], io, co, diag, TOL, coef_storage="f16")
    assert rep.ok, rep.summary() + "\n" + "\n".join(rep.failures)
    assert io[0].tolist() == [0, 1, 1] and np.array_equal(idx[0].view(np.uint16).astype(np.int64), io)
    assert oracle.mp_encode(X[0], D2[0], 3)[0][0].tolist() == [0, 1, 0]


def _gpu_encode_closed(X, D, s, algo):
    idx, coef = csr.csr_encode(torch.from_numpy(X).cuda(), torch.from_numpy(D).cuda(), s, algo=algo, closed_loop=True)
    torch.cuda.synchronize()
    return idx.cpu().numpy(), coef.cpu().numpy()


def test_closed_loop_with_fp32_coefficients_is_the_open_loop():
    H, T, N, d, s = 2, 200, 512, 128, 6
    D = synth.dictionary(102, "dict_k", H, N, d, "f16")
    X = synth.vectors(102, "keys", H, T, d, "f16", outliers=8)
    Xg, Dg = torch.from_numpy(X).cuda(), torch.from_numpy(D).cuda()
    for algo in (csr.CSR_ENCODE_MFMA, csr.CSR_ENCODE_VALU):
        a = csr.csr_encode(Xg, Dg, s, algo=algo, coef_dtype=torch.float32, closed_loop=True)
        b = csr.csr_encode(Xg, Dg, s, algo=algo, coef_dtype=torch.float32)
        torch.cuda.synchronize()
        assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])
    with pytest.raises(csr.CsrError, match="CLOSED_LOOP"):
        csr.csr_encode(Xg[:, :4], Dg[:, :256], s, algo=csr.CSR_ENCODE_GRAM, closed_loop=True)


def _least_us(call, runs=12, calls=4):
    best = np.inf
    for _ in range(runs):
        start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        call()
        start.record()
        for _ in range(calls):
            call()
        end.record()
        end.synchronize()
        best = min(best, start.elapsed_time(end) * 1000 / calls)
    return best


@pytest.mark.parametrize("algo,T,N,d", [("resident", 257, 512, 128), ("resident", 513, 512, 64), ("mfma", 257, 1024, 128), ("mfma", 65, 1024, 64),
                                        ("wide", 33, 1024, 128)])
def test_copies_of_the_last_vector_past_the_end_are_not_resolved(algo, T, N, d):
    # lanes past the last vector work on copies of it.  A last vector that no bound decides (four sums of atoms that are there
    # three times) costs what any undecided vector costs, not a resolve for each of its copies, one after the other
    D = synth.dictionary(110, "dict_k", 1, N, d, "f16")
    D[0, N // 2:N // 2 + 4] = D[0, :4]
    D[0, N - 4:] = D[0, :4]
    X = synth.vectors(110, "values", 1, T, d, "f16")
    tied = X.copy()
    tied[0, -1] = (np.array([8, 4, 2, 1], dtype=np.float32) @ D[0, :4].astype(np.float32)).astype(np.float16)
    Dg, run = torch.from_numpy(D).cuda(), {"wide": csr.CSR_ENCODE_WIDE, **ALGOS}[algo]
    calls = [lambda x=torch.from_numpy(x).cuda(): csr.csr_encode(x, Dg, 4, algo=run) for x in (X, tied)]
    idx = calls[1]()[0].cpu().numpy()
    assert idx[0, -1, 0] == 0
    plain, undecided = (_least_us(c) for c in calls)
    assert undecided < 1.4 * plain, (plain, undecided)   # with the copies 2 to 7 times as long


@pytest.mark.parametrize("heads,T,N,s_n", [(32, 1289, 2048, 2), (3, 31799, 2048, 1), (12, 5666, 640, 1), (8, 4812, 2560, 2), (4, 22694, 4096, 1)])
def test_auto_takes_neither_the_slower_encoder(heads, T, N, s_n):
    # partial generations of the prefill encoder cost nearly a full one: priced below that, it was taken here and 12 to 28 % slower than
    # the wide encoder.  The least of ten times each is repeatable to 2 %
    s, d = 4, 128 // s_n
    gen = torch.Generator(device="cuda")
    gen.manual_seed(111)
    D = torch.randn((heads, s_n, N, d) if s_n > 1 else (heads, N, d), device="cuda", generator=gen)
    D = (D / D.norm(dim=-1, keepdim=True)).half()
    X = torch.randn(heads, T, 128, device="cuda", generator=gen).half()
    auto, mfma, wide = (_least_us(lambda a=a: csr.csr_encode(X, D, s, algo=a), runs=10, calls=2)
                        for a in (csr.CSR_ENCODE_AUTO, csr.CSR_ENCODE_MFMA, csr.CSR_ENCODE_WIDE))
    assert auto < 1.1 * min(mfma, wide), (auto, mfma, wide)
