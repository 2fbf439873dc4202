"""What the compiler made of the kernels that stand or fall with it, from the metadata of the built library: needs no GPU."""
import os
import re
import subprocess

import pytest

from paper_2412_11741_amd import binding

READELF = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-readelf")


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{mangled name: metadata} of every kernel in libcsr_hip.so: its code objects are ELF images inside the host's one."""
    if not os.path.exists(READELF):
        pytest.skip("no llvm-readelf")
    binding.lib()
    image, found = open(binding.LIB_PATH, "rb").read(), {}
    path = tmp_path_factory.mktemp("code") / "object"
    for at in (m.start() for m in re.finditer(rb"\x7fELF\x02\x01\x01\x40", image)):   # 0x40: AMD GPU HSA
        path.write_bytes(image[at:])
        notes = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True).stdout
        for block in re.split(r"\n  - \.", notes):
            name, fields = re.search(r"\.name: +(\S+)", block), dict(re.findall(r"\.?(\w+): +(\d+)", block))
            if name and "private_segment_fixed_size" in fields:
                found[name.group(1)] = {k: int(v) for k, v in fields.items()}
    return found


def test_the_streaming_kernels_keep_their_scores_in_registers(kernels):
    # a thread's scores, one per round and query head, are an array that is only in registers if every loop over it is
    # unrolled and everything that takes it is inlined; else every score goes through scratch memory
    stream = {n: k["private_segment_fixed_size"] for n, k in kernels.items() if "13stream_kernel" in n}
    assert len(stream) > 50

    def scores(name):   # bytes of the array: query heads x rounds
        heads, rounds = re.search(r"stream_kernelILi(\d+)E.*?Lb[01]ELi(\d+)E", name).groups()
        return 4 * int(heads) * int(rounds)
    # (up to 25 spilled registers in the variants for two query heads)
    assert not {n: v for n, v in stream.items() if v >= max(scores(n), 128)}


def test_rotary_kernels_spill_no_more_for_value_codes_requested_ahead(kernels):
    # variants of the same kernel by NP, the pairs of a value code that is requested as a whole; 0: loaded where it is used
    by_shape = {}
    for n, k in kernels.items():
        m = re.search(r"stream_rope_kernelILi(\d+)ELb(\d)ELi(\d+)ELb(\d)ELi\d+ELi(\d+)ELi\d+ELb(\d)E", n)
        if m:
            heads, rotk, pvk, oneb, pairs, rows_gathered = m.groups()
            by_shape.setdefault((heads, rotk, pvk, oneb, rows_gathered), {}).setdefault(int(pairs), []).append(k["private_segment_fixed_size"])
    assert len(by_shape) > 8
    for shape, sizes in by_shape.items():
        assert max(map(max, sizes.values())) <= max(sizes[0]), shape


def test_only_long_chunks_carry_the_cut_by_lengths(kernels):
    # whole codes: a variant with the cut and one without where a chunk may be long enough for it, else one without
    found = {}
    for n in kernels:
        m = re.search(r"stream_kernelILi(\d+)E(t|i)(.*?)Li(\d+)ELb(\d)ELi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)E", n)
        if m:
            heads, index, coef, piece, chunked, rounds, pairs, threads, cut_from = m.groups()
            if int(pairs) > 0:
                found.setdefault((heads, chunked, pairs, int(rounds) * int(threads)), set()).add(int(cut_from))
    assert len(found) > 30
    assert {k: v for k, v in found.items() if v != ({0, 12288} if k[3] >= 12288 else {0})} == {}


def test_the_wide_encoder_spills_little(kernels):
    # vectors of 128 dimensions in passes of 32: with four and five of them a few registers more than there are
    wide = {n: k["vgpr_spill_count"] for n, k in kernels.items() if "encode_wide_kernel" in n}
    assert len(wide) > 20
    assert {n: v for n, v in wide.items() if v > (20 if re.search(r"Li128ELi[01]ELi8ELi[45]E", n) else 0)} == {}


def test_split_encoder_workgroups_of_64_dimensions_share_a_cu(kernels):
    # eight waves a workgroup: two of them on a CU take at most 128 registers a lane.  With four tiles a lane there is one, as with 128 dimensions
    split = {}
    for n, k in kernels.items():
        m = re.search(r"encode_split_kernelILi(\d+)ELi(\d)ELb(\d)E", n)
        if m:
            split[tuple(map(int, m.groups()))] = k
    assert len(split) == 12
    for (dims, held, _), k in split.items():
        if dims == 64 and held <= 2:
            assert k["vgpr_count"] <= 128 and k["vgpr_spill_count"] == 0, (dims, held)
        assert k["vgpr_spill_count"] <= (4 if (dims, held) == (128, 4) else 0), (dims, held)


def test_only_codes_of_whole_vectors_are_requested_past_the_l2s(kernels):
    # a variant with non-temporal requests where they are made: codes of 8 pairs, four query heads, long chunks, with the cut by lengths and without
    past = {}
    for n in kernels:
        m = re.search(r"13stream_kernelILi(\d+)E\w+?Lb(\d)ELi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELb1EE", n)
        if m:
            past[n] = tuple(map(int, m.groups()))
    assert sorted(past.values()) == [(4, 0, 32, 8, 512, 0), (4, 0, 32, 8, 512, 12288)]


def test_the_resident_encoder_spills_little(kernels):
    # 64 dimensions with two workgroups per CU have 128 registers: what is spilled is one vector's place, outside of the loop over the tiles
    resident = {}
    for n, k in kernels.items():
        m = re.search(r"encode_resident_kernelILi(\d+)ELi(\d)ELi(\d)E", n)
        if m:
            resident[tuple(map(int, m.groups()))] = k["vgpr_spill_count"]
    assert len(resident) == 6
    assert {n: v for n, v in resident.items() if v > (8 if n[:2] == (64, 4) else 0)} == {}


def test_streaming_kernels_for_four_heads_spill_little_where_codes_are_not_requested_whole(kernels):
    # the 32 scores of a thread leave few registers for the non-temporal stores' addresses: measured level with plain ones that spill none
    four = {n: k["vgpr_spill_count"] for n, k in kernels.items() if re.search(r"13stream_kernelILi4E\w+?Lb[01]ELi8ELi0E", n)}
    assert len(four) == 24
    assert max(four.values()) <= 6
