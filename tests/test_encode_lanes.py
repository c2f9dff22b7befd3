"""The kernels of the device compressor compiled for the CPU, lane by lane (tests/lanes/hip/hip_runtime.h): the lanes of a
workgroup run one at a time between the places where the source makes them meet, in three orders, with LDS, workspace and
results holding arbitrary bytes at the start.  The blob must be the oracle's in every order: then nothing is read before it is
written, and no access is right only because the lanes of a wave happen to keep in step."""
import os
import subprocess

import numpy as np
import pytest

import oracle.codec as oc
from tests.helpers import lopsided_bytes, weightlike_bytes

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CLANG = "/opt/rocm/llvm/bin/clang++"
ORDERS = {"ascending": 0, "descending": 1, "shuffled": 2}


@pytest.fixture(scope="module")
def encode(tmp_path_factory):
    d = tmp_path_factory.mktemp("lanes")
    exe, src, out = str(d / "encode"), str(d / "source"), str(d / "result")
    # no position-independent code: LDS variables have addresses of 32 bits, as on the device
    subprocess.run([CLANG, "-x", "c++", "-std=c++17", "-O1", "-no-pie", "-fno-pie", "-w", "-I", os.path.join(HERE, "lanes"),
                    "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2502_15443_amd", "csrc"),
                    os.path.join(HERE, "lanes", "encode.cpp"), "-o", exe], check=True)

    def run(order, seed, data, C, S, policy=oc.ALL_HUFF, f=0.0, block=0, codec=oc.HUFFMAN, over=()):
        data.tofile(src)
        done = subprocess.run([exe] + [str(v) for v in (ORDERS[order], seed, C, S, policy, f, block, codec)] + [src, out, *over],
                              capture_output=True, text=True, timeout=100)
        assert done.returncode == 0, (done.returncode, done.stderr)
        b = open(out, "rb").read()
        used, status, nc = (int(v) for v in np.frombuffer(b[:24], np.uint64))
        return used, status, np.frombuffer(b[24:24 + 16 * nc], oc.CHUNK_DTYPE), np.frombuffer(b[24 + 16 * nc:], np.uint8)

    return run


@pytest.mark.parametrize("order", list(ORDERS))
@pytest.mark.parametrize("S,codec", [(32, oc.HUFFMAN), (64, oc.HUFFMAN), (128, oc.HUFFMAN), (256, oc.HUFFMAN),
                                     (64, oc.TANS), (128, oc.TANS), (256, oc.TANS)])
def test_compressor_does_not_depend_on_the_order_of_the_lanes(encode, order, S, codec):
    r = np.random.default_rng(S)
    C = 16384
    tail = r.permutation(256)[np.minimum(r.geometric(0.03, C), 255)].astype(np.uint8)
    cases = [(weightlike_bytes(3 * C + 777, S), {}), (lopsided_bytes(C, S, 7), {}),
             (np.concatenate([np.zeros(C, np.uint8), r.integers(0, 256, C, dtype=np.uint8), tail, weightlike_bytes(C, 3)]),
              dict(policy=oc.RAW_FRACTION, f=0.3)),
             (np.concatenate([r.integers(0, 256, C, dtype=np.uint8), tail[:1234]]), dict(policy=oc.AUTO)),
             (np.array([7], np.uint8), {})]
    for i, (data, options) in enumerate(cases):
        want = oc.compress(data, C, S, options.get("policy", oc.ALL_HUFF), options.get("f", 0.0), codec=codec)
        used, status, table, blob = encode(order, 11 * i + S, data, C, S, codec=codec, **options)
        assert status == 0 and used == want.blob.size, i
        assert np.array_equal(table, want.table), i
        assert np.array_equal(blob, want.blob), i


@pytest.mark.parametrize("order", list(ORDERS))
@pytest.mark.parametrize("over", ["result", "blob"])
@pytest.mark.parametrize("policy", [oc.ALL_HUFF, oc.AUTO])
def test_compressor_results_over_the_workspace(encode, order, over, policy):
    # nothing is written over the chunks' sizes while a workgroup may still add them up
    C = 8192
    data = weightlike_bytes(5 * C + 5, 4)
    want = oc.compress(data, C, 64, policy)
    used, status, table, blob = encode(order, 3, data, C, 64, policy=policy, over=(over,))
    assert status == 0 and used == want.blob.size
    assert np.array_equal(table, want.table) and np.array_equal(blob, want.blob)


def bytes_with_counts(counts, seed):
    """A shuffled string with these counts of the values 0, 1, ..."""
    data = np.repeat(np.arange(len(counts), dtype=np.uint8), counts)
    return np.random.default_rng(seed).permutation(data)


FIBONACCI = [1, 1, 2, 3, 5, 8, 13, 21, 34, 55, 89, 144, 233, 377, 610, 987, 1597, 2584, 4181, 6765]


@pytest.mark.parametrize("order", list(ORDERS))
@pytest.mark.parametrize("counts", [
    [1, 1], [3, 1], [1] * 256, [2] * 255, FIBONACCI,  # ties at every level; the length limit
    [255] * 2 + [256] * 2 + [257] * 2 + [510, 511, 512, 513],  # where a bucket of weights begins to hold several
    [256 + i // 9 for i in range(256)],  # many leaves in a bucket, packages between them
    [1] * 200 + [300 + 2 * i for i in range(56)],
    [2 ** 20 - 255] + [1] * 255])  # the heaviest leaf there is
def test_code_lengths_of_constructed_counts(encode, order, counts):
    # packages are counted among leaves of nearly and exactly their weight
    data = bytes_with_counts(counts, len(counts))
    C = (data.size + 15) // 16 * 16
    S = 256 if C < 1 << 20 else 32
    want = oc.compress(data, C, S)
    used, status, table, blob = encode(order, 5, data, C, S)
    assert status == 0 and used == want.blob.size
    assert np.array_equal(table, want.table) and np.array_equal(blob, want.blob)


@pytest.mark.parametrize("order", list(ORDERS))
@pytest.mark.parametrize("leaves", [2, 3, 63, 64, 65, 66, 128, 129])  # on both sides of the lines up to which a chunk has few
def test_code_lengths_of_few_leaves(encode, order, leaves):
    r = np.random.default_rng(leaves)
    counts = [np.full(leaves, 5), 1 + r.integers(0, 40, leaves), np.minimum(1 + (1.3 ** np.arange(leaves)).astype(int), 900)]
    parts = [np.concatenate([bytes_with_counts(c, leaves), np.zeros(4096, np.uint8)])[:8192] for c in counts]
    C = 8192
    data = np.concatenate([np.resize(p, C) for p in parts])
    want = oc.compress(data, C, 64)
    used, status, table, blob = encode(order, 5, data, C, 64)
    assert status == 0 and used == want.blob.size
    assert np.array_equal(table, want.table) and np.array_equal(blob, want.blob)


@pytest.mark.parametrize("chunks", [1024, 1025])
def test_code_lengths_of_few_leaves_in_many_chunks(encode, chunks):
    # beyond 1024 chunks more leaves are few
    C = 256
    data = np.random.default_rng(chunks).integers(0, 110, chunks * C - 3).astype(np.uint8)
    want = oc.compress(data, C, 64)
    used, status, table, blob = encode("shuffled", 5, data, C, 64)
    assert status == 0 and used == want.blob.size
    assert np.array_equal(table, want.table) and np.array_equal(blob, want.blob)
