"""The decode kernels compiled for the CPU, lane by lane, as in test_encode_lanes.py: bytes, bf16 values and both products must
be the oracle's whatever the order of the lanes between the places where the source makes them meet, and whatever LDS and the
workspace held."""
import os
import subprocess

import numpy as np
import pytest

import oracle.codec as oc
import oracle.quant as oq
import synth
from tests.helpers import oracle_matrix
from tests.test_encode_lanes import CLANG, HERE, ORDERS, ROOT

BYTES, BF16, PRODUCT, PRODUCT_INT8, TRACED = range(5)


@pytest.fixture(scope="module")
def decode(tmp_path_factory):
    d = tmp_path_factory.mktemp("lanes")
    exe, src, out = str(d / "decode"), str(d / "source"), str(d / "result")
    subprocess.run([CLANG, "-x", "c++", "-std=c++17", "-O1", "-no-pie", "-fno-pie", "-w", "-I", os.path.join(HERE, "lanes"),
                    "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2502_15443_amd", "csrc"),
                    os.path.join(HERE, "lanes", "decode.cpp"), "-o", exe], check=True)

    def run(order, c, C, S, codec, mode, rows, cols, *more, units=256):
        parts = [np.array([c.n_chunks, c.blob.size], np.uint64), c.table, c.blob, *more]
        with open(src, "wb") as f:
            f.write(b"".join(np.ascontiguousarray(a).tobytes() for a in parts))
        done = subprocess.run([exe] + [str(v) for v in (ORDERS[order], rows + mode, C, S, codec, mode, rows, cols)] + [src, out, str(units)],
                              capture_output=True, text=True, timeout=100)
        assert done.returncode == 0, (done.returncode, done.stderr)
        run.launched = done.stdout.split("\n")[:-1]
        return np.fromfile(out, np.uint8)

    run.exe = exe
    return run


@pytest.mark.parametrize("order", list(ORDERS))
@pytest.mark.parametrize("S,codec", [(32, oc.HUFFMAN), (64, oc.HUFFMAN), (128, oc.HUFFMAN), (256, oc.HUFFMAN),
                                     (64, oc.TANS), (128, oc.TANS), (256, oc.TANS)])
@pytest.mark.parametrize("rows,cols,C,f", [(8, 4096, 16384, 0.0),   # whole rows
                                           (3, 4096, 4096, 0.0),    # an odd number of chunks
                                           (5, 2064, 4096, 0.4)])   # rows over chunks, a short last chunk, raw ones
def test_decoder_does_not_depend_on_the_order_of_the_lanes(decode, order, S, codec, rows, cols, C, f):
    check_every_mode(decode, order, S, codec, rows, cols, C, f)


@pytest.mark.parametrize("order", list(ORDERS))
@pytest.mark.parametrize("S", [32, 64, 128, 256])
@pytest.mark.parametrize("rows,cols,C,f", [(8, 4096, 16384, 0.0), (3, 4096, 4096, 0.0), (5, 2064, 4096, 0.4)])
def test_general_decoder_does_not_depend_on_the_order_of_the_lanes(decode, order, S, rows, cols, C, f):
    # the kernels that launches of more wavefronts take
    check_every_mode(decode, order, S, oc.HUFFMAN, rows, cols, C, f, units=0)


def check_every_mode(decode, order, S, codec, rows, cols, C, f, units=256):
    if S == 32 and f:
        f, rows, cols = 0.0, 4, 2048  # two chunks to a wavefront that differ in length or kind part its lanes: not modelled
    q, scale = oracle_matrix(rows, cols, synth.matrix_seed(9, S), False)
    c = oc.compress(q, C, S, oc.RAW_FRACTION, f, codec=codec)
    x = synth.gen_activation_bf16(cols, 3)
    xq, sx = oq.quantise_vector(oq.bf16_to_f64(x).astype(np.float32))
    run = lambda mode, *more: decode(order, c, C, S, codec, mode, rows, cols, *more, units=units)
    assert np.array_equal(run(BYTES), q.view(np.uint8).ravel())
    assert np.array_equal(run(BF16, scale).view(np.uint16).reshape(rows, cols), oq.dequant_bf16(q, scale))
    y8 = run(PRODUCT_INT8, scale, np.float32(sx), xq).view(np.uint32)
    assert np.array_equal(y8, oq.gemv_w8a8(q, scale, xq, sx).view(np.uint32))
    # fp32 sums of `cols` products against 64 bits: 2^-24 a step at most, of the sum of the magnitudes
    size = np.abs(q.astype(np.float64)) @ np.abs(oq.bf16_to_f64(x)) * scale
    y = run(PRODUCT, scale, x).view(np.float32)
    assert (np.abs(y - oq.gemv_ref(q, scale, x)) <= cols * 2.0 ** -24 * size).all()


@pytest.mark.parametrize("S", [32, 64, 128, 256])
def test_decoder_of_many_wavefronts(decode, S):
    # just beyond the line up to which a launch has few wavefronts
    C, cols = 512, 64
    chunks = {32: 2050, 64: 2049, 128: 1025, 256: 513}[S]
    q, _ = oracle_matrix(chunks * C // cols, cols, synth.matrix_seed(10, S), False)
    c = oc.compress(q, C, S)
    assert c.n_chunks == chunks
    assert np.array_equal(decode("ascending", c, C, S, oc.HUFFMAN, BYTES, *q.shape), q.view(np.uint8).ravel())


def order_of_work(decode, *launch):  # mode, sub-streams, wavefronts, bytes a chunk, SIMDs
    return subprocess.run([decode.exe, "order"] + [str(v) for v in launch]).returncode


MANY, FEW, FEW_AGAIN = 0, 1, 2


@pytest.mark.parametrize("mode,S,chunk,simds,line", [
    (BYTES, 32, 65536, 1024, 2048), (BYTES, 32, 16368, 1024, 1024), (PRODUCT, 32, 16384, 1024, 2048), (BYTES, 256, 4096, 1024, 1024),
    (BYTES, 256, 16384, 1024, 2048), (PRODUCT, 64, 16368, 1024, 1024), (PRODUCT_INT8, 128, 65536, 1024, 2048),
    (BF16, 32, 65536, 1024, 1024), (BF16, 32, 32768, 1024, 1024), (BF16, 64, 16384, 1024, 1024), (BF16, 64, 32768, 1024, 2048),
    (BYTES, 64, 65536, 128, 256), (BF16, 32, 4096, 128, 128), (BYTES, 64, 65536, 0, 0)])
def test_line_for_launches_of_few_wavefronts(decode, mode, S, chunk, simds, line):
    # in wavefronts a SIMD of the device, and by what a lane has to decode
    few = lambda waves: order_of_work(decode, mode, S, waves, chunk, simds) != MANY
    assert not few(line + 1) and few(max(1, line // 3)) == few(max(1, line)) == (line > 0)


@pytest.mark.parametrize("units,few", [(256, "true"), (0, "false")])
def test_a_traced_launch_is_the_launch_it_stands_for(decode, units, few):
    C, S = 4096, 256
    q, _ = oracle_matrix(4, 4096, synth.matrix_seed(11, S), False)
    c = oc.compress(q, C, S)
    for mode, kernel in ((BYTES, f"(dc_decode_kernel<S, MODE, DC_CODEC_HUFFMAN, {few}>)"),
                         (TRACED, f"(dc_decode_kernel<256, kModeI8, DC_CODEC_HUFFMAN, {few}, true>)")):
        assert np.array_equal(decode("shuffled", c, C, S, oc.HUFFMAN, mode, *q.shape, units=units), q.view(np.uint8).ravel())
        assert decode.launched == [kernel.replace(", false>", ">") if mode == BYTES else kernel]


@pytest.mark.parametrize("S", [32, 64, 128, 256])
@pytest.mark.parametrize("rows,cols,C", [(6, 4096, 12288), (3, 8192, 24576),  # whole rows: counted rounds, spans of 1024 bytes
                                         (7, 3072, 10240), (5, 5120, 4096), (9, 1024, 9216),  # spans, where few wavefronts walk lane by lane
                                         (4, 2064, 4096)])                     # lane by lane
def test_products_have_the_same_bits_with_few_wavefronts_and_many(decode, S, rows, cols, C):
    # the kernels and the walks over rows differ, the additions and their order do not
    q, scale = oracle_matrix(rows, cols, synth.matrix_seed(12, S), False)
    c = oc.compress(q, C, S)
    x = synth.gen_activation_bf16(cols, 7)
    few, many = (decode("ascending", c, C, S, oc.HUFFMAN, PRODUCT, rows, cols, scale, x, units=units) for units in (256, 0))
    assert np.array_equal(few, many) and few.size == 4 * rows


@pytest.mark.parametrize("order", list(ORDERS))
@pytest.mark.parametrize("S,codec", [(32, oc.HUFFMAN), (64, oc.HUFFMAN), (128, oc.HUFFMAN), (256, oc.HUFFMAN),
                                     (64, oc.TANS), (128, oc.TANS), (256, oc.TANS)])
@pytest.mark.parametrize("probabilities", [
    [1.0], [0.5, 0.5], [0.95, 0.05], [2.0 ** -min(i + 1, 14) for i in range(15)],  # runs over several waves' slots; lengths 1 to 11
    [1 / 256] * 256, [0.002] * 200 + [0.6 / 56] * 56, [0.7] + [0.3 / 255] * 255])  # all lengths equal; two lengths; many states and one
def test_tables_of_extreme_codes(decode, order, S, codec, probabilities):
    r = np.random.default_rng(len(probabilities))
    values = r.permutation(256)[:len(probabilities)].astype(np.uint8)
    C, n = 8192, 8192 + 4096  # the second chunk is shorter
    q = values[r.choice(len(values), n, p=np.array(probabilities) / sum(probabilities))]
    if S == 32:
        q = np.concatenate([q, q[:4096]])  # two chunks of a wave alike
    c = oc.compress(q, C, S, codec=codec)
    got = decode(order, c, C, S, codec, BYTES, q.size // 64, 64)
    assert np.array_equal(got, q)


@pytest.mark.parametrize("order", list(ORDERS))
@pytest.mark.parametrize("S,rows,cols,C,f", [(64, 4, 4096, 4096, 0.0), (64, 7, 2064, 4096, 0.4),  # a wavefront a SIMD (four): bytes and products
                                             (128, 32, 4096, 32768, 0.0), (128, 61, 2064, 32768, 0.4)])  # two: every mode
def test_few_wavefronts_that_keep_no_second_copy(decode, order, S, rows, cols, C, f):
    check_every_mode(decode, order, S, oc.HUFFMAN, rows, cols, C, f, units=1)
    assert any("true, false, false" in kernel for kernel in decode.launched)


@pytest.mark.parametrize("mode,S,chunk,simds,line,below,beyond", [
    (BYTES, 32, 16384, 1024, 1024, FEW_AGAIN, FEW), (BYTES, 64, 65536, 1024, 1536, FEW_AGAIN, FEW), (BYTES, 64, 32768, 64, 96, FEW_AGAIN, FEW),
    (BYTES, 64, 32752, 1024, 512, FEW_AGAIN, FEW), (BF16, 64, 32768, 1024, 2048, FEW_AGAIN, MANY), (BF16, 64, 4096, 1024, 1024, FEW_AGAIN, MANY),
    (PRODUCT, 64, 65536, 1024, 768, FEW_AGAIN, FEW), (PRODUCT_INT8, 64, 16384, 1024, 768, FEW_AGAIN, FEW),
    (BYTES, 128, 16384, 1024, 1536, FEW_AGAIN, FEW), (BF16, 128, 32768, 1024, 1536, FEW_AGAIN, FEW), (PRODUCT, 128, 16384, 1024, 1536, FEW_AGAIN, FEW),
    (PRODUCT, 32, 16384, 1024, 2048, FEW_AGAIN, MANY), (BF16, 32, 65536, 1024, 1024, FEW, MANY), (BYTES, 256, 16384, 1024, 2048, FEW, MANY)])
def test_line_for_the_second_copy(decode, mode, S, chunk, simds, line, below, beyond):
    order = lambda waves: order_of_work(decode, mode, S, waves, chunk, simds)
    assert (order(1), order(line), order(line + 1)) == (below, below, beyond)


@pytest.mark.parametrize("mode,S,C,chunks,kernel", [
    (BYTES, 64, 4096, 2, "true"), (BYTES, 64, 4096, 3, "true, false, false"), (BYTES, 64, 4096, 5, ""), (BYTES, 64, 32768, 4, "true"),
    (BF16, 64, 4096, 4, "true"), (BF16, 64, 4096, 5, ""), (PRODUCT_INT8, 64, 4096, 3, "true"), (PRODUCT_INT8, 64, 4096, 4, "true, false, false"),
    (BYTES, 128, 16384, 3, "true"), (BYTES, 128, 16384, 4, "true, false, false"), (BYTES, 128, 16384, 5, ""), (BF16, 128, 32768, 4, "true, false, false"),
    (BYTES, 256, 4096, 1, "true"), (BYTES, 256, 4096, 2, "")])
def test_the_kernel_of_an_order(decode, mode, S, C, chunks, kernel):
    # by the kernel's last parameters, on a device of four SIMDs
    cols = C // 2
    q, scale = oracle_matrix(2 * chunks, cols, synth.matrix_seed(13, S), False)
    c = oc.compress(q, C, S)
    x8 = np.ones(cols, np.int8)
    more = {BYTES: (), BF16: (scale,), PRODUCT_INT8: (scale, np.float32(1), x8)}[mode]
    got = decode("ascending", c, C, S, oc.HUFFMAN, mode, *q.shape, *more, units=1)
    want = {BYTES: lambda: q.view(np.uint8).ravel(), BF16: lambda: oq.dequant_bf16(q, scale).view(np.uint8).ravel(),
            PRODUCT_INT8: lambda: oq.gemv_w8a8(q, scale, x8, np.float32(1)).view(np.uint8).ravel()}[mode]()
    assert np.array_equal(got.view(np.uint8), want)
    assert [k for k in decode.launched if "decode_kernel" in k] == [
        f"(dc_decode_kernel<S, MODE, DC_CODEC_HUFFMAN{kernel and ', ' + kernel}>)"]


@pytest.mark.parametrize("order", list(ORDERS))
def test_32_sub_streams_beyond_a_wavefront_a_simd(decode, order):
    # bytes without the ring's second copy, products with it, the conversion by the kernel for many wavefronts
    check_every_mode(decode, order, 32, oc.HUFFMAN, 64, 2560, 16384, 0.0, units=1)


@pytest.mark.parametrize("mode,C,chunks,kernel", [
    (BYTES, 16384, 8, "true"), (BYTES, 16384, 10, "true, false, false"), (BYTES, 16384, 16, "true, false, false"), (BYTES, 16384, 18, ""),
    (BYTES, 16368, 10, ""), (BF16, 4096, 2, "true, false, false"), (BF16, 4096, 8, "true, false, false"), (BF16, 4096, 10, ""), (BF16, 65536, 10, ""),
    (PRODUCT, 16384, 10, "true"), (PRODUCT, 16384, 16, "true"), (PRODUCT, 16384, 18, ""), (PRODUCT_INT8, 16384, 10, "true"), (PRODUCT_INT8, 8192, 10, "")])
def test_lines_at_32_sub_streams(decode, mode, C, chunks, kernel):
    # by the kernel's last parameters, on a device of four SIMDs
    cols = C // 2
    q, scale = oracle_matrix(2 * chunks, cols, synth.matrix_seed(14, 32), False)
    c = oc.compress(q, C, 32)
    x = synth.gen_activation_bf16(cols, 5)
    xq, sx = oq.quantise_vector(oq.bf16_to_f64(x).astype(np.float32))
    more = {BYTES: (), BF16: (scale,), PRODUCT: (scale, x), PRODUCT_INT8: (scale, np.float32(sx), xq)}[mode]
    decode("ascending", c, C, 32, oc.HUFFMAN, mode, *q.shape, *more, units=1)
    assert [k for k in decode.launched if "decode_kernel" in k] == [f"(dc_decode_kernel<S, MODE, DC_CODEC_HUFFMAN{kernel and ', ' + kernel}>)"]
