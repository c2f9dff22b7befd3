"""The Huffman decode kernels for launches of many wavefronts on the inputs of the edge cases: launches of few wavefronts have
kernels of their own, and a case of a few chunks never leaves those.  Here the chunks of a case come first in a launch that holds a
plain chunk besides, as often as it takes to be beyond every line of the dispatch; in the fused calls it makes up a second matrix."""
import numpy as np
import pytest

import oracle.codec as oc
import oracle.quant as oq
import paper_2502_15443_amd as dc
import synth
from tests.helpers import emptied_buffer_bytes, gemv_workspace, lopsided_bytes, oracle_matrix, weightlike_bytes
from tests.test_gpu_random import draw_case

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

STREAMS = [32, 64, 128, 256]
BF16, PRODUCT, PRODUCT_INT8 = range(3)


def dev(a: np.ndarray):
    return torch.from_numpy(np.ascontiguousarray(a).view(np.uint8).reshape(-1).copy()).cuda()


def stream():
    return torch.cuda.current_stream().cuda_stream


class Crowd:
    """A case's blob and table with so many entries of one further chunk that the launch is none of few wavefronts."""

    def __init__(self, blob, table, C, S):
        self.C, self.S, self.n = C, S, len(table)
        simds = 4 * torch.cuda.get_device_properties(0).multi_processor_count
        self.more = 2 * simds * 64 // S + 2  # chunks of two wavefronts a SIMD, and a workgroup more
        self.extra = weightlike_bytes(C, 3)
        e = oc.compress(self.extra, C, S)
        one = e.table.copy()
        one["off"] += blob.size
        self.blob_bytes = blob.size + e.blob.size
        self.blob, self.table = dev(np.concatenate([blob, e.blob])), dev(np.concatenate([table, np.repeat(one, self.more)]))
        self.chunks, self.params = self.n + self.more, dc.Params(C, S)

    def decode(self):
        """The decoded buffer, up to the case's last chunk; the rest is checked here."""
        size = self.chunks * self.C
        dst = torch.full((size + 4096,), 0x5A, dtype=torch.uint8, device="cuda")
        dc.decompress_chunks(self.blob, self.blob_bytes, self.table, self.chunks, self.params, dst, size, stream())
        torch.cuda.synchronize()
        assert (dst[size:] == 0x5A).all()
        assert (dst[self.n * self.C:size].view(self.more, self.C) == dev(self.extra)).all()
        return dst[:self.n * self.C].cpu().numpy()

    def fused(self, mode, scale, rows, cols, x=None, x_scale=0.0, y_in_workspace=False):
        """The result for a matrix of the case's chunks."""
        cols2 = self.C if self.C <= 16384 else next(c for c in (16384, 8192) if self.C % c == 0)
        assert (rows * cols + self.C - 1) // self.C == self.n
        rows2 = self.more * self.C // cols2
        scale2 = torch.ones(rows2, dtype=torch.float32, device="cuda")
        x_d, x2 = None, None
        if mode != BF16:
            x_d = torch.from_numpy(x.view(np.int16) if mode == PRODUCT else x).cuda()
            x2 = torch.zeros(cols2, dtype=x_d.dtype, device="cuda")
        ws, ws_bytes = gemv_workspace(self.chunks)
        if mode == BF16:
            out = torch.full((rows * cols + 64,), 0x5A5A, dtype=torch.int16, device="cuda")
            out2 = torch.zeros(rows2 * cols2, dtype=torch.int16, device="cuda")
        else:
            out = ws.view(torch.float32)[:rows] if y_in_workspace else torch.full((rows + 64,), 7.0, dtype=torch.float32, device="cuda")
            out2 = torch.full((rows2,), 7.0, dtype=torch.float32, device="cuda")
        mats = []
        for first, r, c, s, o, xx in ((0, rows, cols, torch.from_numpy(scale).cuda(), out, x_d), (self.n, rows2, cols2, scale2, out2, x2)):
            m = dc.Matrix(first, r, c, s)
            if mode == BF16:
                m.dst_bf16_dev, m.dst_cap_elems = o, r * c
            elif mode == PRODUCT:
                m.y_accum_dev, m.x_bf16_dev = o, xx
            else:
                m.y_accum_dev, m.x_i8_dev, m.x_scale = o, xx, float(x_scale)
            mats.append(m)
        call = (self.blob, self.blob_bytes, self.table, self.chunks, self.params, mats)
        if mode == BF16:
            dc.decompress_dequant_bf16_layer(*call, stream())
        elif mode == PRODUCT:
            dc.decompress_gemv_layer(*call, ws, ws_bytes, stream())
        else:
            dc.decompress_gemv_w8a8_layer(*call, stream())
        torch.cuda.synchronize()
        got = out.cpu().numpy()
        if mode == BF16:
            assert (got[rows * cols:] == 0x5A5A).all()
            return got[:rows * cols].view(np.uint16).reshape(rows, cols)
        assert (out2.cpu().numpy() == 0.0).all() and (got[rows:] == 7.0).all()
        return got[:rows]


def check_products(crowd, q, scale, x):
    """Both products of a decoded matrix; the fp32 sums of `cols` products to 2^-24 a step, of the sum of the magnitudes."""
    rows, cols = q.shape
    size = np.abs(q.astype(np.float64)) @ np.abs(oq.bf16_to_f64(x)) * scale
    y = crowd.fused(PRODUCT, scale, rows, cols, x)
    assert (np.abs(y - oq.gemv_ref(q, scale, x)) <= cols * 2.0 ** -24 * size).all()
    xq, sx = oq.quantise_vector(oq.bf16_to_f64(x).astype(np.float32))
    y8 = crowd.fused(PRODUCT_INT8, scale, rows, cols, xq, sx)
    assert np.array_equal(y8.view(np.uint32), oq.gemv_w8a8(q, scale, xq, sx).view(np.uint32))
    return y


@pytest.mark.parametrize("S", STREAMS)
@pytest.mark.parametrize("kind", ["degenerate", "lopsided", "longest codes on one stream", "ragged", "one byte"])
def test_decode_of_edge_cases(S, kind):
    print(f"case general decode S={S} {kind}", flush=True)
    r = np.random.default_rng(0)
    C = 4096
    if kind == "degenerate":
        skew = np.clip(np.rint(r.standard_cauchy(C) * 2), -127, 127).astype(np.int8).view(np.uint8)  # 11-bit codes
        data = np.concatenate([np.zeros(C, np.uint8), np.full(C, 0x81, np.uint8), r.integers(0, 256, C, dtype=np.uint8),
                               np.tile(np.array([3, 250], np.uint8), C // 2), np.arange(C, dtype=np.uint32).astype(np.uint8),
                               skew, np.array([7], np.uint8)])
    elif kind == "lopsided":
        C = 65536
        data = lopsided_bytes(3 * C + 4096 + 50, S, 7 + S)
    elif kind == "longest codes on one stream":
        data = emptied_buffer_bytes(S)
        C = data.size
    elif kind == "ragged":
        data = weightlike_bytes(7 * C + 4095, 9)
    else:
        data = np.array([200], np.uint8)
    for policy, f in ((oc.ALL_HUFF, 0.0), (oc.RAW_FRACTION, 0.3)):
        c = oc.compress(data, C, S, policy, f)
        out = Crowd(c.blob, c.table, C, S).decode()
        assert np.array_equal(out[:data.size], data) and (out[data.size:] == 0x5A).all()


@pytest.mark.parametrize("S", STREAMS)
@pytest.mark.parametrize("rows,cols,C,f", [(1, 16784, 16384, 0.0), (3, 5488, 4096, 0.5), (67, 1040, 65536, 0.0), (40, 2752, 16384, 1.0),
                                           (160, 1024, 16384, 0.0), (50, 5120, 65536, 0.3), (24, 8192, 4096, 0.2), (2048, 64, 16384, 0.3)])
def test_fused_calls_of_edge_cases(S, rows, cols, C, f):
    print(f"case general fused S={S} {rows}x{cols} C={C} f={f}", flush=True)
    q, scale = oracle_matrix(rows, cols, synth.matrix_seed(4, 2), False)
    c = oc.compress(q, C, S, oc.RAW_FRACTION, f)
    crowd = Crowd(c.blob, c.table, C, S)
    assert np.array_equal(crowd.fused(BF16, scale, rows, cols), oq.dequant_bf16(q, scale))
    if cols <= 16384:
        check_products(crowd, q, scale, synth.gen_activation_bf16(cols, 5))


@pytest.mark.parametrize("S", STREAMS)
@pytest.mark.parametrize("rows,cols,C", [(12, 4096, 12288), (6, 8192, 24576), (14, 3072, 12288), (10, 5120, 4096), (9, 1024, 8192),
                                         (50, 2064, 16384), (96, 512, 16384)])
def test_a_matrix_alone_and_in_a_large_layer_have_the_same_bits(S, rows, cols, C):
    """Alone the launch is one of few wavefronts, in the layer call it is not: other kernels and another walk over the rows, the same
    additions in the same order."""
    print(f"case same bits S={S} {rows}x{cols} C={C}", flush=True)
    q, scale = oracle_matrix(rows, cols, synth.matrix_seed(6, 1), False)
    c = oc.compress(q, C, S)
    x = synth.gen_activation_bf16(cols, 9)
    alone = torch.zeros(rows, dtype=torch.float32, device="cuda")
    dc.decompress_gemv(dev(c.blob), c.blob.size, dev(c.table), c.n_chunks, dc.Params(C, S), torch.from_numpy(scale).cuda(), rows, cols,
                       torch.from_numpy(x.view(np.int16)).cuda(), alone, None, *gemv_workspace(c.n_chunks), stream())
    y = check_products(Crowd(c.blob, c.table, C, S), q, scale, x)
    assert np.array_equal(alone.cpu().numpy().view(np.uint32), y.view(np.uint32))


@pytest.mark.parametrize("seed", [21, 22])
def test_decode_of_random_valid_inputs(seed):
    r = np.random.default_rng(seed)
    for it in range(60):
        S, C, n, data, policy, f, block = draw_case(r)
        if C * 64 // S > 131072:
            continue  # the crowd alone would be more than 270 MB
        c = oc.compress(data, C, S, policy, f, block=block)
        out = Crowd(c.blob, c.table, C, S).decode()
        assert np.array_equal(out[:n], data) and (out[n:] == 0x5A).all(), f"case {it} S={S} C={C} n={n} policy={policy}"


@pytest.mark.parametrize("S", STREAMS)
def test_corrupt_payloads_and_table_entries_stay_inside_the_buffers(S):
    """Damaged headers, random payloads and impossible entries: unspecified bytes for those chunks at most, nothing beyond them."""
    print(f"case general corrupt S={S}", flush=True)
    C, rows, cols = 16384, 12 * 16, 1024
    q, scale = oracle_matrix(rows, cols, synth.matrix_seed(5, 1), False)
    data = q.view(np.uint8).ravel()
    c = oc.compress(data, C, S)
    blob, table = c.blob.copy(), c.table.copy()
    r = np.random.default_rng(99 + S)
    off, size = [int(o) for o in table["off"]], [int(x) for x in table["comp_bytes"]]
    blob[off[1]:off[1] + 128] = r.integers(0, 256, 128, dtype=np.uint8)                  # code lengths
    blob[off[2] + 128:off[2] + 128 + 2 * S] = r.integers(0, 256, 2 * S, dtype=np.uint8)  # blocks and head bytes of the streams
    blob[off[3] + 128 + 2 * S:off[3] + 132 + 2 * S] = 0xFF                               # area offset far outside
    blob[off[4]:off[4] + size[4]] = r.integers(0, 256, size[4], dtype=np.uint8)           # everything
    blob[off[5]:off[5] + 128] = 0x11                                                      # 256 codes of one bit
    blob[off[6]:off[6] + 128] = 0                                                         # no code at all
    table["off"][7] += 4                  # misaligned
    table["comp_bytes"][8] = 1 << 30      # beyond the blob
    table["raw_bytes_flags"][9] = C + 16  # longer than a chunk
    table["off"][10] = 1 << 40            # beyond the blob
    good = (0, 11)
    crowd = Crowd(blob, table, C, S)
    out = crowd.decode()
    for k in good:
        assert np.array_equal(out[k * C:(k + 1) * C], data[k * C:(k + 1) * C])
    for k in (7, 8, 9, 10):
        assert (out[k * C:(k + 1) * C] == 0x5A).all()
    wide, want = crowd.fused(BF16, scale, rows, cols).ravel(), oq.dequant_bf16(q, scale).ravel()
    x = synth.gen_activation_bf16(cols, 3)
    xq, sx = oq.quantise_vector(oq.bf16_to_f64(x).astype(np.float32))
    y, y8 = crowd.fused(PRODUCT, scale, rows, cols, x), crowd.fused(PRODUCT_INT8, scale, rows, cols, xq, sx)
    y_ref, y8_ref = oq.gemv_ref(q, scale, x), oq.gemv_w8a8(q, scale, xq, sx)
    size_of = np.abs(q.astype(np.float64)) @ np.abs(oq.bf16_to_f64(x)) * scale
    for k in good:
        assert np.array_equal(wide[k * C:(k + 1) * C], want[k * C:(k + 1) * C])
        of = slice(k * C // cols, (k + 1) * C // cols)
        assert (np.abs(y[of] - y_ref[of]) <= cols * 2.0 ** -24 * size_of[of]).all()
        assert np.array_equal(y8[of].view(np.uint32), y8_ref[of].view(np.uint32))


def test_damaged_blobs_that_still_validate_decode_as_the_oracle_decodes_them():
    r = np.random.default_rng(70)
    accepted = changed = 0
    for it in range(400):
        S, C = int(r.choice([64, 128, 256])), int(r.choice([512, 4096, 16384]))
        n = max(1, int(r.integers(1, 6)) * C - int(r.integers(0, C)))
        data = weightlike_bytes(n, int(r.integers(1 << 30)))
        p = dc.Params(C, S, dc.POLICY_RAW_FRACTION, float(r.choice([0, 0.3])))
        blob, table = dc.compress_chunks(data, p)
        for _ in range(int(r.integers(1, 4))):
            blob[r.integers(blob.size - 64)] ^= 1 << int(r.integers(8))
        try:
            dc.validate(blob, table, p)
        except dc.DCError:
            continue
        accepted += 1
        want = oc.decompress(blob, table, C, S, n)
        changed += not np.array_equal(want, data)
        assert np.array_equal(Crowd(blob, table, C, S).decode()[:n], want), f"case {it} S={S} C={C} n={n}"
    assert accepted >= 15 and changed >= 5


@pytest.mark.parametrize("S", STREAMS)
@pytest.mark.parametrize("rows,cols,C", [(50, 5120, 65536), (16, 13824, 4096), (96, 512, 16384)])
def test_gemv_of_a_chunk_that_is_not_decoded(S, rows, cols, C):
    """It adds nothing; in particular nothing that the workspace held before the call (here NaN)."""
    print(f"case general undecoded S={S} {rows}x{cols} C={C}", flush=True)
    seed = synth.matrix_seed(5, 2)
    q, scale = oracle_matrix(rows, cols, seed, False)
    c = oc.compress(q, C, S)
    x = synth.gen_activation_bf16(cols, seed)
    for j in {0, c.n_chunks // 2, c.n_chunks - 1}:
        size = int(c.table["raw_bytes_flags"][j])
        for decoded in (0, size // 32 * 16):
            table, left = c.table.copy(), q.reshape(-1).copy()
            if decoded:
                table["raw_bytes_flags"][j] = decoded
            else:
                table["comp_bytes"][j] = 1 << 30
            left[j * C + decoded:j * C + size] = 0
            check_products(Crowd(c.blob, table, C, S), left.reshape(rows, cols), scale, x)


@pytest.mark.parametrize("S", [32, 256])
def test_gemv_results_over_the_workspace(S):
    rows, cols, C = 12, 1024, 16384
    print(f"case general over workspace S={S}", flush=True)
    q, scale = oracle_matrix(rows, cols, synth.matrix_seed(5, 3), False)
    c = oc.compress(q, C, S)
    x = synth.gen_activation_bf16(cols, 5)
    crowd = Crowd(c.blob, c.table, C, S)
    got = [crowd.fused(PRODUCT, scale, rows, cols, x, y_in_workspace=over) for over in (False, True)]
    assert np.array_equal(got[0].view(np.uint32), got[1].view(np.uint32))
