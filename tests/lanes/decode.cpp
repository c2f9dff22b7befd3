// The device decoder on the CPU, lane by lane (hip/hip_runtime.h beside this file):
//   decode ORDER SEED chunk_bytes n_streams codec MODE rows cols SOURCE RESULT [COMPUTE_UNITS]
//   decode order MODE n_streams waves chunk_bytes simds
// MODE: 0 the bytes, 1 bf16 values, 2 product, 3 product with int8 activations, 4 the bytes, traced.  SOURCE: the numbers of chunks and of blob
// bytes (u64), the table, the blob, row scales (fp32), activations (bf16, or int8 with their scale in fp32 before them).
// RESULT: what the call writes; standard output: the kernels launched.  COMPUTE_UNITS: of the device (256); 0: no launch is one of few wavefronts.
// order: by which kernel such a launch is decoded (exit status 0: for many wavefronts, 1: for few, 2: for few, with the ring's second copy).
#include "dc_decode.hip"

int main(int argc, char **argv)
{
    if (argc == 7 && !strcmp(argv[1], "order"))
        return order_of_work(atoi(argv[2]), (uint32_t)atoi(argv[3]), strtoull(argv[4], nullptr, 10), (uint32_t)atoi(argv[5]), (uint32_t)atoi(argv[6]));
    if (argc != 11 && argc != 12) return 2;
    if (argc == 12) lanes::config.compute_units = atoi(argv[11]);
    lanes::config.order = (lanes::Order)atoi(argv[1]);
    lanes::config.seed = strtoull(argv[2], nullptr, 10);
    dc_params p = {};
    p.chunk_bytes = (uint32_t)atoi(argv[3]);
    p.n_streams = (uint32_t)atoi(argv[4]);
    p.codec = (uint32_t)atoi(argv[5]);
    p.format = DC_FORMAT_ID;
    const int mode = atoi(argv[6]);
    const uint32_t rows = (uint32_t)atoi(argv[7]), cols = (uint32_t)atoi(argv[8]);
    std::mt19937_64 rng(lanes::config.seed ^ 0xA5A5);
    auto buffer = [&](uint64_t bytes) { // what it holds before the call must not matter
        uint8_t *b = static_cast<uint8_t *>(aligned_alloc(256, (bytes + 511) / 256 * 256));
        for (uint64_t i = 0; i < bytes; i++) b[i] = (uint8_t)rng();
        return b;
    };
    FILE *f = fopen(argv[9], "rb");
    if (!f) return 4;
    auto part = [&](uint64_t bytes) {
        uint8_t *b = buffer(bytes);
        if (fread(b, 1, bytes, f) != bytes) lanes::fail("the source is too short");
        return b;
    };
    uint64_t nc, blob_bytes;
    memcpy(&nc, part(8), 8);
    memcpy(&blob_bytes, part(8), 8);
    const dc_chunk *table = reinterpret_cast<dc_chunk *>(part(nc * sizeof(dc_chunk)));
    const uint8_t *blob = part(blob_bytes);
    const uint64_t n = (uint64_t)rows * cols;
    int rc;
    uint64_t out_bytes = mode == 0 || mode == 4 ? n : mode == 1 ? 2 * n : 4ull * rows;
    uint8_t *out = buffer(out_bytes);
    if (mode == 0) {
        rc = dc_decompress_chunks(blob, blob_bytes, table, nc, &p, reinterpret_cast<int8_t *>(out), n, nullptr);
    } else if (mode == 4) {
        rc = dc_decompress_chunks_traced(blob, blob_bytes, table, nc, &p, reinterpret_cast<int8_t *>(out), n,
                                         reinterpret_cast<uint64_t *>(buffer(32 * nc)), nullptr);
    } else {
        const float *scale = reinterpret_cast<float *>(part(4ull * rows));
        if (mode == 1) {
            rc = dc_decompress_dequant_bf16(blob, blob_bytes, table, nc, &p, scale, rows, cols, reinterpret_cast<uint16_t *>(out), n, nullptr);
        } else if (mode == 2) {
            const uint16_t *x = reinterpret_cast<uint16_t *>(part(2ull * cols));
            uint64_t ws_bytes = 0;
            dc_decompress_gemv_workspace(nc, &ws_bytes);
            rc = dc_decompress_gemv(blob, blob_bytes, table, nc, &p, scale, rows, cols, x, reinterpret_cast<float *>(out), nullptr,
                                    buffer(ws_bytes), ws_bytes, nullptr);
        } else {
            float x_scale;
            memcpy(&x_scale, part(4), 4);
            const int8_t *x = reinterpret_cast<int8_t *>(part(cols));
            rc = dc_decompress_gemv_w8a8(blob, blob_bytes, table, nc, &p, scale, rows, cols, x, x_scale, reinterpret_cast<float *>(out),
                                         nullptr, nullptr);
        }
    }
    fclose(f);
    if (rc) return 5;
    for (const char *kernel : lanes::launched) puts(kernel);
    f = fopen(argv[10], "wb");
    if (!f) return 6;
    fwrite(out, 1, out_bytes, f);
    return fclose(f);
}
