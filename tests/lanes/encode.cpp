// The device compressor on the CPU, lane by lane (hip/hip_runtime.h beside this file):
//   encode ORDER SEED chunk_bytes n_streams policy raw_fraction block_chunks codec SOURCE RESULT [OVER]
// SOURCE holds the bytes to compress; RESULT gets the two result words, the number of chunks (u64), the table and the blob.
// OVER: "result" or "blob" lies over the chunks' sizes, the last part of the workspace of a Huffman call.
#include "dc_encode.hip"

#include <string>

int dc_launch_status() { return DC_OK; }

int main(int argc, char **argv)
{
    if (argc != 11 && argc != 12) return 2;
    const std::string over = argc == 12 ? argv[11] : "";
    lanes::config.order = (lanes::Order)atoi(argv[1]);
    lanes::config.seed = strtoull(argv[2], nullptr, 10);
    dc_params p = {};
    p.chunk_bytes = (uint32_t)atoi(argv[3]);
    p.n_streams = (uint32_t)atoi(argv[4]);
    p.policy = (uint32_t)atoi(argv[5]);
    p.raw_fraction = (float)atof(argv[6]);
    p.block_chunks = (uint32_t)atoi(argv[7]);
    p.codec = (uint32_t)atoi(argv[8]);
    p.format = DC_FORMAT_ID;
    std::vector<uint8_t> source;
    if (FILE *f = fopen(argv[9], "rb")) {
        int c;
        while ((c = getc(f)) != EOF) source.push_back((uint8_t)c);
        fclose(f);
    }
    const uint64_t n = source.size(), nc = (n + p.chunk_bytes - 1) / p.chunk_bytes;
    uint64_t ws_bytes = 0;
    if (dc_compress_chunks_dev_workspace(n, &p, &ws_bytes)) return 4;
    const uint64_t cap = 2 * n + nc * 4096 + DC_BLOB_TAIL_BYTES;
    std::mt19937_64 rng(lanes::config.seed ^ 0x5A5A);
    auto buffer = [&](uint64_t bytes) { // what it holds before the call must not matter
        uint8_t *b = static_cast<uint8_t *>(aligned_alloc(256, (bytes + 511) / 256 * 256));
        for (uint64_t i = 0; i < bytes; i++) b[i] = (uint8_t)rng();
        return b;
    };
    const uint64_t sizes = (nc * 4 + 255) / 256 * 256;
    uint8_t *src = buffer(n), *ws = buffer(ws_bytes + cap), *blob = over == "blob" ? ws + ws_bytes - sizes : buffer(cap);
    memcpy(src, source.data(), n);
    dc_chunk *table = reinterpret_cast<dc_chunk *>(buffer(nc * sizeof(dc_chunk)));
    uint64_t words[2] = {1, 1};
    uint64_t *result = over == "result" ? reinterpret_cast<uint64_t *>(ws + ws_bytes - sizes) : words;
    if (dc_compress_chunks_dev(reinterpret_cast<int8_t *>(src), n, &p, blob, cap, table, nc, ws, ws_bytes, result, nullptr)) return 5;
    FILE *f = fopen(argv[10], "wb");
    if (!f) return 6;
    fwrite(result, 8, 2, f);
    fwrite(&nc, 8, 1, f);
    fwrite(table, sizeof(dc_chunk), nc, f);
    fwrite(blob, 1, result[0] <= cap ? result[0] : 0, f);
    return fclose(f);
}
