// Host-only driver for the clearance grid: packs a mesh read from a binary file
// (as tests/pack_driver.cpp reads it) and prints the grid's size, its cells per
// unit length and, one line per x and y, its bytes.
#include <cstdint>
#include <cstdio>
#include <string>
#include <vector>

#include "pack.h"

int main(int argc, char** argv) {
    if (argc != 2) return 2;
    FILE* f = fopen(argv[1], "rb");
    int64_t hdr[2];
    if (!f || fread(hdr, sizeof hdr, 1, f) != 1) return 2;
    std::vector<float> P(size_t(3 * hdr[0]));
    std::vector<int32_t> tets(size_t(4 * hdr[1])), nbrs(size_t(4 * hdr[1]));
    std::vector<uint8_t> cflag(size_t(4 * hdr[1]));
    if (fread(P.data(), 4, P.size(), f) != P.size() || fread(tets.data(), 4, tets.size(), f) != tets.size() ||
        fread(nbrs.data(), 4, nbrs.size(), f) != nbrs.size() || fread(cflag.data(), 1, cflag.size(), f) != cflag.size())
        return 2;
    fclose(f);
    tetrt::PackedMesh m;
    std::string err;
    const int rc = tetrt::pack_mesh(P.data(), hdr[0], tets.data(), nbrs.data(), cflag.data(), hdr[1],
                                    tm_upload_opts{1, 0, 1, 0, 0}, &m, &err);
    if (rc) { printf("rc %d %s\n", rc, err.c_str()); return 1; }
    printf("%zu %d %d %d %.9g %.9g %.9g\n", m.clear.size(), m.R[0], m.R[1], m.R[2], m.clear_inv[0], m.clear_inv[1],
           m.clear_inv[2]);
    for (size_t i = 0; i < m.clear.size(); ++i) printf("%d%c", m.clear[i], i + 1 == m.clear.size() ? '\n' : ' ');
    return 0;
}
