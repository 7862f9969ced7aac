// Host check of the "groups" field of a launch table's BATCHED entries: read,
// written back, absent, and of a kind that is skipped as any unknown key.
#include "../paper_1105_2279_amd/csrc/qdpx_impl.hpp"

#include <cstdio>

using namespace qdpx;

int main(int argc, char **argv) {
    if (argc < 2) return 2;
    const std::string path = std::string(argv[1]) + "/t.json";
    FILE *f = fopen(path.c_str(), "wb");
    if (!f) return 2;
    const char *e = "{\"op\": \"BATCHED\", \"prec\": \"F64\", \"fmt\": \"LINK18\", \"L\": [8, 8, 8, %d], "
                    "\"launch\": [256, 1, 1, 1, 0]%s}%s";
    fprintf(f, "{\"device\": \"gfx950\", \"entries\": [");
    fprintf(f, e, 8, ", \"groups\": 225168", ",");
    fprintf(f, e, 9, "", ",");
    fprintf(f, e, 10, ", \"groups\": \"many\"", ",");
    fprintf(f, e, 11, ", \"groups\": -3", ",");
    fprintf(f, e, 12, ", \"groups\": 1e300", "]}");
    fclose(f);
    const int want[5] = {225168, 0, 0, 0, 0};
    for (int pass = 0; pass < 2; ++pass) {  // as given, and as written back
        std::vector<TuneEntry> in;
        std::string err;
        if (tune_table_read(path.c_str(), "gfx950", in, err) != 0 || in.size() != 5) return 1;
        for (int i = 0; i < 5; ++i)
            if (in[i].groups != want[i] || in[i].L[3] != 8 + i || in[i].cfg.block != 256) return 1;
        if (tune_table_write(path.c_str(), "gfx950", in, err) != 0) return 1;
    }
    std::printf("ok\n");
    return 0;
}
