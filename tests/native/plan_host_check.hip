// Host build of the rules by which the line and the stride-2 kernel and their neighbours share the 3x3 layers
// (csrc/bwd_line_choice.h, csrc/bwd_stride2_shapes.h).  Test infrastructure, not product code; built without optimisation, so that what the rules compute
// for shapes that do not fit is computed.
//   columns B H Wd C_in C_out n m ranker   columns of the line kernel's tile for n <= 2
//   alone H Wd                               1 if the whole gradient leaves the line kernel one workgroup on a CU
//   row MODE m BLOCKS ROWS COLUMNS LINE      who takes a layer there, the row kernel's plan and the line kernel's workgroups given
//   plan MODE m B H Wd C_in                  whether the row kernel is planned for such a layer: "search" or "line"
//   stride2 B H Wd C_in C_out LDS    the shape chosen within LDS bytes: "bn rows lds blocks", or "none"
//   classes AHEAD B H Wd C_in C_out  who takes a layer that the parity-class kernel could take: "classes" or "stride2"
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>

#include "bwd_line_choice.h"
#include "bwd_stride2_shapes.h"

using namespace sdgp;

int main(int argc, char** argv) {
    int64_t v[16] = {};
    for (int i = 2; i < argc && i < 16; ++i) v[i - 2] = atoll(argv[i]);
    if (argc == 10 && !strcmp(argv[1], "columns")) {
        const int64_t row_tiles = (v[0] * v[1] * v[2] + kLineRows - 1) / kLineRows;
        printf("%d\n", tile_columns(row_tiles, (int)v[1], (int)v[2], v[3], v[4], (int)v[5], (int)v[6], (int)v[7]));
        return 0;
    }
    if (argc == 4 && !strcmp(argv[1], "alone")) return printf("%d\n", line_alone((int)v[0], (int)v[1])), 0;
    if (argc == 8 && !strcmp(argv[1], "row"))
        return puts(row_faster_than_lone_line((int)v[0], (int)v[1], v[2], (int)v[3], (int)v[4], v[5]) ? "row" : "line"), 0;
    if (argc == 8 && !strcmp(argv[1], "plan")) {
        const int64_t pixels = v[2] * v[3] * v[4], line = (pixels + 255) / 256 * ((v[5] + 63) / 64);
        return puts(row_worth_planning((int)v[0], (int)v[1], pixels, v[3], v[4], v[5], line) ? "search" : "line"), 0;
    }
    if (argc == 8 && !strcmp(argv[1], "stride2")) {
        const int64_t P = (v[1] + 1) / 2, Q = (v[2] + 1) / 2;
        Stride2Shape s;
        if (stride2_choose(v[0] * P * Q, (int)P, (int)Q, v[3], 2 * (int)((v[4] + 31) / 32), (int)v[5], s) < 0) return puts("none"), 0;
        printf("%d %d %d %lld\n", s.bn, s.rows, s.lds, (long long)s.blocks);
        return 0;
    }
    if (argc == 8 && !strcmp(argv[1], "classes")) {
        const int64_t P = (v[2] + 1) / 2, Q = (v[3] + 1) / 2;
        Stride2Shape s;
        const bool fits = stride2_choose(v[1] * P * Q, (int)P, (int)Q, v[4], 2 * (int)((v[5] + 31) / 32), 80 * 1024, s) >= 0;
        puts(!fits || stride2_classes_faster(v[0] != 0, v[2], v[3], v[4], v[5], s.blocks) ? "classes" : "stride2");
        return 0;
    }
    return 2;
}
