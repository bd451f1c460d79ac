// Host-side checks of the rules that choose a hopping launch (compiled for the host only):
//  * the eight-threads-per-point kernel takes small FP64 / FP32 launches of the default
//    configuration, and CG's scalar steps fold into them;
//  * a configuration that asks for another block, an occupancy cap or non-temporal hints gets
//    the two-threads-per-point kernel with that block;
//  * FP64 refreshes are hinted from 200 MB on between 16-bit iterations, else like any launch.
// Prints "ok" and exits 0, or prints the first failure and exits 1.
#include <cstdio>

#include "wl_dslash.h"

using namespace wl;

#define CHECK(c)                                                \
    if (!(c)) {                                                 \
        printf("line %d: %s (prec %d)\n", __LINE__, #c, prec);  \
        return 1;                                               \
    }

int main() {
    for (int prec : {(int)WL_F64, (int)WL_F32}) {
        LaunchCfg def;
        def.block = hop_default_block(prec);
        def.tps = 2;
        const long most = prec == WL_F64 ? 8192 : 16384;
        for (long n : {16L, 2048L, most / 2, most}) {
            // both parities of n / 2 points, or one of n
            CHECK(hop_launch_blocks(2, def, n, 1, 8, n / 8, prec, 1) == (n * 8 + 255) / 256);
            CHECK(hop_launch_blocks(2, def, n / 2, 1, 8, n / 16, prec, 2) == (n / 2 * 8 + 255) / 256);
            CHECK(cg_fold_ok(prec, 2, def, n, 1, 1));
            LaunchCfg off = def;
            off.nt = 0;  // no hints: as the kernel has it
            CHECK(hop_launch_blocks(2, off, n, 1, 8, n / 8, prec, 1) == (n * 8 + 255) / 256);
            for (int block : {64, 128, 192, 256})
                for (int nt : {-1, 0, 1})
                    for (int occ : {0, 2}) {
                        LaunchCfg c = def;
                        c.block = block;
                        c.nt = nt;
                        c.occ = occ;
                        if (block == def.block && nt != 1 && occ == 0) continue;
                        CHECK(hop_launch_blocks(2, c, n, 1, 8, n / 8, prec, 1) == (n * 2 + block - 1) / block);
                        CHECK(!cg_fold_ok(prec, 2, c, n, 1, 1));
                    }
            CHECK(hop_launch_blocks(1, def, n, 1, 8, n / 8, prec, 1) == (n + def.block - 1) / def.block);
        }
        CHECK(hop_launch_blocks(2, def, most + 1, 1, 8, most / 8, prec, 1) == (2 * (most + 1) + def.block - 1) / def.block);
        CHECK(!cg_fold_ok(prec, 2, def, most + 1, 1, 1));
        CHECK(nt_refresh_limit(prec) == NT_WORKING_SET);
    }
    for (int prec : {(int)WL_F16N, (int)WL_BF16N, (int)WL_I16N}) {
        LaunchCfg c;
        c.tps = 2;
        CHECK(hop_launch_blocks(2, c, 1024, 1, 8, 128, prec, 1) == 8);
        CHECK(nt_refresh_limit(prec) == 200e6);
    }
    printf("ok\n");
    return 0;
}
