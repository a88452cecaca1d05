// CPU check of the arithmetic in csrc/encode_plan.hpp: the numerators that the deciding threads ask for are those of their
// own tokens and heads, and whatever lies behind the last token is beyond the range that the load compares with.
#include <stdio.h>
#include <initializer_list>

#include "../../paper_2411_10803_amd/csrc/encode_plan.hpp"

using namespace md;

int main() {
    long looked = 0, bad = 0;
    for (int M : {1, 5, 575, 1023, 1024, 1025, 2048, 2049, 3071, 3072, 4095, 4096, 4097, 4608, 5119, 5120})
        for (int Hc = 4; Hc <= 16; Hc += 4) {
            bool ok = true;
            for (int t = 0; t < (M + 1023) / 1024; ++t)
                for (int tid = 0; tid < 1024; ++tid)
                    for (int q = 0; q < 4; ++q) {
                        const int token = tid + 1024 * t, byte = numerator_vector(tid, t, q, M, Hc);
                        ++looked;
                        if (token < M && 4 * q < Hc) ok &= byte == (token * Hc + 4 * q) * 4 && byte + 16 <= numerator_bytes(M, Hc);
                        else ok &= byte >= numerator_bytes(M, Hc);
                    }
            if (!ok && ++bad <= 10) printf("M=%d Hc=%d\n", M, Hc);
        }
    printf("%ld requests, %ld shapes wrong\n", looked, bad);
    return bad != 0;
}
