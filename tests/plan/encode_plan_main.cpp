// CPU check of the arithmetic in csrc/encode_plan.hpp: the numerators that the deciding threads ask for are those of their
// own tokens and heads, and whatever lies behind the last token is beyond the range that the load compares with; and every
// output is noticed that shares a byte with the masses or the flags, wherever it begins.
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
    const size_t B = 3, M = 100, W = 30, row = 64, keys = 7;
    char* const base = reinterpret_cast<char*>(0x10000000);                     // never read
    const size_t size[] = {B * M * row, 4 * B * M, 4 * B * M, B * M, B * M, 4 * B, 4 * B * keys, 4 * B, 4 * B * M, 4 * B * W};
    char *const mass = base, *const flags = base + 4 * B * M + 4096;
    for (int i = 0; i < 10; ++i)
        for (int in = 0; in < 2; ++in) {
            char* const p = in ? flags : mass;
            const long n = in ? B * M : 4 * B * M, len = (long)size[i];
            for (long at : {-len, -len + 1, -len + 4, -1l, 0l, 1l, n / 2, n - 1, n, n + 4}) {
                const void* out[10];
                for (int k = 0; k < 10; ++k) out[k] = k == 5 ? nullptr : base + ((long)(k + 1) << 20);
                out[i] = p + at;
                const EncodeOutputs o{out[0], out[1], out[2], out[3], out[4], out[5], out[6], out[7], out[8], out[9]};
                // the other input is out of the way: it is not given
                const bool got = outputs_over(o, B, M, W, row, keys, in ? nullptr : mass, in ? flags : nullptr), want = at > -len && at < n;
                if (got != want && ++bad <= 10) printf("output %d at %ld of input %d\n", i, at, in);
            }
        }
    printf("%ld requests, %ld wrong\n", looked, bad);
    return bad != 0;
}
