// Where the factor tiles' epilogue asks for the old values of a running average (factor_tile.h), counted on the CPU: a lane's offset and the
// step to a pass are either the vector that the lane then writes, wholly inside the matrix, or an offset outside every result and no step.
// Only then does it not matter whether the buffer's bounds check leaves the step out or takes it from the buffer's size.
#include <cstdio>

#include "../paper_1811_12019_amd/csrc/factor_tile.h"

using namespace kfac;

static long faults = 0, inside = 0;

template <int TW, int ES>
static void check(int D, int d) {
    typedef TileShape<TW, ES> S;
    constexpr int W = S::NB * 32, VPR = W / 4, NV = 32 * W / 256;
    const unsigned ud = 4u * d;
    const unsigned long long bytes = 4ull * d * d;
    const int tiles = ceil_div(D, TW);
    for (int I = 0; I < tiles; ++I)
        for (int J = 0; J <= I; ++J)
            for (int wave = 0; wave < S::WM * S::WN; ++wave) {
                const int wr = wave / S::WN * S::MB * 32, wc = wave % S::WN * W;
                if (I * TW + wr >= D || J * TW + wc >= D) continue;
                for (int p = 0; p < S::MB; ++p) {
                    const bool whole = block_whole(I == J, I * TW, wr + p * 32, J * TW, wc, W, D);
                    for (int lane = 0; lane < 64; ++lane)
                        for (int k = 0; k < NV; ++k) {
                            const unsigned row = I * TW + wr + lane / VPR, col = J * TW + wc + lane % VPR * 4;
                            const OldAt at = old_at(whole, row * ud + 4u * col, ud);
                            const unsigned long long step = (unsigned long long)pass_row(W, p, k) * at.row;
                            if (at.offset == OUTSIDE) {
                                faults += whole || step != 0 || OUTSIDE < bytes;
                                continue;
                            }
                            ++inside;
                            const unsigned r = row + pass_row(W, p, k);
                            faults += r >= (unsigned)D || col + 4 > (unsigned)D || at.offset + step != 4ull * ((unsigned long long)r * d + col) ||
                                      at.offset + step + 16 > bytes;
                        }
                }
            }
}

int main() {
    for (int D = 1; D <= 700; D = D < 300 ? D + 1 : D + 97)
        for (int bias = 0; bias < 2; ++bias) {
            if (D <= 64) { check<64, 2>(D, D + bias); check<64, 4>(D, D + bias); }
            else { check<128, 2>(D, D + bias); check<128, 4>(D, D + bias); }
            if (D > 128) check<256, 2>(D, D + bias);
        }
    check<128, 2>(32766, 32767);
    check<256, 2>(32766, 32767);
    printf("%ld faults\n", faults + (inside == 0));
    return faults != 0;
}
