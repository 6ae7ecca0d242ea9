// The addresses of the loads that write LDS (DmaOperand, tiles.hpp), host code
// only: every lane's address, range and place in LDS against 64-bit addresses,
// in both forms (narrow; wide for operands of 2 GiB and more).  No memory is
// read.  Prints one line per operand; exit code 1 at a mismatch.
#include <cstdio>
#include <vector>

#include "tiles.hpp"

using namespace selinv;

static int bad = 0, forms[2] = {0, 0};

// The operand at address P0 (row r, k at r ld + k for KC, else r + k ld), its
// tile at row r0; the chunks first, at and after the middle, and the last two.
template <typename T, int R, bool KC>
void check(const char *name, int64_t ld, int r0, int rows, int K) {
    typedef DmaOperand<T, R, KC> Op;
    constexpr int E = sizeof(T), BK = Op::BK;
    const int64_t P0 = int64_t(1) << 40;  // the operand's address, nominal
    const int64_t end = P0 + ((KC ? (int64_t)(rows - 1) * ld + K : (int64_t)(K - 1) * ld + rows) * E);
    const int nch = (K + BK - 1) / BK;
    const int before = bad;
    bool wide = false;
    std::vector<int> chunks = {0, 1, nch / 2, nch / 2 + 1, nch - 2, nch - 1};
    for (int c : chunks) {
        if (c < 0 || c >= nch) continue;
        // source address of every 16-byte unit of the stage (0: read as zero), and
        // how many of its bytes are in range
        std::vector<int64_t> src(R * 128 / 16, -1);
        std::vector<int> len(R * 128 / 16, 0);
        for (int wave = 0; wave < 4; wave++)
            for (int lane = 0; lane < 64; lane++) {
                Op o;
                o.init((const void *)P0, ld, r0, rows, K, lane, wave);
                wide = o.wide;
                for (int i = 0; i < Op::NI; i++) {
                    int64_t off = 0, so = 0;
                    uint32_t num;
                    if (!o.wide) {
                        so = o.chunk_at(c);
                        num = (uint32_t)o.size;
                        // 32-bit arithmetic of the load itself
                        if (so < 0 || so > (int64_t)num || (int64_t)o.voff[i] + so > 0xffffffffll) bad++;
                    } else {
                        off = o.load_at(c, wave * Op::NI + i);
                        num = Op::range_of(o.size - off);
                    }
                    const int unit = (wave * Op::NI + i) * 64 + lane;
                    if (src[unit] != -1) bad++;
                    const int64_t left = (int64_t)num - so - o.voff[i];  // bytes of the unit in range
                    len[unit] = left >= 16 ? 16 : left > 0 ? (int)(left / 4 * 4) : 0;
                    src[unit] = (int64_t)o.base + off + so + o.voff[i];
                    // what is read lies in the operand (or its last unit's slack)
                    if (len[unit] > 0 && (src[unit] < P0 || src[unit] + len[unit] > end + 16 - E)) bad++;
                }
            }
        for (int r = 0; r < R; r++)
            for (int k = 0; k < BK; k++) {
                if (r0 + r >= rows || c * BK + k >= K) continue;
                const int at = Op::at(r, k), unit = at / 16;
                const int64_t row = r0 + r, kk = (int64_t)c * BK + k;
                const int64_t want = P0 + (KC ? row * ld + kk : row + kk * ld) * E;
                if (src[unit] + at % 16 != want || at % 16 + E > len[unit]) {
                    if (bad++ - before < 3)
                        std::printf("  %s r %d k %d chunk %d: %lld for %lld, %d bytes in range\n", name, r, k, c,
                                    (long long)(src[unit] + at % 16 - P0), (long long)(want - P0), len[unit]);
                }
            }
    }
    forms[wide]++;
    std::printf("%s ld %lld r0 %d rows %d K %d %s: %s\n", name, (long long)ld, r0, rows, K, wide ? "wide" : "narrow",
                bad == before ? "ok" : "BAD");
}

template <typename T, int R>
void both(const char *name) {
    constexpr int64_t E = sizeof(T), two = int64_t(1) << 31;
    // ordinary and ragged operands
    for (int rows : {1, 63, 64, 65, 200})
        for (int K : {1, 3, 15, 33, 64, 257})
            for (int r0 = 0; r0 < rows; r0 += R) {
                check<T, R, true>(name, K + 5, r0, rows, K);
                check<T, R, false>(name, rows + 3, r0, rows, K);
            }
    // square operands (a G_K) around 2 GiB, first, middle and last tile
    int c = 1;
    while ((int64_t)c * c * E < two) c++;
    for (int n : {c - 40, c + 1, 2 * c + 7})
        for (int r0 : {0, n / 2 / R * R, (n - 1) / R * R}) {
            check<T, R, true>(name, n, r0, n, n);
            check<T, R, false>(name, n, r0, n, n);
        }
    // leading dimensions up to the bound of these tiles
    for (int64_t ld : {int64_t(1) << 22, (int64_t(1) << 26) - 1, int64_t(1) << 26}) {
        check<T, R, true>(name, ld, 0, 70, 100);
        check<T, R, true>(name, ld, 64 / R * R, 64 / R * R + 1, 100);
        check<T, R, false>(name, ld, 1000, 1010, 100);
    }
}

int main() {
    both<double, 64>("FP64 64");
    both<float, 64>("FP32 64");
    both<float, 128>("FP32 128");
    both<Pk32, 64>("split-BF16 64");
    both<Pk32, 128>("split-BF16 128");
    std::printf("mismatches %d, narrow %d, wide %d\n", bad, forms[0], forms[1]);
    return bad ? 1 : 0;
}
