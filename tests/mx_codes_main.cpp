// The direct-to-LDS MXFP4 kernel's loads of packed codes, walked on the host: every lane of every wave over all K tiles, in the kernel's order (K tiles 0 to 2 of
// both operands and 3 of A ahead; then, in K tile kt, B's kt + 3 and A's kt + 4, past the end the fillers).  A load stays inside its own operand's bytes of
// a matrix that ends with its last row (a slab: with its 256th), and the loads of a K tile are its bytes, each once.  Prints "mx-codes ok".
#include <stdio.h>

#include <vector>

#include "../paper_2505_19115_amd/csrc/mx_codes.h"

using namespace nvfp4;

struct Operand {
    std::vector<uint8_t> bytes;  // (never read: addresses only)
    std::vector<int> seen;       // loads of each 16 bytes
    int64_t K;
    bool ok = true;
};

// The loads of one K tile (or fillers, `real` false) of all lanes, whose pointers stand the same
template <bool SLAB>
void fetch(Operand &O, const std::vector<MxCodes<SLAB>> &lanes, bool real)
{
    for (const MxCodes<SLAB> &L : lanes)
        for (int u = 0; u < 4; ++u) {
            const int64_t at = (L.p - O.bytes.data()) + L.off[SLAB ? 0 : u] + L.more(u);
            if (at < 0 || at % 16 != 0 || at + 16 > (int64_t)O.bytes.size()) {
                fprintf(stderr, "%s, K %ld, %s: bytes %ld to %ld of %ld\n", SLAB ? "slab" : "rows", (long)O.K, real ? "K tile" : "filler", (long)at, (long)at + 16, (long)O.bytes.size());
                O.ok = false;
                return;
            }
            if (real) ++O.seen[at / 16];
        }
}

// `rows` rows in the last tile of 256, `before` rows before it; `ahead` K tiles requested before the loop, at K tile kt the one of kt + ahead
template <bool SLAB>
bool walk(int64_t rows, int64_t before, int64_t K, int ahead)
{
    const int nkt = (int)(K / 128);
    const int64_t Kb = K / 2;
    Operand O;
    O.K = K;
    O.bytes.resize(SLAB ? (before + 256) * Kb : (before + rows) * Kb);
    O.seen.assign(O.bytes.size() / 16, 0);
    const uint8_t *first = O.bytes.data() + before * Kb;  // (256 rows of slabs are as many bytes as 256 rows)
    std::vector<MxCodes<SLAB>> lanes;
    for (int wave = 0; wave < 4; ++wave)
        for (int lane = 0; lane < 64; ++lane) {
            MxCodes<SLAB> L;
            L.lane_offsets(wave, lane, lane & 3, rows, Kb);  // (any choice that takes each chunk of four lanes once)
            L.start(first);
            lanes.push_back(L);
        }
    for (int kt = -ahead; kt < nkt; ++kt) {
        const bool real = kt + ahead < nkt;
        if (!real)
            for (auto &L : lanes) L.past_end();
        fetch(O, lanes, real);
        for (auto &L : lanes) L.advance();
    }
    for (int64_t i = 0; i < (int64_t)O.seen.size(); ++i) {
        const int64_t row = i * 16 / Kb - before;
        // (row-major: the last row once more for every row past the edge)
        const int want = i * 16 < before * Kb ? 0 : SLAB || row < rows - 1 ? 1 : (int)(256 - rows + 1);
        if (O.ok && O.seen[i] != want) {
            fprintf(stderr, "%s, %ld rows, K %ld: 16 bytes at %ld fetched %d times, not %d\n", SLAB ? "slab" : "rows", (long)rows, (long)K, (long)i * 16, O.seen[i], want);
            O.ok = false;
        }
    }
    return O.ok;
}

int main()
{
    bool ok = true;
    for (int64_t K = 512; K <= 1280; K += 128)
        for (int64_t rows : {1, 2, 17, 255, 256})
            for (int64_t before : {0, 256})
                for (int ahead : {3, 4}) ok = walk<false>(rows, before, K, ahead) && walk<true>(rows, before, K, ahead) && ok;
    if (ok) puts("mx-codes ok");
    return ok ? 0 : 1;
}
