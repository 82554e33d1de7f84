// How an attention call is divided by the scratch that it is lent, on the CPU (test_attn_parts_rule.py links this with
// the library).  Prints one line per rule: its name, then "ok" or what is wrong.
#include <cstdio>

#include "qvg_internal.hpp"

using namespace qvg;

struct Shape { int H; int64_t n_q; };
static const Shape kShapes[] = {{1, 1}, {1, 64}, {1, 300}, {2, 64}, {8, 64}, {3, 700}, {9, 64}, {16, 200}, {5, 600}, {12, 600}, {64, 64}, {65, 64},
                                {40, 700}, {128, 256}, {129, 64}, {256, 64}, {266, 256}, {43, 1290}, {12, 4680}};
constexpr int64_t kTiles = 300, kChunk = (int64_t)1 << 20, kTile = 64;
constexpr size_t kState = 66 * 512 * 4;            // bytes of a query block's part

static AttnParts parts(const Shape &s, int64_t tiles, bool lengths, size_t room = SIZE_MAX) {
    return attn_parts(s.H, s.n_q, tiles * kTile - 3, kChunk, lengths, room);
}
static size_t asked(const Shape &s, int64_t tiles, bool lengths) { return attn_state_bytes(s.H, s.n_q, parts(s, tiles, lengths)); }
static int64_t blocks(const Shape &s) { return s.H * ((s.n_q + 255) / 256); }
static int64_t longest(int64_t tiles, int64_t parts) { return (tiles + parts - 1) / parts; }

// scratch for the longest cache divides every shorter one at least into parts of four tiles, as far as the chip holds them
static const char *longer_caches() {
    for (const Shape &s : kShapes)
        for (int lengths = 0; lengths < 2; ++lengths)
            for (int64_t most = 1; most <= kTiles; ++most) {
                const size_t room = asked(s, most, lengths);
                for (int64_t tiles = 1; tiles <= most; ++tiles) {
                    const AttnParts p = parts(s, tiles, lengths, room), best = parts(s, tiles, lengths);
                    if (blocks(s) > 256 || (lengths && blocks(s) > 128)) {
                        if (p.parts != best.parts || p.whole != best.whole || p.part_tiles != best.part_tiles) return "more than a round of blocks";
                        continue;
                    }
                    const int64_t four = blocks(s) > 64 && tiles < 10 ? 1 : 256 / blocks(s) < tiles / 4 ? 256 / blocks(s) : tiles / 4;
                    if (four > 1 && longest(tiles, p.parts) > longest(tiles, four)) return "longer parts than of four tiles";
                    if (best.parts < four) return "fewer parts than of four tiles";
                    if (p.parts > best.parts && longest(tiles, p.parts) < longest(tiles, best.parts)) return "more than the best";
                }
            }
    return "ok";
}

// with what a call asks for it is divided as with any more, and never into more parts than the scratch holds
static const char *what_is_asked_for() {
    for (const Shape &s : kShapes)
        for (int lengths = 0; lengths < 2; ++lengths)
            for (int64_t tiles = 1; tiles <= kTiles; ++tiles) {
                const AttnParts best = parts(s, tiles, lengths);
                const size_t room = asked(s, tiles, lengths);
                if (parts(s, tiles, lengths, room).parts != best.parts) return "asked for too little";
                if ((best.parts > 1) != (room > 0)) return "asked for nothing";
                for (size_t states = 0; states <= 260; ++states) {
                    const AttnParts p = parts(s, tiles, lengths, states * kState + kState - 1);
                    if (p.parts < 1 || (p.parts > 1 && (size_t)(p.parts * (blocks(s) - p.whole)) > states)) return "does not fit";
                    if (p.parts == 1 && p.whole) return "whole";
                    if (p.parts == 1 && best.aligned && states >= (size_t)(best.aligned * blocks(s))) return "undivided";
                }
            }
    return "ok";
}

int main() {
    std::printf("longer_caches %s\n", longer_caches());
    std::printf("what_is_asked_for %s\n", what_is_asked_for());
    return 0;
}
