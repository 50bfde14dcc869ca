// The candidates that a ranking's sample takes (plain C++; constexpr functions run on either side).
//
// A tile of the sample has 32 rows, row r of part r of the table.  The parts lie apart by gaps that grow evenly, a 32nd of the table in all, so
// that a period of the table is at another phase in every part.  A part is cut into as many pieces as the sample has tiles, and a
// tile takes one piece's candidate of every part, at a place that moves on by 0.618 of the piece with every piece: all phases of a period.
// No candidate is taken twice - as many as KP maxima over groups of them stand for as many candidates.
#pragma once
#include <cstdint>

struct TopkSample {
    int32_t part, gap;                  // row r: the candidates first(r) .. first(r) + part - 1
    int32_t w, rem;                     // pieces of w of them (the first rem pieces one longer)
    constexpr int32_t first(int row) const { return row * part + row * (row + 1) / 2 * gap; }
    constexpr uint32_t place(uint32_t piece) const {
        const uint32_t longer = piece < (uint32_t)rem;
        return piece * (uint32_t)w + (longer ? piece : (uint32_t)rem) + (uint32_t)((uint64_t)(piece * 0x9E3779B1u) * ((uint32_t)w + longer) >> 32);
    }
};

constexpr TopkSample topk_sample(int64_t ncand, int64_t tiles) {        // (32 tiles <= ncand)
    constexpr int64_t GAPS = 32 * 31 / 2;
    int64_t gap = ncand / (32 * GAPS);
    if (gap > 1 && gap % 2 == 0) --gap;
    if ((ncand - GAPS * gap) / 32 < tiles) gap = 0;
    const int64_t part = (ncand - GAPS * gap) / 32;
    return TopkSample{(int32_t)part, (int32_t)gap, (int32_t)(part / tiles), (int32_t)(part % tiles)};
}
