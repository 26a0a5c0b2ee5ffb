// wide_table.cpp -- term schedule of the tracker kernel that gives a whole
// wave to one path (ph_track_wide.hpp): which lane sweeps which term, and
// which lane adds which partial into the Jacobian.
//
// The terms of all equations, in an order that keeps every equation's own term
// order, are dealt to the 64 lanes of a wave in rounds of 64; WIDE_ROUNDS
// rounds form a chunk whose partials and values are handed over through LDS
// slots.  After the sweeps of a chunk each Jacobian entry has one lane that
// adds the chunk's partials of that entry in term order, so every sum is made
// of the same additions in the same order as when one lane sweeps a whole
// equation.  The entries are dealt to the lanes longest list first.
#include <algorithm>
#include <numeric>

#include "ph_internal.hpp"

namespace ph {

void build_wide(int n, const std::vector<int32_t> &eq_off, const std::vector<int4> &tdesc,
                const std::vector<uint32_t> &fac, const std::vector<double> &coef, WideTable &w)
{
    w = WideTable{};
    struct Item {
        int key, pos, eq, term;
    };
    // by shape, the order of the terms inside each equation of the table, then by
    // position, then by equation: two counting sorts of the terms as they come
    std::vector<Item> items;
    int positions = 0, keys = 0;
    for (int e = 0; e < n; ++e) {
        positions = std::max(positions, eq_off[e + 1] - eq_off[e]);
        for (int t = eq_off[e]; t < eq_off[e + 1]; ++t) {
            int extra = 0;
            for (int l = 0; l < tdesc[t].x; ++l) extra += fac_exp(fac[tdesc[t].y + l]) - 1;
            items.push_back({tdesc[t].x * (8 * 63 + 1) + extra, t - eq_off[e], e, t});  // k <= 8, exponents <= 64
            keys = std::max(keys, items.back().key + 1);
        }
    }
    std::vector<Item> sorted(items.size());
    std::vector<int> at;
    auto counting_sort = [&](int range, auto &&digit) {
        at.assign(range + 1, 0);
        for (const Item &i : items) ++at[digit(i) + 1];
        std::partial_sum(at.begin(), at.end(), at.begin());
        for (const Item &i : items) sorted[at[digit(i)]++] = i;
        items.swap(sorted);
    };
    counting_sort(positions, [](const Item &i) { return i.pos; });
    counting_sort(keys, [](const Item &i) { return i.key; });
    int np = 4;
    while (np < n) np *= 2;
    const int per = 64 * WIDE_ROUNDS;
    w.rounds = int((items.size() + 63) / 64);
    const int chunks = (w.rounds + WIDE_ROUNDS - 1) / WIDE_ROUNDS;
    w.meta.assign(size_t(w.rounds) * 64, WIDE_NONE);
    w.fac.assign(size_t(w.rounds) * 8 * 64, 0u);
    w.coef.assign(size_t(w.rounds) * 8 * 64, 0.0);
    for (size_t q = 0; q < items.size(); ++q) {
        const size_t r = q / 64, lane = q % 64;
        const int4 d = tdesc[items[q].term];
        w.meta[r * 64 + lane] = uint32_t(d.x) | (uint32_t(d.z) << 8);
        for (int l = 0; l < d.x; ++l) w.fac[(r * 8 + l) * 64 + lane] = fac[d.y + l];
        for (int c = 0; c < 8; ++c) w.coef[(r * 8 + c) * 64 + lane] = coef[size_t(items[q].term) * 8 + c];
    }
    // partials of each entry (column j of equation e: j * np + e) of a chunk, in
    // term order, as ranges of one array; the same for the values of each equation
    std::vector<uint32_t> part, val, cursor;
    std::vector<int> p_off(size_t(np) * np + 1), v_off(n + 1), order, by_count;
    std::vector<uint32_t> lane_list[64];
    std::vector<uint64_t> by_length;
    for (int ch = 0; ch < chunks; ++ch) {
        const size_t q0 = size_t(ch) * per, q1 = std::min(items.size(), q0 + per);
        std::fill(p_off.begin(), p_off.end(), 0);
        std::fill(v_off.begin(), v_off.end(), 0);
        for (size_t q = q0; q < q1; ++q) {
            const int4 d = tdesc[items[q].term];
            for (int l = 0; l < d.x; ++l) ++p_off[size_t(fac_var(fac[d.y + l])) * np + items[q].eq + 1];
            ++v_off[items[q].eq + 1];
        }
        int longest = 0, steps = 0;
        for (size_t e = 0; e + 1 < p_off.size(); ++e) longest = std::max(longest, p_off[e + 1]);
        for (int e = 0; e < n; ++e) steps = std::max(steps, v_off[e + 1]);
        // the entries with partials by their number, most first, then by index
        by_count.assign(longest + 2, 0);
        for (size_t e = 0; e + 1 < p_off.size(); ++e)
            if (p_off[e + 1] > 0) ++by_count[longest - p_off[e + 1] + 1];
        std::partial_sum(by_count.begin(), by_count.end(), by_count.begin());
        order.resize(by_count.back());
        for (size_t e = 0; e + 1 < p_off.size(); ++e)
            if (p_off[e + 1] > 0) order[by_count[longest - p_off[e + 1]]++] = int(e);
        std::partial_sum(p_off.begin(), p_off.end(), p_off.begin());
        std::partial_sum(v_off.begin(), v_off.end(), v_off.begin());
        part.resize(p_off.back());
        val.resize(v_off.back());
        cursor.assign(p_off.begin(), p_off.end() - 1);
        std::vector<int> v_next(v_off.begin(), v_off.end() - 1);
        for (size_t q = q0; q < q1; ++q) {
            const int4 d = tdesc[items[q].term];
            const uint32_t slot = uint32_t(q - q0);
            for (int l = 0; l < d.x; ++l)
                part[cursor[size_t(fac_var(fac[d.y + l])) * np + items[q].eq]++] = uint32_t(l * per) + slot;
            val[v_next[items[q].eq]++] = slot;
        }
        // each to the lane with the shortest list so far (the lanes by the length
        // of their lists, as masks)
        for (auto &v : lane_list) v.clear();
        by_length.assign(part.size() + 1, 0);
        by_length[0] = ~uint64_t(0);
        size_t shortest = 0;
        for (int e : order) {
            while (by_length[shortest] == 0) ++shortest;
            const int l = __builtin_ctzll(by_length[shortest]);
            std::vector<uint32_t> &best = lane_list[l];
            for (int q = p_off[e]; q < p_off[e + 1]; ++q)
                best.push_back(part[q] | (uint32_t(e) << 16) | (q == p_off[e] ? WIDE_FIRST : 0u) |
                               (q + 1 == p_off[e + 1] ? WIDE_LAST : 0u));
            by_length[shortest] &= by_length[shortest] - 1;
            by_length[best.size()] |= uint64_t(1) << l;
        }
        // lane 2 e + c sums component c of equation e; lists are padded to
        // four steps at a time
        size_t gsteps = 0;
        for (auto &v : lane_list) gsteps = std::max(gsteps, v.size());
        const size_t all = (std::max(size_t(steps), gsteps) + 3) / 4 * 4;
        const size_t first = w.list.size();
        w.chunk.push_back(int4{int(first / 64), int(all), int(gsteps), 0});
        w.list.resize(first + all * 64, uint2{0u, WIDE_NONE});
        for (int l = 0; l < 64; ++l) {
            for (size_t s = 0; s < lane_list[l].size(); ++s) w.list[first + s * 64 + l].x = lane_list[l][s];
            const int e = l >> 1;
            if (e < n)
                for (int s = v_off[e]; s < v_off[e + 1]; ++s) w.list[first + size_t(s - v_off[e]) * 64 + l].y = val[s];
        }
    }
}

}  // namespace ph
