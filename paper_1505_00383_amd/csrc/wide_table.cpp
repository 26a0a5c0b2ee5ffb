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
    std::vector<Item> items;
    for (int e = 0; e < n; ++e)
        for (int t = eq_off[e]; t < eq_off[e + 1]; ++t) {
            int extra = 0;
            for (int l = 0; l < tdesc[t].x; ++l) extra += fac_exp(fac[tdesc[t].y + l]) - 1;
            // by shape, the order of the terms inside each equation of the table
            items.push_back({(tdesc[t].x << 16) | extra, t - eq_off[e], e, t});
        }
    std::stable_sort(items.begin(), items.end(), [](const Item &a, const Item &b) {
        return a.key != b.key ? a.key < b.key : (a.pos != b.pos ? a.pos < b.pos : a.eq < b.eq);
    });
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
    for (int ch = 0; ch < chunks; ++ch) {
        const size_t q0 = size_t(ch) * per, q1 = std::min(items.size(), q0 + per);
        // partials of each entry (column j of equation e: j * np + e) and
        // values of each equation, in term order
        std::vector<std::vector<uint32_t>> entry(size_t(np) * np), value(n);
        for (size_t q = q0; q < q1; ++q) {
            const int4 d = tdesc[items[q].term];
            const uint32_t slot = uint32_t(q - q0);
            for (int l = 0; l < d.x; ++l)
                entry[size_t(fac_var(fac[d.y + l])) * np + items[q].eq].push_back(uint32_t(l * per) + slot);
            value[items[q].eq].push_back(slot);
        }
        std::vector<int> order;
        for (size_t e = 0; e < entry.size(); ++e)
            if (!entry[e].empty()) order.push_back(int(e));
        std::stable_sort(order.begin(), order.end(),
                         [&](int a, int b) { return entry[a].size() > entry[b].size(); });
        std::vector<std::vector<uint32_t>> lane(64);
        for (int e : order) {
            int best = 0;
            for (int l = 1; l < 64; ++l)
                if (lane[l].size() < lane[best].size()) best = l;
            for (size_t q = 0; q < entry[e].size(); ++q)
                lane[best].push_back(entry[e][q] | (uint32_t(e) << 16) | (q == 0 ? WIDE_FIRST : 0u) |
                                     (q + 1 == entry[e].size() ? WIDE_LAST : 0u));
        }
        // lane 2 e + c sums component c of equation e; lists are padded to
        // four steps at a time
        size_t gsteps = 0, steps = 0;
        for (auto &v : lane) gsteps = std::max(gsteps, v.size());
        for (auto &v : value) steps = std::max(steps, v.size());
        steps = (std::max(steps, gsteps) + 3) / 4 * 4;
        w.chunk.push_back(int4{int(w.list.size() / 64), int(steps), int(gsteps), 0});
        for (size_t s = 0; s < steps; ++s)
            for (int l = 0; l < 64; ++l) {
                const int e = l >> 1;
                w.list.push_back(uint2{s < lane[l].size() ? lane[l][s] : 0u,
                                       e < n && s < value[e].size() ? value[e][s] : WIDE_NONE});
            }
    }
}

}  // namespace ph
