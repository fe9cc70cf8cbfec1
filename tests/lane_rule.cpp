// The choice of the lane kernel (csrc/sa_host.cpp, lane_waves) and its image, checked on the host.  argv[1]
// names a check; prints "ok".
#include <cmath>
#include <cstdio>
#include <cstring>
#include <random>
#include <set>
#include <string>
#include <vector>

#include "../paper_2511_17245_amd/csrc/sa_internal.h"

namespace {

int failures = 0;
void expect(bool c, const char *what, int n, double d, int w) {
    if (c) return;
    ++failures;
    std::fprintf(stderr, "FAILED: %s (N %d, degree %g, W %d)\n", what, n, d, w);
}

// A random pair graph of mean degree d, variable 0 joined to `hub` others; W values per variable.
sa::Packed graph(int n, double d, int W, int hub, unsigned seed, int64_t jmax = 10) {
    std::mt19937_64 g(seed);
    std::set<std::pair<int, int>> edges;
    while ((double)edges.size() < d * n / 2) {
        const int a = (int)(g() % (unsigned)n), b = (int)(g() % (unsigned)n);
        if (a != b) edges.insert({std::min(a, b), std::max(a, b)});
    }
    for (int j = 1; j <= hub; ++j) edges.insert({0, j});
    std::vector<int64_t> ptr{0}, coef;
    std::vector<int32_t> fac, lo((size_t)n, -(W / 2)), hi((size_t)n, -(W / 2) + W - 1);
    for (auto &e : edges) {
        fac.push_back(e.first);
        fac.push_back(e.second);
        ptr.push_back((int64_t)fac.size());
        coef.push_back(1 + (int64_t)(g() % (uint64_t)jmax));
    }
    sa_instance in{n, (int64_t)coef.size(), ptr.data(), fac.data(), coef.data()};
    sa_bounds bd{lo.data(), hi.data()};
    sa::Canonical c;
    sa::Packed pk;
    std::string err;
    if (sa::canonicalize(&in, &bd, c, err) != SA_OK || sa::pack(c, pk, err) != SA_OK) expect(false, "packs", n, d, W);
    return pk;
}

int waves(const sa::Packed &pk, int reads, bool quad, sa::LaneImage &im) {
    sa::build_lane_chunks(pk, im);
    return sa::lane_waves(im, pk, true, reads, quad ? 128 : 0, 256, 160 * 1024);
}

// Given to the lane kernel or not, as measured (with the quad kernel for up to 128 values per variable)
void choice() {
    struct Case {
        int n;
        double d;
        int W, hub;
        bool lane;
    };
    const Case cases[] = {
        {100, 3, 40, 0, true},     {300, 8, 40, 0, true},      {1000, 8, 2, 0, true},       {1000, 16, 40, 0, true},
        {4000, 25, 40, 0, true},   {10000, 8, 101, 0, true},   {12000, 25, 300, 0, true},   {12000, 16, 2, 0, true},
        {1000, 40, 40, 0, false},  {4000, 80, 2, 0, false},    {4000, 150, 300, 0, false},  {4000, 250, 40, 0, false},
        {12000, 80, 40, 0, false}, {12000, 250, 40, 0, false}, {10000, 4, 20, 9999, false}, {30000, 4, 20, 29999, false},
        {10000, 4, 20, 500, true},
    };
    for (const Case &c : cases) {
        const sa::Packed pk = graph(c.n, c.d, c.W, c.hub, 7);
        for (int reads : {1, 64, 1024}) {
            sa::LaneImage im;
            expect((waves(pk, reads, c.W <= 128, im) > 0) == c.lane, c.lane ? "lane kernel" : "another kernel", c.n, c.d, c.W);
            expect(im.recs.empty(), "no records before the choice", c.n, c.d, c.W);
        }
    }
}

// Every record of every variable is in its lane's rows, the rest is empty; rounds cover the chunks in order
void image() {
    for (bool compact : {true, false}) {
        const sa::Packed pk = graph(700, 6, 30, 90, 3, compact ? 10 : 100000);
        expect(pk.pair16 == compact, "16-bit records", 700, 6, 30);
        sa::LaneImage im;
        sa::build_lane_chunks(pk, im);
        sa::build_lane_records(pk, compact, im);
        const size_t rb = compact ? 4 : 8;
        expect(im.recs.size() == (size_t)(im.n_rows + sa::kLaneReach) * 64 * rb, "rows and the reach past them", 700, 6, 30);
        std::vector<int> seen((size_t)pk.n, 0);
        size_t used = 0, full = 0;
        for (size_t c = 0; c < im.chunks.size(); ++c)
            for (size_t q = 0; q < 64; ++q) {
                const int32_t k = im.slots[c * 64 + q].k;
                if (k < 0) continue;
                seen[(size_t)k]++;
                expect(im.slots[c * 64 + q].h == pk.pair_h[(size_t)k], "linear coefficient", 700, 6, 30);
                expect(pk.pair_deg[(size_t)k] <= im.chunks[c].rows, "rows hold the degree", 700, 6, 30);
                for (int32_t i = 0; i < pk.pair_deg[(size_t)k]; ++i, ++used) {
                    const sa::PairRec &want = pk.pair[(size_t)pk.pair_row[(size_t)k] + (size_t)i];
                    const uint8_t *at = im.recs.data() + ((size_t)(im.chunks[c].first + i) * 64 + q) * rb;
                    if (compact) {
                        uint32_t w;
                        std::memcpy(&w, at, 4);
                        expect((int32_t)(w & 0xFFFFu) == want.j && (int32_t)w >> 16 == want.J, "record", 700, 6, 30);
                    } else {
                        expect(std::memcmp(at, &want, 8) == 0, "record", 700, 6, 30);
                    }
                }
            }
        for (int v : seen) expect(v == 1, "every variable once", 700, 6, 30);
        for (size_t i = 0; i < im.recs.size(); i += rb) {
            bool any = false;
            for (size_t b = 0; b < rb; ++b) any = any || im.recs[i + b];
            full += any;
        }
        expect(full == used, "the rest is empty", 700, 6, 30);
        for (int w : {1, 2, 4, 8}) {
            std::vector<sa::LaneRows> rounds;
            sa::build_lane_rounds(im, w, rounds);
            int32_t next = 0;
            for (const sa::LaneRows &r : rounds) {
                const int32_t end = r.rows < 0 ? ~r.rows : r.rows;
                expect(r.first == next && (r.rows < 0) == (r.first + w >= end), "rounds in order", 700, 6, 30);
                next = std::min(r.first + w, end);
            }
            expect(next == (int32_t)im.chunks.size(), "rounds cover the chunks", 700, 6, 30);
        }
    }
}

}  // namespace

// Levels from neighbours that two kernels share, and by definition: after all lower neighbours, as many as
// the longest chain.  With long terms, repeated factors and fixed variables.
void levels() {
    std::mt19937_64 g(11);
    for (int rep = 0; rep < 60; ++rep) {
        const int n = 2 + (int)(g() % 90), m = 1 + (int)(g() % (unsigned)(3 * n)), most = rep % 3 == 0 ? 2 : 6;
        std::vector<int64_t> ptr{0}, coef;
        std::vector<int32_t> fac, lo((size_t)n, 0), hi((size_t)n, 3);
        for (int k = 0; k < n; k += 5) hi[(size_t)k] = (int32_t)(g() % 2) * 3;
        for (int t = 0; t < m; ++t) {
            const int d = 1 + (int)(g() % (unsigned)most);
            for (int i = 0; i < d; ++i) fac.push_back((int32_t)(g() % (unsigned)n));
            ptr.push_back((int64_t)fac.size());
            coef.push_back(1 + (int64_t)(g() % 9));
        }
        sa_instance in{n, (int64_t)coef.size(), ptr.data(), fac.data(), coef.data()};
        sa_bounds bd{lo.data(), hi.data()};
        sa::Canonical c;
        std::string err;
        sa::Packed p;
        if (sa::canonicalize(&in, &bd, c, err) != SA_OK || sa::pack(c, p, err) != SA_OK) {
            expect(false, err.c_str(), n, m, rep);
            continue;
        }
        sa::LevelGraph graph;
        for (int32_t quads : {64, 16, 64, 1}) {
            std::vector<int32_t> s0, s1;
            std::vector<sa::SchedRec> a, b;
            const int32_t n0 = sa::build_levels(p, quads, s0, a), n1 = sa::build_levels(p, quads, s1, b, &graph);
            expect(n0 == n1 && s0 == s1 && a.size() == b.size() &&
                       (a.empty() || std::memcmp(a.data(), b.data(), a.size() * sizeof(a[0])) == 0), "shared neighbours", n, m, quads);
            std::vector<int> at((size_t)n, -1), first((size_t)n, 0);
            for (int32_t l = 0; l < n0; ++l)
                for (int32_t i = s0[(size_t)l]; i < s0[(size_t)l + 1]; ++i) at[(size_t)a[(size_t)i].k] = l;
            int longest = 0;
            for (int k = 0; k < n; ++k) {
                expect((at[(size_t)k] >= 0) == (hi[(size_t)k] > 0), "every variable that is not fixed", n, m, k);
                if (at[(size_t)k] < 0) continue;
                // (of the packed problem: pairs whose coefficients cancel are no neighbours)
                for (int64_t t = 0; t < (int64_t)c.t_coef.size(); ++t) {
                    bool has = false;
                    for (int64_t q = c.t_off[(size_t)t]; q < c.t_off[(size_t)t + 1]; ++q) has = has || c.t_var[(size_t)q] == k;
                    for (int64_t q = c.t_off[(size_t)t]; has && q < c.t_off[(size_t)t + 1]; ++q) {
                        const int j = c.t_var[(size_t)q];
                        if (j >= k || at[(size_t)j] < 0) continue;
                        expect(at[(size_t)j] < at[(size_t)k], "after its lower neighbours", n, m, k);
                        first[(size_t)k] = std::max(first[(size_t)k], first[(size_t)j] + 1);
                    }
                }
                longest = std::max(longest, first[(size_t)k] + 1);
            }
            if (!p.dense) expect(n0 == longest, "as many levels as the longest chain", n, m, n0);
        }
    }
}

int main(int argc, char **argv) {
    const std::string which = argc > 1 ? argv[1] : "";
    if (which == "choice") choice();
    else if (which == "image") image();
    else if (which == "levels") levels();
    else return 2;
    if (failures) return 1;
    std::printf("ok\n");
    return 0;
}
