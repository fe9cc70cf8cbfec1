// Checks of what csrc/sa_host.cpp prepares for the settled sweeps, one by name (argv[1]); prints "ok".
#include <cstdio>
#include <cstring>
#include <random>
#include <string>
#include <vector>

#include "../paper_2511_17245_amd/csrc/sa_internal.h"

namespace {

int failures = 0;
void expect(bool c, const char *what, int rep) {
    if (c) return;
    if (failures++ < 10) std::fprintf(stderr, "FAILED: %s (problem %d)\n", what, rep);
}

struct Raw {
    int32_t n = 0;
    std::vector<int64_t> ptr{0};
    std::vector<int32_t> fac;
    std::vector<int64_t> coef;
    std::vector<int32_t> lo, hi;
    Raw(int32_t vars, int32_t l, int32_t h) : n(vars), lo((size_t)vars, l), hi((size_t)vars, h) {}
    void term(int64_t c, std::vector<int32_t> v) {
        fac.insert(fac.end(), v.begin(), v.end());
        ptr.push_back((int64_t)fac.size());
        coef.push_back(c);
    }
};

bool pack(const Raw &r, sa::Packed &pk) {
    sa_instance in{r.n, (int64_t)r.coef.size(), r.ptr.data(), r.fac.data(), r.coef.data()};
    sa_bounds bd{r.lo.data(), r.hi.data()};
    sa::Canonical c;
    std::string err;
    return sa::canonicalize(&in, &bd, c, err) == SA_OK && sa::check_int64_bound(c, err, nullptr) == SA_OK &&
           sa::pack(c, pk, err) == SA_OK;
}

// The problems: the two products in which a variable's own record is short and another's is long,
// then random terms of up to six factors with repeated ones, some variables fixed.
std::vector<Raw> problems() {
    std::vector<Raw> out;
    Raw a(30, -2, 3), b(30, -2, 3);
    a.term(3, {0, 0, 1, 2, 3});
    b.term(3, {0, 0, 1, 1, 2});
    for (int32_t i = 0; i + 1 < 30; ++i) {
        a.term(1 + i % 3, {i, i + 1});
        b.term(1 + i % 3, {i, i, i + 1});
    }
    out.push_back(a);
    out.push_back(b);
    // a chain whose only squares are on fixed variables; all variables fixed
    Raw c(40, -2, 3), d(33, 1, 1);
    for (int32_t i = 0; i + 1 < 40; ++i) c.term(1 + i % 3, {i, i + 1});
    c.term(2, {0, 0, 1});
    c.term(2, {7, 7});
    c.lo[0] = c.hi[0] = 2;
    c.lo[7] = c.hi[7] = -1;
    for (int32_t i = 0; i < 33; ++i) d.term(3, {i, i});
    out.push_back(c);
    out.push_back(d);
    std::mt19937_64 g(11);
    for (int rep = 0; rep < 200; ++rep) {
        Raw r(2 + (int32_t)(g() % 40), -2, 3);
        const int m = 1 + (int)(g() % 12);
        const uint64_t most = 1 + g() % 6;
        for (int t = 0; t < m; ++t) {
            std::vector<int32_t> v(1 + g() % most);
            for (size_t q = 0; q < v.size(); ++q)
                v[q] = q > 0 && g() % 3 == 0 ? v[q - 1] : (int32_t)(g() % (uint64_t)r.n);
            r.term(1 + (int64_t)(g() % 9), v);
        }
        for (int32_t i = 0; i < r.n; ++i)
            if (rep % 2 && g() % 4 == 0) r.hi[(size_t)i] = r.lo[(size_t)i];
        out.push_back(r);
    }
    return out;
}

// A change reaches the caches of its neighbours through records of at most three other factors: so no
// cached variable lies in a longer record's list, and the flags are those of the cached variables.
void cached(const sa::Packed &pk, int rep) {
    if (pk.dense) return;
    for (const sa::IncRec &r : pk.inc) {
        const uint32_t no = r.meta >> 8;
        for (uint32_t f = 0; no > 3 && f < no; ++f)
            expect(!pk.cached[(size_t)pk.overflow[(size_t)r.o[0] + f]], "no cached variable in a long record", rep);
    }
    bool any = false, square = false;
    for (int32_t k = 0; k < pk.n; ++k) {
        const bool on = pk.cached[(size_t)k] && pk.var[(size_t)k].width > 1;
        any = any || on;
        square = square || (on && (pk.emask[(size_t)k] & 4u));
    }
    expect(any == pk.any_cached && square == pk.any_square, "flags of the cached variables", rep);
}

// The settled kernel reads a^(2) of every slot that is marked cached and has a power above one, also where no
// update follows: there must be a cache to read. A fixed variable's slot asks for nothing.
void slots(const sa::Packed &pk, int rep) {
    std::vector<sa::SchedRec> order;
    const int32_t n_order = sa::build_order(pk, order);
    int32_t movable = 0;
    for (int32_t k = 0; k < pk.n; ++k) {
        const sa::SchedRec &s = order[(size_t)k];
        const bool fixed = pk.var[(size_t)k].width == 1;
        movable += fixed ? 0 : 1;
        expect(s.k == (fixed ? -1 : k), "slot in index order", rep);
        expect(!fixed || (s.emask == 0 && s.pad[1] == 0), "a fixed variable's slot asks for nothing", rep);
        if (pk.dense || !s.pad[1]) continue;
        expect(pk.any_cached, "a cached slot has a cache", rep);
        expect((s.emask & ~2u) == 0 || pk.any_square, "a cached slot with a square has its cache", rep);
    }
    expect((int32_t)order.size() == pk.n && n_order == movable, "slots of every variable", rep);
}

}  // namespace

int main(int argc, char **argv) {
    const std::string which = argc > 1 ? argv[1] : "";
    int rep = 0;
    for (const Raw &r : problems()) {
        sa::Packed pk;
        if (!pack(r, pk)) {
            expect(false, "packs", rep);
        } else if (which == "cached") {
            cached(pk, rep);
        } else if (which == "slots") {
            slots(pk, rep);
        } else {
            std::fprintf(stderr, "no check named %s\n", which.c_str());
            return 2;
        }
        ++rep;
    }
    if (failures) return 1;
    std::printf("ok\n");
    return 0;
}
