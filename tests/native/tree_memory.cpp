// Host checks of the tree's memory management (csrc/sph_impl.h), on regions
// that stand in for device memory: addresses are compared, nothing is read.
// Prints "ok <check>" per check; a failing one ends the program.
#include <cstdio>
#include <cstdlib>
#include <random>
#include <utility>
#include <vector>

#include "../../paper_1309_3783_amd/csrc/sph_impl.h"

namespace sph {
// as in sph_prims.hip, whose kernels these checks do without
size_t scan_tmp_words(int64_t n) { return (size_t)((n + 4095) / 4096) + 1; }
}  // namespace sph

static void expect(bool ok, const char* what) {
    if (!ok) {
        std::printf("FAILED %s\n", what);
        std::exit(1);
    }
}

static bool inside(const void* p, const char* region, size_t bytes) {
    return (const char*)p >= region && (const char*)p < region + bytes;
}

// The scan scratch lies in the memory that the tree holds now: after another
// workspace was attached, and after an allocation failed.
static void scratch_follows_the_memory() {
    const size_t MB = (size_t)1 << 20;
    char* a = (char*)std::aligned_alloc(256, 8 * MB);
    char* b = (char*)std::aligned_alloc(256, 8 * MB);
    sph_tree t;
    expect(!t.set_workspace(a, 8 * MB, 0).st && !t.scratch(10000).st, "attach a");
    expect(inside(t.sc_a, a, 8 * MB) && inside(t.sc_tmp, a, 8 * MB), "scratch in a");
    expect(!t.set_workspace(b, 8 * MB, 0).st && !t.scratch(9000).st, "attach b");
    for (const void* p : {(void*)t.sc_a, (void*)t.sc_b, (void*)t.sc_c, (void*)t.sc_d, (void*)t.sc_tmp,
                          (void*)t.d_total, (void*)t.d_maxleaf, (void*)t.d_npairs})
        expect(inside(p, b, 8 * MB), "scratch moved to b");
    // the same region attached again: a block of the tree's, not only an address in it
    expect(!t.set_workspace(b, 8 * MB, 0).st && !t.scratch(9000).st && t.b_sc.p == (void*)t.sc_a, "scratch is a block");
    // too large for the region: what there was is gone, the next call takes it anew
    expect(t.scratch(1 << 20).st == SPH_E_WORKSPACE, "too large");
    expect(!t.scratch(9000).st && t.b_sc.p == (void*)t.sc_a && t.b_sc.p, "scratch after a failure");
    t.release();
    std::free(a);
    std::free(b);
    std::printf("ok scratch_follows_the_memory\n");
}

// The reduction table kept for the next call of the same sets counts only
// while its block is held: not after it made way for one that did not fit.
static void reduction_table_needs_its_block() {
    const size_t MB = (size_t)1 << 20;
    char* a = (char*)std::aligned_alloc(256, MB);
    sph_tree t;
    void* p = nullptr;
    expect(!t.set_workspace(a, MB, 0).st, "attach");
    t.off = {0, 1000};
    expect(!t.red_made(), "none yet");
    expect(!t.alloc(t.b_red, 1000, &p).st, "table");
    t.red_off = t.off;
    expect(t.red_made(), "made");
    expect(t.alloc(t.b_red, 2 * MB, &p).st == SPH_E_WORKSPACE, "does not fit");
    expect(!t.red_made(), "gone");
    expect(!t.alloc(t.b_red, 1000, &p).st, "table again");
    t.red_off = t.off;
    t.off = {0, 500, 1000};
    expect(!t.red_made(), "other sets");
    t.release();
    std::free(a);
    std::printf("ok reduction_table_needs_its_block\n");
}

// The blocks that a tree can do without change nothing for the others: in
// every workspace the same allocations succeed, at the same places, as without
// them, and no two blocks held overlap.
static void optional_blocks_refuse_nothing() {
    const size_t room = (size_t)4 << 20;
    char* a = (char*)std::aligned_alloc(256, room);
    char* b = (char*)std::aligned_alloc(256, room);
    std::mt19937 rng(12345);
    auto pick = [&](int lo, int hi) { return std::uniform_int_distribution<int>(lo, hi)(rng); };
    int refused = 0, dropped = 0;
    for (int trial = 0; trial < 2000; ++trial) {
        sph_tree with, without;
        const size_t bytes = (size_t)pick(1 << 20, (int)room);
        expect(!with.set_workspace(a, bytes, 0).st && !without.set_workspace(b, bytes, 0).st, "attach");
        sph::DevBuf sph_tree::*bufs[] = {&sph_tree::b_key, &sph_tree::b_pos, &sph_tree::b_cell, &sph_tree::b_sc,
                                         &sph_tree::b_plist, &sph_tree::b_part, &sph_tree::b_red, &sph_tree::b_force};
        const int scale = pick(100, (int)(bytes / 3));
        for (int step = 0; step < 60; ++step) {
            void *p = nullptr, *q = nullptr;
            if (pick(0, 3) == 0) {
                sph::DevBuf& opt = pick(0, 1) ? with.b_order : with.b_park;
                const bool ok = with.try_alloc(opt, (size_t)pick(1, scale), &p);
                expect(!ok || p == opt.p, "optional block");
            } else {
                auto m = bufs[pick(0, 7)];
                const size_t want = (size_t)pick(1, scale);
                const bool held = with.b_order.p || with.b_park.p;
                const bool grows = pick(0, 4) == 0;
                const sph::Err e1 = grows ? with.grow(with.*m, 0, want, &p) : with.alloc(with.*m, want, &p);
                const sph::Err e2 = grows ? without.grow(without.*m, 0, want, &q) : without.alloc(without.*m, want, &q);
                expect(e1.st == e2.st, "refused with optional blocks only");
                expect(e1.st || (char*)p - a == (char*)q - b, "place");
                expect((with.*m).cap == (without.*m).cap && with.ws_needed == without.ws_needed, "size");
                refused += e1.st ? 1 : 0;
                dropped += held && !with.b_order.p && !with.b_park.p ? 1 : 0;
            }
            std::vector<std::pair<char*, size_t>> at;
            size_t sum = 0;
            for (const sph::DevBuf* d : with.bufs())
                if (d->p) {
                    at.emplace_back((char*)d->p, d->cap);
                    sum += d->cap;
                }
            std::sort(at.begin(), at.end());
            for (size_t k = 0; k < at.size(); ++k)
                expect(at[k].first >= a && at[k].first + at[k].second <= (k + 1 < at.size() ? at[k + 1].first : a + bytes),
                       "overlap");
            expect(with.bytes() == sum && with.ar.high >= sum, "held");
        }
        with.drop_optional();
        expect(with.ar.in_use == without.ar.in_use && with.ar.free_ == without.ar.free_, "free");
    }
    expect(refused > 500 && dropped > 500, "both met");
    std::free(a);
    std::free(b);
    std::printf("ok optional_blocks_refuse_nothing\n");
}

int main() {
    optional_blocks_refuse_nothing();
    reduction_table_needs_its_block();
    scratch_follows_the_memory();
    return 0;
}
