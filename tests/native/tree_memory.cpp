// Host checks of the tree's memory management (csrc/sph_impl.h), on regions
// that stand in for device memory: addresses are compared, nothing is read.
// Prints "ok <check>" per check; a failing one ends the program.
#include <cstdio>
#include <cstdlib>

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

int main() {
    reduction_table_needs_its_block();
    scratch_follows_the_memory();
    return 0;
}
