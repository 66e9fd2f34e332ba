// Checks of single host+device functions that need no search; prints "ok".
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <sys/mman.h>

#include "fit.h"

thread_local long long pcms_emu_rows, pcms_emu_cands, pcms_emu_walks, pcms_emu_exact, pcms_emu_nodes;

using namespace pcms;

static void check(bool ok, const char *what)
{
    if (ok) return;
    std::printf("failed: %s\n", what);
    std::exit(1);
}

// The words of a target hold its list, the sources ranked for it and the bins,
// and 64 targets fit a one-wave block of 67,840 bytes at most.
static void words()
{
    int most = 0;
    for (int dim = 1; dim <= kMaxDim; ++dim)
        for (int k_cap = 1; k_cap <= kMaxKcap; ++k_cap) {
            for (int mode : {PCMS_RADIUS_FIXED, PCMS_RADIUS_GROW}) {
                const int w = target_words(mode, 0, k_cap, dim);
                check(w >= k_cap && w >= 2, "list in words");
                check(mode == PCMS_RADIUS_FIXED || w >= k_cap + 8, "selection in words");
                most = w > most ? w : most;
            }
            for (int k = 1; k <= 300; ++k) {
                const int w = target_words(PCMS_RADIUS_KNN, k, k_cap, dim);
                check(w >= (k + 8 < k_cap ? k : k_cap) + 8, "nearest list in words");
                check(w >= target_kept(PCMS_RADIUS_KNN, k, k_cap), "kept list in words");
                most = w > most ? w : most;
            }
        }
    std::printf("most words %d\n", most);
    check(most <= kMaxWords && (kMaxWords | 1) * 64 * 4 == 67840, "64 targets in 67,840 bytes");
}

// A ball over all of 2^30 buckets, the most a grid has, reaches the last one
// (offsets of untouched pages: zero).
static void most_buckets()
{
    const int n = 1 << 30;
    const size_t bytes = sizeof(int) * ((size_t)n + 1);
    void *m = mmap(nullptr, bytes, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE,
                   -1, 0);
    check(m != MAP_FAILED, "mmap");
    int *cs = (int *)m;
    cs[n] = 9;
    GridParams gp{};
    gp.dim = gp.sub = 1;
    gp.n[0] = gp.n_cells = n;
    gp.stride[0] = 1;
    gp.hi[0] = n;
    gp.w[0] = gp.inv_w[0] = gp.g[0] = gp.wm = 1.0;
    for (double at : {0.5, 1e9, (double)n - 0.5, 3.0 * n, -2.0 * n}) {
        const double t[1] = {at};
        RowLines<1, false> it(gp, cs, t, 16.0 * n * (double)n);
        int beg[kRows], end[kRows];
        check(it.next(beg, end) && beg[0] == 0 && end[0] == 9, "the ball's range ends at the last bucket");
        check(!it.next(beg, end), "one row");
    }
    munmap(m, bytes);
}

int main()
{
    words();
    most_buckets();
    std::puts("ok");
    return 0;
}
