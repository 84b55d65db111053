// CPU driver of tests/test_large_ranges.py: functions of the kernels and of their launches, compiled for
// the host, over all sizes the API accepts.  Prints "ok" when every result is right.
#include <sys/mman.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "ustd_kernels.hpp"

using namespace ustd;

constexpr long long kEnd = (1ll << 31) - 2;  // one past the last slot: nnz is even and below 2^31
constexpr long long kRow = 8192;             // readable slots below it
constexpr int kVerts = 1000;

// The column and weight arrays are reserved address space of the largest size, readable only at the
// row itself, so an access outside ends the process.
// entries [kEnd - kRow, kEnd) of an array that is addressed from its entry 0; 2^31 entries below
// entry 0 are reserved too, where a wrapped index would land
template <typename T>
T *reserve() {
    const size_t half = sizeof(T) << 31;
    void *map = mmap(nullptr, 2 * half, PROT_NONE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    if (map == MAP_FAILED) exit(2);
    char *m = static_cast<char *>(map);
    T *base = reinterpret_cast<T *>(m + half);
    const size_t page = 4096, lo = (size_t)(kEnd - kRow) * sizeof(T) / page * page;
    if (mprotect(reinterpret_cast<char *>(base) + lo, half - lo, PROT_READ | PROT_WRITE) != 0) exit(2);
    return base;
}

void check(bool ok, const char *what, long long a, long long b) {
    if (ok) return;
    printf("wrong: %s %lld %lld\n", what, a, b);
    exit(1);
}

template <int U>
void sums(const int *col, const double *w, const std::vector<double> &p, uint32_t threads) {
    for (long long len : {1ll, 31ll, 129ll, 255ll, 256ll, 257ll, 1000ll, 2047ll, 2048ll, 2049ll, 5000ll, kRow}) {
        const long long lo = kEnd - len;
        for (const double *wt : {(const double *)nullptr, w}) {
            double want = 0, got = 0;
            for (long long e = lo; e < kEnd; ++e) want += (wt ? wt[e] : 1.0) * p[col[e]];
            for (uint32_t t = 0; t < threads; ++t)
                got += row_sum<double, U>(0.0, col, wt, p.data(), (int)lo, (int)kEnd, t, threads);
            check(got == want, "row_sum", U, len);
        }
    }
}

// the row sums of the product on rows that end at the largest slot
void row_sums() {
    int *col = reserve<int>();
    double *w = reserve<double>();
    for (long long e = kEnd - kRow; e < kEnd; ++e) {
        col[e] = (int)(e * 7 % kVerts);
        w[e] = (double)(1 + e % 3);
    }
    std::vector<double> p(kVerts);  // small integers: sums are exact in any order
    for (int v = 0; v < kVerts; ++v) p[v] = v - 400;
    sums<8>(col, w, p, 256);   // heavy rows of the multi-kernel engine
    sums<8>(col, w, p, 1024);  // and of the one-workgroup engine
    for (uint32_t g : {4u, 8u, 16u, 32u}) sums<4>(col, w, p, g);  // light rows
}

// every slot of a row that ends at the largest slot once, by threads in strides; a grid of threads over
// all slots
void row_loops() {
    for (uint32_t step : {4u, 64u, 256u, 1024u})
        for (long long len : {1ll, 63ll, 64ll, 65ll, 255ll, 257ll, 3000ll}) {
            const long long lo = kEnd - len;
            std::vector<int> seen(len, 0);
            for (uint32_t t = 0; t < step; ++t)
                row_each((int)lo, (int)kEnd, t, step, [&](uint32_t e) {
                    check((long long)e >= lo && (long long)e < kEnd, "row_each slot", e, len);
                    ++seen[(long long)e - lo];
                });
            for (long long i = 0; i < len; ++i) check(seen[i] == 1, "row_each count", i, len);
        }
    const uint32_t grid = 8192u * 256u;
    for (uint32_t first : {0u, 1u, grid - 2, grid - 1}) {
        long long count = 0, want = (kEnd - first + grid - 1) / grid;
        row_each(0, (int)kEnd, first, grid, [&](uint32_t e) {
            check((long long)e < kEnd && e % grid == first, "grid slot", e, first);
            check(++count <= want, "grid count", count, first);
        });
        check(count == want, "grid count", count, first);
    }
}

// running sums of a weighted row that ends at the largest slot
void running_sums() {
    double *w = reserve<double>(), *cw = reserve<double>();
    for (long long e = kEnd - kRow; e < kEnd; ++e) w[e] = 1.0 + 1.0 / (double)(e % 97 + 1);
    for (long long len : {1ll, 7ll, 8ll, 9ll, 15ll, 16ll, 1024ll}) {
        double want = 0;
        const double run = row_running_sums(w, cw, (int)(kEnd - len), (int)kEnd);
        for (long long e = kEnd - len; e < kEnd; ++e) check(cw[e] == (want += w[e]), "running sum", e, len);
        check(run == want, "row total", 0, len);
    }
}

// every column of an ascending row that ends at the largest slot, and columns it does not hold
void row_searches() {
    int *col = reserve<int>();
    for (long long e = kEnd - kRow; e < kEnd; ++e) col[e] = (int)(2 * (e - (kEnd - kRow)) + 5);
    for (long long len : {1ll, 2ll, 3ll, 100ll, kRow}) {
        const int lo = (int)(kEnd - len), hi = (int)kEnd;
        for (long long e = lo; e < kEnd; ++e) {
            check(find_in_row(col, lo, hi, col[e]) == e, "find_in_row", e, len);
            check(row_lower_bound(col, lo, hi, col[e]) == e, "row_lower_bound", e, len);
            check(find_in_row(col, lo, hi, col[e] + 1) == -1, "find_in_row absent", e, len);
            check(row_lower_bound(col, lo, hi, col[e] + 1) == (int)(e + 1), "row_lower_bound absent", e, len);
        }
    }
}

// the walk counts of the largest trees: 2^30 - 3 starts past the bitmap, 2^17 within it
template <bool LDS>
void walk_counts_of(long long starts) {
    uint32_t steps = 0, draws = 0;  // lane 0
    long long wave_steps = 0, wave_draws = 0;
    const long long longs = starts / 2;  // walks of 250 steps; the other starts are batch walks by lane 0
    for (long long i = 0; i < longs; ++i) {
        steps += long_walk_lane<LDS>(250, 0) + long_walk_lane<LDS>(250, 1);
        wave_steps += long_walk_wave<LDS>(250);
    }
    for (long long i = longs; i < starts; ++i) steps += kBatchSteps;
    check(wave_steps + steps == 250 * longs + 4 * (starts - longs), "steps", wave_steps, steps);
    for (int w = 0; w < starts; w += 256) {  // a window of starts, each walked to its last recorded step
        if (!LDS && draws_move(w)) {
            wave_draws += draws;
            draws = 0;
        }
        draws += 256 * kWalkDraws;
    }
    const long long want = (starts + 255) / 256 * 256 * kWalkDraws;
    check(wave_draws + draws == want, "draws", wave_draws, draws);
}
void walk_counts() {
    walk_counts_of<false>((1ll << 30) - 3);
    walk_counts_of<true>(1ll << 17);
}

// the one-workgroup solve takes the whole workgroup from one workgroup of row lanes on, at any size
void solve_threads() {
    for (int G : {4, 8, 16, 32})
        for (long long n : {2ll, 1024ll / G - 1, 1024ll / G, 16384ll, 1ll << 26, 1ll << 27, 1ll << 28, 1ll << 29})
            check(small_solve_threads((int)n, G) == (n * G < 1024 ? 256 : 1024), "solve threads", n, G);
}

// kernels launched behind the end of a multi-kernel solve, when the host learns of the end one chunk
// late.  They are to be no more than those of an engine of eight kernels an iteration, with the updates
// inside, enqueued 8, 16, ... 256 iterations at a time (what the three kernels a slot took the place of).
template <typename Next>
long long launched(long long needed, int chunk, Next next) {
    long long total = chunk;
    for (; total < needed; total += chunk) chunk = next(chunk);
    return total + next(chunk);
}
void solve_chunks() {
    for (int it = 1; it <= 3000; ++it)
        for (int updates = 1; updates <= 6 && updates <= it; ++updates) {
            const long long slots = it + updates;
            const long long now = 3 * (launched(slots, kSolveChunkFirst, solve_chunk_after) - slots);
            const long long then = 8 * (launched(it, 8, [](int c) { return c < 128 ? 2 * c : 256; }) - it);
            check(now <= then, "empty kernels", it, updates);
        }
}

// the largest vertex of the largest graph (of the largest block-split graph) is no free mark, and keeps
// clear of a word's flag bits
void vertex_ids() {
    for (long long count : {2ll, (1ll << 30) - 2}) check(ids_fit(count), "ids", count, 0);
    for (long long count : {(1ll << 30) - 1, 1ll << 30, (1ll << 31) - 6}) check(!ids_fit(count), "ids", count, 1);
}

int main(int argc, char **argv) {
    const char *what = argc > 1 ? argv[1] : "";
    if (!strcmp(what, "row_sums")) row_sums();
    else if (!strcmp(what, "row_loops")) row_loops();
    else if (!strcmp(what, "running_sums")) running_sums();
    else if (!strcmp(what, "row_searches")) row_searches();
    else if (!strcmp(what, "walk_counts")) walk_counts();
    else if (!strcmp(what, "solve_threads")) solve_threads();
    else if (!strcmp(what, "solve_chunks")) solve_chunks();
    else if (!strcmp(what, "vertex_ids")) vertex_ids();
    else return 2;
    puts("ok");
    return 0;
}
