// Checks of the library's host runtime without a GPU: fh_runtime.cpp itself,
// compiled for the host against a stand-in HIP runtime, so that allocations
// can fail, addresses be reused and threads meet.  Usage: runtime_test NAME;
// exit status 0 passed, 1 failed, 77 not applicable here.
#include "../../paper_1407_8333_amd/csrc/fh_runtime.cpp"
#include "launches.h"

#include <thread>

#define CHECK(x)                                                              \
    do {                                                                      \
        if (!(x)) {                                                           \
            std::printf("line %d: %s (%s)\n", __LINE__, #x, fh_last_error()); \
            std::exit(1);                                                     \
        }                                                                     \
    } while (0)

namespace {

const double kSky[3 * 4] = {1, 0, 0, 0, 1, 0, 0, 0, 1, 0, 1, 0};
const fh_select kSel{1000, 4, 8, 2.5};

fh_ctx *make_ctx() {
    fh_ctx *c = nullptr;
    CHECK(fh_ctx_create(0, &c) == FH_OK);
    return c;
}

// n_fft FFTs of `per` peaks each at natural bins 1000, 1002, ...
fh_peakmap *upload(fh_ctx *c, int n_fft, int per) {
    std::vector<int64_t> off(n_fft + 1);
    std::vector<int32_t> bins((size_t)n_fft * per);
    std::vector<double> t(n_fft), v(3 * (size_t)n_fft, 1e-5);
    for (int i = 0; i < n_fft; ++i) {
        off[i + 1] = off[i] + per;
        t[i] = 1000.0 * i;
        for (int k = 0; k < per; ++k) bins[(size_t)i * per + k] = 1000 + 2 * k;
    }
    const fh_peakmap_desc d{n_fft, off[n_fft], off.data(), bins.data(), t.data(), v.data(), 1024.0};
    fh_peakmap *pm = nullptr;
    CHECK(fh_peakmap_upload(c, &d, nullptr, &pm) == FH_OK);
    return pm;
}

fh_grid grid(int nf, int ns) { return fh_grid{10, 10000, nf, ns, -1e-12, 1e-13, 0.0}; }

const fake::Launch *last(const char *what) {
    for (size_t k = fake::launches.size(); k-- > 0;)
        if (!std::strcmp(fake::launches[k].what, what)) return &fake::launches[k];
    return nullptr;
}

fh_candidate g_out[4096];
int g_stream;  // its address stands for a created stream

fh_status search(fh_ctx *c, fh_peakmap *pm, const fh_grid &g, int n_sky, bool graph) {
    const fh_options o{FH_SCHED_PERSISTENT, 0, 0, graph ? 1 : 0};
    return fh_hough_candidates(c, pm, n_sky, kSky, nullptr, 0, &g, &kSel, &o, g_out, (hipStream_t)&g_stream);
}

// A captured search belongs to its peakmap, not to the address: another
// peakmap that takes a released one's address is captured anew.
void captured_search_of_a_released_peakmap() {
    fh_ctx *c = make_ctx();
    const fh_grid g = grid(4000, 17);
    fh_peakmap *a = upload(c, 200, 50);
    CHECK(search(c, a, g, 2, true) == FH_OK && fake::graphs == 1);
    CHECK(search(c, a, g, 2, true) == FH_OK && fake::graphs == 1);
    fh_peakmap_release(c, a);
    fh_peakmap *b = upload(c, 200, 40);
    if (b != a) std::exit(77);
    CHECK(search(c, b, g, 2, true) == FH_OK && fake::graphs == 2);
    CHECK(last("tiles")->n_peaks == 200 * 40);
    fh_peakmap_release(c, b);
    fh_ctx_destroy(c);
}

// A peakmap built from n_fft spectra, of `total` peaks.
fh_status from_spectra(fh_ctx *c, int n_fft, int n_bins, int64_t total, fh_peakmap **pm) {
    static const float sp[1] = {0.0f};
    std::vector<double> t(n_fft), v(3 * (size_t)n_fft, 1e-5);
    for (int i = 0; i < n_fft; ++i) t[i] = 1000.0 * i;
    fake::meta_total = total;
    fake::meta_most = total / n_fft + 1;
    return fh_peakmap_from_spectra(c, n_fft, n_bins, n_bins, sp, nullptr, 1000, 2.5f, t.data(), v.data(), 1024.0,
                                   nullptr, pm);
}

constexpr int64_t kMB = 1 << 20;

// An allocation that succeeds once the released peakmaps' blocks are given
// back leaves no error for the launches after it.
void allocation_after_trimming() {
    fh_ctx *c = make_ctx();
    fh_peakmap *a = upload(c, 1000, 4000), *b = nullptr;  // 16 MB
    fh_peakmap_release(c, a);
    fake::limit = fake::used.load() + 8 * kMB;
    CHECK(from_spectra(c, 1000, 8000, 100000, &b) == FH_OK);  // 16 MB of rows; pool given back
    fake::limit = INT64_MAX;
    fh_peakmap_release(c, b);
    a = upload(c, 1000, 4000);
    fh_peakmap_release(c, a);
    fh_peakmap *d = upload(c, 100, 100);
    fake::limit = fake::used.load() + 8 * kMB;
    fh_server *srv = nullptr;
    CHECK(fh_server_create(c, 16 * kMB, 2, 16, &srv) == FH_OK);
    fake::limit = INT64_MAX;
    CHECK(search(c, d, grid(2000, 17), 2, false) == FH_OK);
    fh_server_destroy(srv);
    fh_peakmap_release(c, d);
    fh_ctx_destroy(c);
}

// A refused allocation fails its own call, not the next one.
void search_after_a_failed_allocation() {
    fh_ctx *c = make_ctx();
    fh_peakmap *d = upload(c, 100, 100);
    fh_server *srv = nullptr;
    fake::limit = fake::used.load() + 8 * kMB;
    CHECK(fh_server_create(c, 16 * kMB, 2, 16, &srv) == FH_E_NOMEM);
    CHECK(search(c, d, grid(2000, 17), 2, false) == FH_OK);
    fake::limit = fake::used.load();
    CHECK(search(c, d, grid(400000, 17), 2, false) == FH_E_NOMEM);
    fake::limit = INT64_MAX;
    CHECK(search(c, d, grid(2000, 17), 2, false) == FH_OK);
    fh_peakmap_release(c, d);
    fh_ctx_destroy(c);
}

// Partial tiles and the rank table are left out where there is no room for
// them; the search runs all the same.
void search_without_room_for_optional_buffers() {
    fh_ctx *c = make_ctx();
    const fh_grid g = grid(4000, 17);
    fh_peakmap *pm = upload(c, 3000, 80);
    const int64_t before = fake::used;
    CHECK(search(c, pm, g, 4, false) == FH_OK);
    CHECK(last("tiles")->parts > 1 && last("front")->rank);
    const int64_t all = fake::used - before, part = (int64_t)c->main_ws.part.bytes, rank = (int64_t)c->main_ws.rank.bytes;
    fh_peakmap_release(c, pm);
    fh_ctx_destroy(c);
    c = make_ctx();
    pm = upload(c, 3000, 80);
    fake::limit = fake::used + all - part - rank;
    for (const bool graph : {false, true}) {
        CHECK(search(c, pm, g, 4, graph) == FH_OK);
        CHECK(last("tiles")->parts == 1 && !last("front")->rank);
    }
    fake::limit = fake::used + rank;
    CHECK(search(c, pm, g, 4, false) == FH_OK);
    CHECK(last("tiles")->parts == 1 && last("front")->rank);
    fake::limit = fake::used + part;
    CHECK(search(c, pm, g, 4, true) == FH_OK);
    CHECK(last("tiles")->parts > 1 && last("front")->rank);
    fh_peakmap_release(c, pm);
    fh_ctx_destroy(c);
}

// Whatever a context keeps only to save time makes room for a call that needs
// it: the row scratch of peakmap construction (16 MB here), partial tiles and
// the rank table, released peakmaps' blocks.
void kept_memory_makes_room() {
    fh_ctx *c = make_ctx();
    fh_peakmap *a = nullptr, *b = nullptr, *pm = upload(c, 3000, 80);
    CHECK(from_spectra(c, 1000, 8000, 100000, &a) == FH_OK);
    const int64_t rows = (int64_t)c->pm_rows.bytes;
    CHECK(rows >= 15 * kMB);
    // a search of more memory than is left without the rows
    fake::limit = fake::used + rows / 2;
    CHECK(search(c, pm, grid(200000, 17), 1, false) == FH_OK);
    CHECK(c->pm_rows.ptr == nullptr);
    // a histogram that takes the place of partial tiles
    fake::limit = INT64_MAX;
    CHECK(search(c, pm, grid(4000, 17), 4, false) == FH_OK && last("tiles")->parts > 1);
    const int64_t part = (int64_t)c->main_ws.part.bytes;
    fake::limit = fake::used + part / 2;
    double stats[2];
    CHECK(fh_robust_stats(c, (const int32_t *)g_out, 100, (int32_t)(part / 8 * 3 / 4), stats, nullptr) == FH_OK);
    CHECK(c->main_ws.part.ptr == nullptr);
    // a peakmap's bins, which do the same while the rows are in use
    fake::limit = INT64_MAX;
    CHECK(from_spectra(c, 1000, 8000, 100000, &b) == FH_OK);
    fh_peakmap_release(c, b);
    CHECK(search(c, pm, grid(4000, 17), 4, false) == FH_OK && last("tiles")->parts > 1);
    fake::limit = fake::used + part / 2;
    CHECK(from_spectra(c, 1000, 8000, part / 4 * 3 / 4, &b) == FH_OK);
    CHECK(c->main_ws.part.ptr == nullptr && c->pm_rows.ptr != nullptr);
    fake::limit = INT64_MAX;
    fh_peakmap_release(c, a);
    fh_peakmap_release(c, b);
    fh_peakmap_release(c, pm);
    fh_ctx_destroy(c);
    CHECK(fake::used == 0);
}

// A request's directions run in one launch when a lane's share of the budget
// holds the search itself: what only saves time is left out first.
void request_in_a_tight_budget() {
    fh_ctx *c = make_ctx();
    const fh_grid g = grid(4000, 17);
    fh_peakmap *pm = upload(c, 3000, 80);
    double sky[3 * 16];
    for (int k = 0; k < 3 * 16; ++k) sky[k] = kSky[k % 3];
    const fh_request q{pm, g, kSel, 16, sky, nullptr, 0, g_out, 0};
    auto served = [&](int64_t budget, int lanes) {
        fh_server *srv = nullptr;
        uint64_t id = 0;
        fh_completion done{};
        int32_t n = 0;
        CHECK(fh_server_create(c, budget, lanes, 16, &srv) == FH_OK);
        CHECK(fh_server_submit(srv, &q, &id) == FH_OK);
        fake::launches.clear();
        CHECK(fh_server_drain(srv) == FH_OK);
        CHECK(fh_server_poll(srv, &done, 1, &n) == FH_OK && n == 1 && done.status == FH_OK);
        CHECK(done.footprint <= budget);
        fh_server_destroy(srv);
        return done.footprint;
    };
    // (the rank table is the last piece of a layout)
    auto bare = [&](int width, int chunk) {
        return (int64_t)search_layout(c, pm, &g, make_plan(g, width), chunk, 16, false).rank;
    };
    const int wide = choose_tile_bins(c, pm, &g, 0), narrow = search_tile_bins(c, pm, &g, 16);
    CHECK(wide > narrow && bare(wide, 16) < bare(narrow, 16));
    CHECK(served(256 * kMB, 2) == bare(wide, 16));
    CHECK(last("tiles")->slots == 16 && last("tiles")->parts > 1 && last("front")->rank);
    for (const int width : {narrow, wide}) {
        CHECK(served(2 * bare(width, 16), 2) == bare(wide, 16));
        CHECK(last("tiles")->slots == 16 && last("tiles")->parts == 1 && !last("front")->rank);
    }
    CHECK(served(2 * (bare(wide, 16) - 256), 2) == bare(wide, 8));
    CHECK(last("tiles")->slots == 8);
    // the least that one direction takes, with a share of half of it
    CHECK(served(bare(wide, 1), 2) == bare(wide, 1));
    CHECK(last("tiles")->slots == 1);
    fh_peakmap_release(c, pm);
    fh_ctx_destroy(c);
}

// Peakmaps released on another thread (as a garbage collector does) while the
// context's own thread builds others: for the thread sanitizer.
void peakmaps_released_on_another_thread() {
    fh_ctx *c = make_ctx();
    for (int rep = 0; rep < 20; ++rep) {
        std::vector<fh_peakmap *> old;
        for (int k = 0; k < 6; ++k) old.push_back(upload(c, 100, 10 + 20 * k));
        std::thread other([&] {
            for (fh_peakmap *p : old) fh_peakmap_release(c, p);
        });
        std::vector<fh_peakmap *> made;
        for (int k = 0; k < 6; ++k) made.push_back(upload(c, 100, 12 + 20 * k));
        fake::limit = fake::used.load();
        fh_server *srv = nullptr;
        CHECK(fh_server_create(c, 64 * kMB, 1, 1, &srv) == FH_E_NOMEM);  // gives the blocks back
        fake::limit = INT64_MAX;
        other.join();
        for (fh_peakmap *p : made) fh_peakmap_release(c, p);
    }
    fh_ctx_destroy(c);
    CHECK(fake::used == 0);
}

// Releasing a peakmap leaves a capture of another thread alone, as freeing
// memory does; during one of its own thread, no block is handed on (the device
// could not be waited for), and no error stays behind.
void peakmap_released_during_a_capture() {
    fh_ctx *c = make_ctx();
    fh_peakmap *a = upload(c, 100, 100), *b = upload(c, 100, 100), *d = upload(c, 100, 100);
    const void *bins = b->d_bins;
    fake::capturing_elsewhere = true;
    fh_peakmap_release(c, a);
    a = upload(c, 200, 200);
    fake::limit = fake::used.load();
    fh_server *srv = nullptr;
    CHECK(fh_server_create(c, 64 * kMB, 1, 1, &srv) == FH_E_NOMEM);  // gives the blocks back
    fake::limit = INT64_MAX;
    CHECK(fake::captures_broken == 0);
    fake::capturing_elsewhere = false;
    fake::capturing_here = true;
    fh_peakmap_release(c, b);
    fake::capturing_here = false;
    CHECK(fake::last_error == hipSuccess);
    b = upload(c, 100, 100);
    CHECK(b->d_bins != bins);
    CHECK(search(c, d, grid(2000, 17), 2, false) == FH_OK);
    for (fh_peakmap *p : {a, b, d}) fh_peakmap_release(c, p);
    fh_ctx_destroy(c);
}

// "tile_parts" is for searches with few tiles: it asks for no gigabytes of
// partial tiles, and a width tuned meanwhile is tuned without it.
void forced_tile_parts() {
    fh_ctx *c = make_ctx();
    fh_peakmap *pm = upload(c, 3000, 80);
    CHECK(fh_ctx_set_option(c, "tile_parts", 16) == FH_OK);
    const fh_options narrow{FH_SCHED_PERSISTENT, 64, 0, 0};
    for (const int nf : {64 * 100, 64 * 1000, 64 * 20000}) {  // tiles of one direction
        const fh_grid g = grid(nf, 15);
        CHECK(fh_hough_candidates(c, pm, 1, kSky, nullptr, 0, &g, &kSel, &narrow, g_out, nullptr) == FH_OK);
        CHECK(last("tiles")->parts == (nf == 64 * 100 ? 16 : nf == 64 * 1000 ? 2 : 1));
        CHECK(c->main_ws.part.bytes < 400 * kMB);
    }
    std::vector<double> sky(3 * 2000);
    for (size_t k = 0; k < sky.size(); ++k) sky[k] = kSky[k % 3];
    std::vector<fh_candidate> out(2 * 7 * 2000);
    const fh_grid g = grid(7000, 15);
    fake::launches.clear();
    CHECK(fh_hough_candidates(c, pm, 2000, sky.data(), nullptr, 0, &g, &kSel, nullptr, out.data(), nullptr) == FH_OK);
    int tuning = 0;
    for (const fake::Launch &l : fake::launches) {
        if (std::strcmp(l.what, "tiles") || l.slots != 128) continue;
        CHECK(l.parts == 1);
        ++tuning;
    }
    CHECK(tuning > 1 && c->tile_parts == 16);
    fh_peakmap_release(c, pm);
    fh_ctx_destroy(c);
}

// Pinned memory that stages a peakmap's times and velocities is bounded, and
// done without where there is none.
void spectra_without_pinned_memory() {
    fh_ctx *c = make_ctx();
    fh_peakmap *pm = nullptr;
    const int64_t pinned = fake::pinned;
    for (const int n_fft : {1000, 600000}) {  // 32 KB and 19 MB
        fake::pinned_limit = n_fft == 1000 ? pinned : INT64_MAX;
        CHECK(from_spectra(c, n_fft, 8, 100, &pm) == FH_OK);
        CHECK(fake::pinned < 16 * kMB);
        for (int i = 0; i < n_fft; i += 999)
            CHECK(pm->d_t[i] == 1000.0 * i && pm->d_v[3 * i] == 1e-5 && pm->d_v[3 * i + 2] == 1e-5);
        fh_peakmap_release(c, pm);
    }
    fh_ctx_destroy(c);
}

// A call that the device refuses (here: one that waits, in a capture) fails
// alone: the next one's launches do not report its error.
void search_after_a_refused_call() {
    fh_ctx *c = make_ctx();
    fh_peakmap *pm = upload(c, 100, 100);
    double stats[2];
    for (const bool capturing : {false, true}) {  // (the first grows the buffers)
        fake::capturing_here = capturing;
        CHECK(fh_robust_stats(c, (const int32_t *)g_out, 10, 100, stats, nullptr) == (capturing ? FH_E_DEVICE : FH_OK));
    }
    fake::capturing_here = false;
    CHECK(search(c, pm, grid(2000, 17), 2, false) == FH_OK);
    fh_peakmap_release(c, pm);
    fh_ctx_destroy(c);
}

// A queued request runs with the window method that its block was laid out
// for: another one needs the full edges, for which there is no place.
void option_changed_behind_a_queued_request() {
    fh_ctx *c = make_ctx();
    fh_peakmap *pm = upload(c, 100, 100);
    const fh_request q{pm, grid(2000, 17), kSel, 2, kSky, nullptr, 0, g_out, 0};
    fh_server *srv = nullptr;
    uint64_t id = 0;
    CHECK(fh_server_create(c, 64 * kMB, 1, 4, &srv) == FH_OK);
    for (const int method : {2, 0}) {
        CHECK(fh_ctx_set_option(c, "window_method", method) == FH_OK);
        CHECK(fh_server_submit(srv, &q, &id) == FH_OK);
        CHECK(fh_ctx_set_option(c, "window_method", 2 - method) == FH_OK);
        fake::launches.clear();
        CHECK(fh_server_drain(srv) == FH_OK);
        CHECK((last("prep") != nullptr) == (method == 0) && c->window_method == 2 - method);
    }
    fh_server_destroy(srv);
    fh_peakmap_release(c, pm);
    fh_ctx_destroy(c);
}

struct Case {
    const char *name;
    void (*run)();
};
const Case kCases[] = {
    {"captured_search_of_a_released_peakmap", captured_search_of_a_released_peakmap},
    {"allocation_after_trimming", allocation_after_trimming},
    {"search_after_a_failed_allocation", search_after_a_failed_allocation},
    {"search_without_room_for_optional_buffers", search_without_room_for_optional_buffers},
    {"kept_memory_makes_room", kept_memory_makes_room},
    {"request_in_a_tight_budget", request_in_a_tight_budget},
    {"peakmaps_released_on_another_thread", peakmaps_released_on_another_thread},
    {"peakmap_released_during_a_capture", peakmap_released_during_a_capture},
    {"forced_tile_parts", forced_tile_parts},
    {"spectra_without_pinned_memory", spectra_without_pinned_memory},
    {"search_after_a_refused_call", search_after_a_refused_call},
    {"option_changed_behind_a_queued_request", option_changed_behind_a_queued_request},
};

}  // namespace

int main(int argc, char **argv) {
    for (const Case &k : kCases)
        if (argc > 1 && !std::strcmp(argv[1], k.name)) {
            k.run();
            return 0;
        }
    std::printf("no such case\n");
    return 1;
}
