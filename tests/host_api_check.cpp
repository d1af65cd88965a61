// Host code of the C ABI (csrc/lskum_api.hip) compiled with g++ on a stand-in
// for the HIP runtime (host_runtime/): the kernels that move fields really move
// them, the others do nothing.  One check per command-line name; exit code 0 if
// it holds.
#include "../paper_2406_07441_amd/csrc/lskum_api.hip"

#include <condition_variable>
#include <thread>

// Time (ms) that the timed kernels take, by the form that they are launched in.
static std::function<double(const lskum::State&)> residual_ms, sweep_ms, qgrad_ms;

namespace lskum {
static hipError_t ok() { return hipSuccess; }
static hipError_t timed(const std::function<double(const State&)>& ms, const State& s) {
    if (ms) fake::now_ms += ms(s);
    return hipSuccess;
}
hipError_t launch_precompute(Cloud&, hipStream_t) { return ok(); }
hipError_t launch_sweep_weights(Cloud&, hipStream_t) { return ok(); }
hipError_t launch_free_stream(State&) { return ok(); }
hipError_t launch_q_from_U(State&) { return ok(); }
hipError_t launch_q_derivatives(State& s, bool) { return timed(qgrad_ms, s); }
hipError_t launch_residual(State& s, int, bool) { return timed(residual_ms, s); }
hipError_t launch_norm(State&, int) { return ok(); }
hipError_t launch_reset_components(State&) { return ok(); }
hipError_t launch_sweeps(State&) { return ok(); }
hipError_t launch_sweep_dir(State& s, bool) { return timed(sweep_ms, s); }
hipError_t launch_update(State&) { return ok(); }
hipError_t launch_explicit_update(State&) { return ok(); }
hipError_t launch_forces(State&) { return ok(); }
hipError_t launch_clear_flags(int32_t*, hipStream_t) { return ok(); }
hipError_t clear_increment(State&, int64_t, int64_t) { return ok(); }
hipError_t reset_cfl(State&) { return ok(); }
hipError_t launch_scratch_begin(State&, double, double, const double*) { return ok(); }
hipError_t launch_residual_out(State&, double*, double*) { return ok(); }
hipError_t launch_soa_to_aos(const double* soa, D4* aos, int64_t n, hipStream_t) {
    for (int64_t p = 0; p < n; ++p) aos[p] = {soa[p], soa[n + p], soa[2 * n + p], soa[3 * n + p]};
    return ok();
}
template <class V>
static hipError_t to_soa(const V* aos, double* soa, int64_t n) {
    for (int64_t p = 0; p < n; ++p) {
        soa[p] = aos[p].x;
        soa[n + p] = aos[p].y;
        soa[2 * n + p] = aos[p].z;
        soa[3 * n + p] = aos[p].w;
    }
    return ok();
}
hipError_t launch_aos_to_soa(const D4* aos, double* soa, int64_t n, hipStream_t) {
    return to_soa(aos, soa, n);
}
hipError_t launch_aosf_to_soa(const F4* aos, double* soa, int64_t n, hipStream_t) {
    return to_soa(aos, soa, n);
}
}  // namespace lskum

static int failures = 0;
#define CHECK(cond)                                                  \
    do {                                                             \
        if (!(cond)) {                                               \
            std::fprintf(stderr, "line %d: %s\n", __LINE__, #cond);  \
            ++failures;                                              \
        }                                                            \
    } while (0)

// A row of n points, each the neighbour of the next.
static lskum_cloud* chain(int64_t n) {
    std::vector<double> x(n), y(n, 0.0);
    std::vector<int8_t> type(n, 1);
    std::vector<int32_t> off(1, 0), idx;
    for (int64_t p = 0; p < n; ++p) {
        x[p] = (double)p;
        if (p) idx.push_back((int32_t)p - 1);
        if (p + 1 < n) idx.push_back((int32_t)p + 1);
        off.push_back((int32_t)idx.size());
    }
    lskum_cloud* c = nullptr;
    CHECK(lskum_cloud_create(n, x.data(), y.data(), type.data(), nullptr, nullptr, off.data(),
                             idx.data(), nullptr, &c) == LSKUM_OK);
    return c;
}

static std::vector<double> field(int64_t n, double base) {
    std::vector<double> U(4 * n);
    for (size_t k = 0; k < U.size(); ++k) U[k] = base + (double)k;
    return U;
}

static lskum_params params() {
    lskum_params p;
    lskum_default_params(&p);
    return p;
}

// Two threads read two conditions of one batch (and one state twice): the
// second call runs while the first waits for its last transposition.
static void concurrent_copies() {
    for (int64_t n : {100, 40000, 140000}) {
        lskum_cloud* c = chain(n);
        const int32_t which[2] = {0, 0};
        const double mach[2] = {0.5, 0.6}, aoa[2] = {0.0, 1.0};
        const lskum_params p = params();
        lskum_batch* b = nullptr;
        CHECK(lskum_batch_create(1, &c, 2, which, mach, aoa, &p, nullptr, &b) == LSKUM_OK);
        const std::vector<double> U0 = field(n, 1.0), U1 = field(n, -1e9);
        CHECK(lskum_batch_set_U(b, 0, U0.data(), 0) == LSKUM_OK);
        CHECK(lskum_batch_set_U(b, 1, U1.data(), 0) == LSKUM_OK);
        std::mutex mu;
        std::condition_variable cv;
        bool go = false, done = false;
        const std::thread::id first = std::this_thread::get_id();
        std::vector<double> got0(4 * n), got1(4 * n);
        std::thread other([&] {
            {
                std::unique_lock<std::mutex> lk(mu);
                cv.wait(lk, [&] { return go; });
            }
            CHECK(lskum_batch_get_U(b, 1, got1.data(), 0) == LSKUM_OK);
            std::lock_guard<std::mutex> lk(mu);
            done = true;
            cv.notify_all();
        });
        fake::on_wait = [&] {
            if (std::this_thread::get_id() != first) return;
            std::unique_lock<std::mutex> lk(mu);
            go = true;
            cv.notify_all();
            // calls that take turns make the other one wait for this one
            cv.wait_for(lk, std::chrono::milliseconds(300), [&] { return done; });
        };
        CHECK(lskum_batch_get_U(b, 0, got0.data(), 0) == LSKUM_OK);
        other.join();
        fake::on_wait = nullptr;
        CHECK(got0 == U0);
        CHECK(got1 == U1);
        lskum_batch_destroy(b);
        lskum_cloud_destroy(c);
    }
    CHECK(fake::pinned_live == 0);
    CHECK(fake::events_live == 0);
}

// Host copies of a state while another device is current: its streams and
// events stay those of its own device, and the caller's device stays current.
static void other_device_current() {
    const int64_t n = 140000;  // more chunks than slots: events both ways
    lskum_cloud* c = chain(n);
    const lskum_params p = params();
    lskum_state* s = nullptr;
    CHECK(lskum_state_create(c, 0.5, 0.0, &p, nullptr, &s) == LSKUM_OK);
    const std::vector<double> U = field(n, 1.0);
    std::vector<double> got(4 * n);
    fake::device = 1;
    CHECK(lskum_state_set_U(s, U.data(), 0) == LSKUM_OK);
    CHECK(lskum_state_get_U(s, got.data(), 0) == LSKUM_OK);
    CHECK(got == U);
    CHECK(fake::foreign_events == 0);
    CHECK(fake::device == 1);
    fake::device = 0;
    lskum_state_destroy(s);
    lskum_cloud_destroy(c);
}

// Pinned memory outlives the states that it served: a program that makes a
// state, reads it and drops it, again and again, pays for it once, also where
// clouds of other sizes come between; all is given back with the last cloud.
static void short_lived_states() {
    lskum_cloud* c[3] = {chain(100), chain(40000), chain(140000)};
    const lskum_params p = params();
    for (int round = 0; round < 4; ++round)
        for (lskum_cloud* cl : c) {
            const int64_t n = cl->c.n;
            lskum_state* s = nullptr;
            CHECK(lskum_state_create(cl, 0.5, 0.0, &p, nullptr, &s) == LSKUM_OK);
            const std::vector<double> U = field(n, round);
            std::vector<double> got(4 * n);
            const int before = fake::event_records;
            CHECK(lskum_state_set_U(s, U.data(), 0) == LSKUM_OK);
            CHECK(n > 98304 || fake::event_records == before);
            CHECK(lskum_state_get_U(s, got.data(), 0) == LSKUM_OK);
            CHECK(got == U);
            lskum_state_destroy(s);
        }
    CHECK(fake::pinned_allocs <= 2);
    CHECK(fake::pinned_live <= 2);
    for (lskum_cloud* cl : c) lskum_cloud_destroy(cl);
    CHECK(fake::pinned_live == 0);
    CHECK(fake::events_live == 0);
}

// Where no memory can be pinned, fields cross all the same, and the failed attempt
// is not reported by a later launch.
static void nothing_to_pin() {
    fake::no_pinned = true;
    for (int64_t n : {100, 40000}) {
        lskum_cloud* c = chain(n);
        const lskum_params p = params();
        lskum_state* s = nullptr;
        CHECK(lskum_state_create(c, 0.5, 0.0, &p, nullptr, &s) == LSKUM_OK);
        const std::vector<double> U = field(n, 1.0);
        std::vector<double> got(4 * n);
        CHECK(lskum_state_set_U(s, U.data(), 0) == LSKUM_OK);
        CHECK(lskum_state_get_U(s, got.data(), 0) == LSKUM_OK);
        CHECK(got == U);
        CHECK(fake::last_error == 0);
        lskum_state_destroy(s);
        lskum_cloud_destroy(c);
    }
    CHECK(fake::events_live == 0);
    fake::no_pinned = false;
}

// The lanes of the q-derivative passes leave the residual's form alone; so does
// asking for the two lanes that the library takes by itself.
static void residual_form() {
    for (int64_t n : {1000, 20000, 200000}) {
        lskum_cloud* c = chain(n);
        for (int32_t lanes : {0, 1, 2, 4, 8}) {
            lskum_params p = params();
            p.residual_lanes = lanes;
            lskum_state* s = nullptr;
            CHECK(lskum_state_create(c, 0.5, 0.0, &p, nullptr, &s) == LSKUM_OK);
            const lskum::ResidualForm want = lskum::residual_form(s->s);
            const bool threads = lanes == 0 || lanes == 2;
            CHECK(want.tiled == (n > 16384 || threads));
            CHECK(want.sub == (!threads || n > 163840 ? 1 : n > 16384 ? 2 : 4));
            for (int32_t q : {1, 2, 4, 8}) {
                p.qgrad_lanes = q;
                CHECK(lskum_state_set_params(s, &p) == LSKUM_OK);
                const lskum::ResidualForm got = lskum::residual_form(s->s);
                CHECK(got.tiled == want.tiled && got.sub == want.sub);
            }
            lskum_state_destroy(s);
        }
        lskum_cloud_destroy(c);
    }
}

// The staged arrays of a tile (112 bytes a listed point, LDS handed out by 1,280
// bytes) take no blocks from a CU that the cloud's longest list leaves room for, of
// the four that the kernels' registers allow.
static void tile_strides() {
    auto blocks = [](int points) { return std::min(4, 128 / ((112 * points + 1279) / 1280)); };
    for (int h = 1; h <= lskum::kQTileMax; ++h) {
        const int s = lskum::tile_stride(h);
        CHECK(s >= h && s <= lskum::kQTileMax);
        CHECK(blocks(s) == blocks(h));
    }
}

// The forms that a state's kernels are launched in.
struct Forms {
    int sweep_lanes, residual_lanes, sub, qgrad_lanes;
    bool tiled, qgrad_tiled;
    explicit Forms(const lskum::State& s)
        : sweep_lanes(s.sweep_lanes), residual_lanes(s.residual_lanes),
          sub(lskum::residual_form(s).sub), qgrad_lanes(s.qgrad_tiled ? 0 : s.qgrad_lanes),
          tiled(lskum::residual_form(s).tiled), qgrad_tiled(s.qgrad_tiled) {}
    bool sweep(const Forms& o) const { return sweep_lanes == o.sweep_lanes; }
    bool residual(const Forms& o) const {
        return residual_lanes == o.residual_lanes && sub == o.sub && tiled == o.tiled;
    }
    bool qgrad(const Forms& o) const {
        return qgrad_tiled == o.qgrad_tiled && qgrad_lanes == o.qgrad_lanes;
    }
};

// Where the forms that the library picks by itself are the fastest, tuning a
// batch leaves it with them, and so do the reported values as parameters; where
// another lane count is the fastest, that one is kept.
static void autotune() {
    for (int64_t n : {500, 9000, 20000, 50000, 100000}) {
        lskum_cloud* c = chain(n);
        const int32_t which[2] = {0, 0};
        const double mach[2] = {0.5, 0.6}, aoa[2] = {0.0, 1.0};
        for (int32_t fastest : {0, 1, 4}) {
            lskum_params p = params();
            p.sweep_lanes = p.residual_lanes = p.qgrad_lanes = fastest;
            lskum_batch* b = nullptr;
            CHECK(lskum_batch_create(1, &c, 2, which, mach, aoa, &p, nullptr, &b) == LSKUM_OK);
            const Forms want(b->s);
            residual_ms = [&](const lskum::State& s) { return Forms(s).residual(want) ? 1.0 : 1.5; };
            sweep_ms = [&](const lskum::State& s) { return Forms(s).sweep(want) ? 1.0 : 1.5; };
            qgrad_ms = [&](const lskum::State& s) { return Forms(s).qgrad(want) ? 1.0 : 1.5; };
            CHECK(lskum_batch_autotune(b, 2, &p.sweep_lanes, &p.residual_lanes, &p.qgrad_lanes) ==
                  LSKUM_OK);
            const Forms tuned(b->s);
            CHECK(tuned.sweep(want) && tuned.residual(want) && tuned.qgrad(want));
            CHECK(lskum_batch_set_params(b, &p) == LSKUM_OK);
            const Forms again(b->s);
            CHECK(again.sweep(want) && again.residual(want) && again.qgrad(want));
            residual_ms = sweep_ms = qgrad_ms = nullptr;
            lskum_batch_destroy(b);
        }
        lskum_cloud_destroy(c);
    }
}

// The runs of a wall of 70 points (two of 32 and one of 6): boxes, coordinates and
// offsets, in one copy to the device.
static void wall_runs() {
    const int64_t n = 140, nwall = 70;
    auto make = [&](int64_t walls) {
        std::vector<double> x(n), y(n), tx(n, 1.0), ty(n, 0.0);
        std::vector<int8_t> type(n, 1);
        std::vector<int32_t> off(1, 0), idx;
        for (int64_t p = 0; p < n; ++p) {
            x[p] = std::cos(0.05 * (double)p);
            y[p] = std::sin(0.05 * (double)p);
            if (p < walls) type[p] = 0;
            if (p) idx.push_back((int32_t)p - 1);
            if (p + 1 < n) idx.push_back((int32_t)p + 1);
            off.push_back((int32_t)idx.size());
        }
        lskum_cloud* c = nullptr;
        CHECK(lskum_cloud_create(n, x.data(), y.data(), type.data(), tx.data(), ty.data(),
                                 off.data(), idx.data(), nullptr, &c) == LSKUM_OK);
        return c;
    };
    int before = fake::device_copies;
    lskum_cloud* none = make(0);
    const int without = fake::device_copies - before;
    before = fake::device_copies;
    lskum_cloud* c = make(nwall);
    CHECK(fake::device_copies - before <= without + 1);  // the list of wall points
    CHECK(none->c.wall_run_off[1] == 0);
    const lskum::Cloud& w = c->c;
    CHECK(w.wall_run_off[0] == 0 && w.wall_run_off[1] == 3);
    CHECK((void*)w.wall_xy == (void*)(w.wall_box + 3));
    for (int r = 0; r < 3; ++r)
        for (int k = 0; k < lskum::kWallRun; ++k) {
            const int64_t p = std::min<int64_t>(r * lskum::kWallRun + k, nwall - 1);
            const lskum::D2 q = w.wall_xy[r * lskum::kWallRun + k];
            const lskum::D4 b = w.wall_box[r];
            CHECK(q.x == w.h_x[p] && q.y == w.h_y[p]);
            CHECK(b.x <= q.x && q.x <= b.y && b.z <= q.y && q.y <= b.w);
        }
    lskum_cloud_destroy(c);
    lskum_cloud_destroy(none);
}

int main(int argc, char** argv) {
    const std::string name = argc > 1 ? argv[1] : "";
    if (name == "concurrent_copies") concurrent_copies();
    else if (name == "other_device_current") other_device_current();
    else if (name == "short_lived_states") short_lived_states();
    else if (name == "nothing_to_pin") nothing_to_pin();
    else if (name == "residual_form") residual_form();
    else if (name == "autotune") autotune();
    else if (name == "tile_strides") tile_strides();
    else if (name == "wall_runs") wall_runs();
    else return 2;
    return failures ? 1 : 0;
}
