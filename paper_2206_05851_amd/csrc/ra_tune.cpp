// ra_tune.cpp — cost-model and timing autotuner for the per-group tile and
// the launch's wavefronts per workgroup.
#include "ra_tune.hpp"

#include "ra_launch.hpp"

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <fstream>
#include <map>
#include <mutex>
#include <tuple>

namespace ra {

const std::vector<int>& family_beads_per_lane(int family) {
    static const std::vector<int> small{1, 2, 3, 4};
    static const std::vector<int> large{6, 8, 12, 16};
    return family == 4 ? small : large;
}

static bool legal(int n_beads, int M) { return (n_beads + M - 1) / M <= 64; }

bool map_allows(int nmap, int M) { return nmap != 2 || M % 4 == 0; }

int choose_beads_per_lane(int n_beads, int n_replicas, int family, int forced, int nmap, int widest) {
    const auto& cand = family_beads_per_lane(family);
    if (forced > 0 && legal(n_beads, forced) && map_allows(nmap, forced))
        for (int m : cand)
            if (m == forced) return m;
    int best = -1;
    long long best_cost = 0;
    for (int M : cand) {
        if (!legal(n_beads, M) || !map_allows(nmap, M)) continue;
        if (best > 0 && M > widest) break;
        const int L = (n_beads + M - 1) / M;
        const int P = 64 / L;
        const long long cost = (long long)M * ((n_replicas + P - 1) / P);
        if (best < 0 || cost < best_cost) { best = M; best_cost = cost; }
    }
    return best < 0 ? cand.back() : best;
}

// Time of a launch of few items, the widest with M beads per lane: measured, us
// per 400 steps, up to 256, 512, 768, 1024, 1536 and 2048 items (the split forward's
// workgroups go one to a CU, the others' wavefronts one to a SIMD).
static constexpr int FEW_ITEMS[6] = {256, 512, 768, 1024, 1536, 2048};
static int few_items_class(int64_t n_items) {
    int i = 0;
    while (n_items > FEW_ITEMS[i]) ++i;
    return i;
}
static double few_items_cost(int M, int64_t n_items, int precision) {
    static constexpr double f32[4][6] = {{61, 74, 85, 100, 143, 147},
                                         {90, 115, 170, 184, 260, 265},
                                         {119, 223, 226, 230, 357, 367},
                                         {143, 272, 281, 290, 450, 455}};
    static constexpr double f64[6] = {100, 195, 290, 355, 590, 600};   // times M
    const int i = few_items_class(n_items);
    return precision == 64 ? M * f64[i] : f32[M - 1][i];
}

std::vector<int> choose_tiles(const ra_chain_desc* groups, int n_groups, int family, int precision, int forced,
                              int nmap) {
    auto tiles = [&](int widest, int64_t& n_items, int& max_m) {
        std::vector<int> Ms(n_groups);
        n_items = 0;
        max_m = 1;
        for (int i = 0; i < n_groups; ++i) {
            const int N = groups[i].n_beads, R = groups[i].n_replicas;
            Ms[i] = choose_beads_per_lane(N, R, family, forced, nmap, widest);
            const int P = std::max(1, 64 / ((N + Ms[i] - 1) / Ms[i]));
            n_items += (R + P - 1) / P;
            max_m = std::max(max_m, Ms[i]);
        }
        return Ms;
    };
    int64_t n_items;
    int max_m;
    std::vector<int> best = tiles(64, n_items, max_m);
    if (forced > 0 || family != 4 || n_items > FEW_ITEMS[5]) return best;
    double cost = few_items_cost(max_m, n_items, precision);
    for (int widest = max_m - 1; widest >= 1; --widest) {
        std::vector<int> Ms = tiles(widest, n_items, max_m);
        if (n_items > FEW_ITEMS[5]) break;
        const double t = few_items_cost(max_m, n_items, precision);
        if (t <= cost) {
            cost = t;
            best = Ms;
        }
    }
    return best;
}

namespace {

// One tuning result: the fastest M for a chain length and spring law under a
// precision, kernel family, wavefronts per workgroup and noise map, and its
// time per replica for 96 steps (to compare workgroup sizes across a batch); for
// work lists of at most that many items where they do not fill the chip (FEW_ITEMS),
// 0 for longer ones. Lines of a cache file without "items" hold for every list.
using Key = std::tuple<int, int, int, int, int, int, int>;   // N, spring, precision, family, wpb, noise_map, items
constexpr int ANY_ITEMS = -1;
struct Entry {
    int M;
    double ms_per_replica;
};
constexpr int TUNE_WAVES_PER_SIMD = 4;             // timing runs fill every SIMD at least this many times
constexpr double TUNE_TILE_GAIN = 0.97;            // a tile other than the cost model's has to be this much faster

// The process keeps one table of results per cache file (the empty path when
// RA_AUTOTUNE_CACHE is unset): the library's only process-wide state. Tuning
// results depend on the device model and the library build, not on a
// context, so contexts with the same groups share them.
std::mutex g_mu;
std::map<std::string, std::map<Key, Entry>> g_tables;

std::map<Key, Entry>& table_for(const std::string& path) {
    auto it = g_tables.find(path);
    if (it != g_tables.end()) return it->second;
    std::map<Key, Entry>& t = g_tables[path];
    if (path.empty()) return t;
    std::ifstream f(path);
    // one entry per line: {"N": .., "spring": .., "precision": .., "family": .., "wpb": ..,
    //                      "noise_map": .., "items": .., "M": .., "ms_per_replica": ..}
    std::string line;
    while (f && std::getline(f, line)) {
        int v[7], items = ANY_ITEMS;
        double ms = 0.0;
        if (std::sscanf(line.c_str(),
                        " {\"N\": %d, \"spring\": %d, \"precision\": %d, \"family\": %d, \"wpb\": %d, "
                        "\"noise_map\": %d, \"items\": %d, \"M\": %d, \"ms_per_replica\": %lf}",
                        &v[0], &v[1], &v[2], &v[3], &v[4], &v[5], &items, &v[6], &ms) == 9) {
            t[Key{v[0], v[1], v[2], v[3], v[4], v[5], items}] = Entry{v[6], ms};
            continue;
        }
        if (std::sscanf(line.c_str(),
                        " {\"N\": %d, \"spring\": %d, \"precision\": %d, \"family\": %d, \"wpb\": %d, "
                        "\"noise_map\": %d, \"M\": %d, \"ms_per_replica\": %lf}",
                        &v[0], &v[1], &v[2], &v[3], &v[4], &v[5], &v[6], &ms) == 8)
            t[Key{v[0], v[1], v[2], v[3], v[4], v[5], ANY_ITEMS}] = Entry{v[6], ms};
    }
    return t;
}

void append_cache_file(const std::string& path, const Key& k, const Entry& e) {
    if (path.empty()) return;
    std::ofstream f(path, std::ios::app);
    char buf[256];
    std::snprintf(buf, sizeof buf,
                  "{\"N\": %d, \"spring\": %d, \"precision\": %d, \"family\": %d, \"wpb\": %d, "
                  "\"noise_map\": %d, \"items\": %d, \"M\": %d, \"ms_per_replica\": %.9g}\n",
                  std::get<0>(k), std::get<1>(k), std::get<2>(k), std::get<3>(k), std::get<4>(k),
                  std::get<5>(k), std::get<6>(k), e.M, e.ms_per_replica);
    f << buf;
}

// Time 96 fused steps of one group with a forced tile M of the batch's kernel
// family (a short chain in a wide-lane batch runs the wide-lane kernels). few = 0:
// enough replicas to give every SIMD TUNE_WAVES_PER_SIMD wavefronts of the densest
// packing, so the candidates are ranked by throughput (as in a saturated batch), not by
// the latency of a few wavefronts. It is the same number for all: with four wavefronts
// of its own packing the narrowest tile ran the shortest, and its launch and its last
// wavefronts weighed the most (64 beads, 12500 replicas, noise map 1: M = 4 chosen, 3.79
// ms for 2000 steps, M = 1 2.90). few > 0: that many replicas, those of a batch that
// does not fill the chip, whose kernels and best tiles are others (40 beads, 300
// replicas, 400 steps: the saturated ranking's M = 2 135 us, M = 1 67). Returns ms per
// replica, or -1.
double time_tile(const ra_chain_desc& d, const ra_run_desc& run, int family, int M, int wpb, int few, hipStream_t st) {
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1)
        cus = 256;
    int per_wave = 1;
    for (int m : family_beads_per_lane(family))
        if (legal(d.n_beads, m) && map_allows(run.noise_map, m))
            per_wave = std::max(per_wave, 64 / ((d.n_beads + m - 1) / m));
    ra_chain_desc g = d;
    g.n_replicas = few > 0 ? few : TUNE_WAVES_PER_SIMD * 4 * cus * per_wave;
    // a short list's launch is short: the best of three times as many steps each
    const int steps = few > 0 ? 288 : 96, runs = few > 0 ? 3 : 1;
    ra_run_desc r{};
    r.seed = run.seed;
    r.precision = run.precision;
    r.sample_every = 64;
    r.max_windows = (32 + runs * steps) / 64;
    r.tile_policy = 1000 + M;
    r.waves_per_block = wpb;
    r.noise_map = run.noise_map;
    ra_ctx* ctx = nullptr;
    if (create_context(&ctx, &g, 1, &r, st, family) != RA_OK) return -1.0;
    // straight parent along x; its bonds stay inside the FENE extension
    // (half of Q0 = sqrt(b kT/H), at most 0.5), so the timed kernel does the
    // work of a valid chain
    double bond = 0.5;
    if (d.spring == RA_FENE) bond = std::min(0.5, 0.5 * std::sqrt(d.b * d.kT / d.H));
    std::vector<double> parent(3 * (size_t)d.n_beads, 0.0);
    for (int i = 0; i < d.n_beads; ++i) parent[3 * i] = bond * i;
    double* dp = nullptr;
    double ms = -1.0;
    hipEvent_t e0, e1;
    if (hipMalloc((void**)&dp, parent.size() * sizeof(double)) == hipSuccess &&
        hipMemcpy(dp, parent.data(), parent.size() * sizeof(double), hipMemcpyHostToDevice) == hipSuccess &&
        hipEventCreate(&e0) == hipSuccess) {
        if (hipEventCreate(&e1) == hipSuccess) {
            if (ra_init_chains(ctx, dp) == RA_OK && ra_step(ctx, 32) == RA_OK) {
                for (int i = 0; i < runs; ++i) {
                    (void)hipEventRecord(e0, st);
                    if (ra_step(ctx, steps) != RA_OK) break;
                    (void)hipEventRecord(e1, st);
                    if (hipEventSynchronize(e1) != hipSuccess) break;
                    float t = 0.f;
                    (void)hipEventElapsedTime(&t, e0, e1);
                    const double per = (double)t * 96 / steps / g.n_replicas;
                    ms = ms < 0 ? per : std::min(ms, per);
                }
            }
            (void)hipEventDestroy(e1);
        }
        (void)hipEventDestroy(e0);
    }
    // a timing probe: failures above leave ms < 0 and the candidate unused;
    // an invalid parent would time a kernel that skips its work
    if (ms >= 0 && ra_sync_status(ctx) != RA_OK) ms = -1.0;
    (void)hipStreamSynchronize(st);
    if (dp) (void)hipFree(dp);
    ra_destroy(ctx);
    return ms;
}

}  // namespace

ra_status autotune_tiles(const std::vector<ra_chain_desc>& descs, const ra_run_desc& run, int family,
                         int& waves_per_block, hipStream_t stream, std::vector<int>& Ms, std::string& why) {
    std::lock_guard<std::mutex> lk(g_mu);
    const char* env = std::getenv("RA_AUTOTUNE_CACHE");
    const std::string path = env ? env : "";
    std::map<Key, Entry>& table = table_for(path);
    double best_total = -1.0;
    std::vector<int> best_Ms = Ms;
    int64_t n_items = 0;
    double beads = 0.0;
    for (size_t i = 0; i < descs.size(); ++i) {
        const int P = std::max(1, 64 / ((descs[i].n_beads + Ms[i] - 1) / Ms[i]));
        n_items += (descs[i].n_replicas + P - 1) / P;
        beads += (double)descs[i].n_beads * descs[i].n_replicas;
    }
    const bool few = family == 4 && n_items <= FEW_ITEMS[5];
    const int items = few ? FEW_ITEMS[few_items_class(n_items)] : 0;
    // candidate workgroup sizes: the caller's, or all three when it left the choice open. Most
    // short lists run kernels with a workgroup size of their own: there the default
    // stays unless another one is clearly faster (contexts of a cycle need the same).
    const std::vector<int> wpbs = waves_per_block ? std::vector<int>{waves_per_block}
                                  : few           ? std::vector<int>{4, 1, 2}
                                                  : std::vector<int>{1, 2, 4};
    const double gain = few ? 0.95 : 1.0;
    int best_wpb = waves_per_block ? waves_per_block : 4;
    for (int wpb : wpbs) {
        std::vector<int> Mw(descs.size());
        double total = 0.0;   // predicted batch time: sum over groups of R x time per replica
        for (size_t i = 0; i < descs.size(); ++i) {
            const ra_chain_desc& d = descs[i];
            const Key k{d.n_beads, d.spring, run.precision, family, wpb, run.noise_map, items};
            auto it = table.find(k);
            if (it == table.end())
                it = table.find(Key{d.n_beads, d.spring, run.precision, family, wpb, run.noise_map, ANY_ITEMS});
            if (it == table.end()) {
                Entry best{Ms[i], -1.0};
                double keep = -1.0;   // time of the cost model's tile
                for (int M : family_beads_per_lane(family)) {
                    if (!legal(d.n_beads, M) || !map_allows(run.noise_map, M)) continue;
                    // a short list: as many of these chains as make up the whole batch
                    const int replicas = few ? std::max(d.n_replicas, (int)std::ceil(beads / d.n_beads)) : 0;
                    const double ms = time_tile(d, run, family, M, wpb, replicas, stream);
                    if (ms < 0) { why = "timing run failed"; return RA_EDEVICE; }
                    if (best.ms_per_replica < 0 || ms < best.ms_per_replica) best = Entry{M, ms};
                    if (M == Ms[i]) keep = ms;
                }
                if (!few && keep >= 0 && best.ms_per_replica > TUNE_TILE_GAIN * keep) best = Entry{Ms[i], keep};
                it = table.emplace(k, best).first;
                append_cache_file(path, k, best);
            }
            Mw[i] = it->second.M;
            total += it->second.ms_per_replica * d.n_replicas;
        }
        if (best_total < 0 || total < gain * best_total) {
            best_total = total;
            best_Ms = Mw;
            best_wpb = wpb;
        }
    }
    Ms = best_Ms;
    waves_per_block = best_wpb;
    return RA_OK;
}

}  // namespace ra
