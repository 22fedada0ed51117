// Model of the protocol by which the workgroups of the large-tensor packer (k_pack_stream in fmtc_coder_kernels.hip) share a
// tensor's ranges, with the rules of fmtc_pack_ranges.h.  A workgroup's step is one access to what the others see; between
// two steps any other workgroup may take any number of its own, and a place on the device that one leaves may be taken by any
// that has not started.  No step repeats, so a run ends; what can go wrong is a state in which nobody can go on although
// ranges are left, a range that is stored before all sizes before it are known, or a chunk that is packed twice or never.
//
//   pack_ranges_model all  CHUNKS GRID IMAGES RESIDENT [index]             every order of steps
//   pack_ranges_model walk CHUNKS GRID IMAGES RESIDENT RUNS SEED [index]   random orders, with workgroups of very different speed
//   pack_ranges_model cut                                                   the rules over many sizes
//
// "index": ranges by the workgroup's index instead of a ticket (a rule that gets stuck).  Prints "ok ..." or what went wrong.
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <random>
#include <string>
#include <unordered_set>
#include <vector>

#include "fmtc_pack_ranges.h"

using namespace fmtc;

static uint32_t N, GRID, IMAGES, RESIDENT;
static bool by_index = false;
static Ranges R;
static std::string wrong;

enum Pc : uint8_t { WAITING, CLAIM, CLAIM_NEXT, PUBLISH, LOOK, STORE, END };
struct Group {
    uint8_t pc;
    uint16_t range, next;
};
struct State {
    uint32_t ticket, running;
    std::vector<Group> g;
    std::vector<uint8_t> size, stored;
};

static void fail(const char* what, uint32_t range) {
    if (wrong.empty()) wrong = std::string(what) + ", range " + std::to_string(range);
}
static State initial() { return {0, 0, std::vector<Group>(GRID, Group{WAITING, 0, 0}), std::vector<uint8_t>(R.count, 0), std::vector<uint8_t>(R.count, 0)}; }
static uint16_t claim(State& s, uint32_t i, bool first) {
    if (by_index) return (uint16_t)(first ? i : s.g[i].range + GRID);
    return (uint16_t)s.ticket++;
}

// One step of workgroup i; false: it cannot go on in this state.
static bool step(State& s, uint32_t i) {
    Group& a = s.g[i];
    switch (a.pc) {
        case WAITING:
            if (s.running >= RESIDENT) return false;
            s.running++;
            a.pc = CLAIM;
            return true;
        case CLAIM:
            a.range = claim(s, i, true);
            a.pc = a.range < R.count ? CLAIM_NEXT : END;
            if (a.pc == END) s.running--;
            return true;
        case CLAIM_NEXT:
            a.next = claims_another(R, GRID) ? claim(s, i, false) : (uint16_t)R.count;
            a.pc = PUBLISH;
            return true;
        case PUBLISH:  // (packed by now)
            if (s.size[a.range]) fail("packed twice", a.range);
            s.size[a.range] = 1;
            a.pc = LOOK;
            return true;
        case LOOK:
            for (uint32_t r = 0; r < a.range; r++)
                if (!s.size[r]) return false;
            a.pc = STORE;
            return true;
        case STORE:
            for (uint32_t r = 0; r < a.range; r++)
                if (!s.size[r]) fail("stored without the sizes before it", a.range);
            s.stored[a.range] = 1;
            a.range = a.next;
            a.pc = a.range < R.count ? CLAIM_NEXT : END;
            if (a.pc == END) s.running--;
            return true;
    }
    return false;
}

static bool ended(const State& s) {
    for (auto& a : s.g)
        if (a.pc != END) return false;
    for (uint32_t r = 0; r < R.count; r++)
        if (!s.stored[r]) fail("never stored", r);
    return true;
}
static int report(size_t steps) {
    printf("%s %zu\n", wrong.empty() ? "ok" : wrong.c_str(), steps);
    return wrong.empty() ? 0 : 1;
}
static int stuck(const State& s) {
    uint32_t n = 0;
    for (uint8_t v : s.size) n += v;
    printf("stuck: %u of %u sizes published, %u workgroups running\n", n, R.count, s.running);
    return 2;
}

static std::string key(const State& s) {
    std::string k(reinterpret_cast<const char*>(&s.ticket), 4);
    std::vector<std::string> groups;
    for (auto& a : s.g) groups.push_back({(char)a.pc, (char)a.range, (char)a.next});
    if (!by_index)  // (which workgroup is which makes no difference)
        for (size_t i = 1; i < groups.size(); i++)
            for (size_t j = i; j > 0 && groups[j] < groups[j - 1]; j--) std::swap(groups[j], groups[j - 1]);
    for (auto& q : groups) k += q;
    k.append(s.size.begin(), s.size.end());
    k.append(s.stored.begin(), s.stored.end());
    return k;
}

static int all() {
    std::unordered_set<std::string> seen;
    std::vector<State> todo{initial()};
    seen.insert(key(todo[0]));
    while (!todo.empty()) {
        const State s = todo.back();
        todo.pop_back();
        bool moved = false;
        for (uint32_t i = 0; i < GRID; i++) {
            State t = s;
            if (!step(t, i)) continue;
            if (!wrong.empty()) return report(seen.size());
            moved = true;
            if (seen.insert(key(t)).second) todo.push_back(t);
        }
        if (!moved && !ended(s)) return stuck(s);
        if (!wrong.empty()) return report(seen.size());
    }
    return report(seen.size());
}

static int walk(int runs, uint32_t seed) {
    std::mt19937 rng(seed);
    size_t steps = 0;
    for (int run = 0; run < runs; run++) {
        State s = initial();
        std::vector<double> weight(GRID);
        std::vector<uint32_t> can;
        while (!ended(s)) {
            if (rng() % 512 == 0 || weight[0] == 0.0)
                for (auto& w : weight) w = std::exp2(-(double)(rng() % 11));  // up to a thousand times slower than the fastest
            double total = 0;
            can.clear();
            for (uint32_t i = 0; i < GRID; i++) {
                // (a copy would cost more than a look: the only steps that cannot be taken are a start and a look)
                const Group& a = s.g[i];
                bool ok = a.pc != END && (a.pc != WAITING || s.running < RESIDENT);
                if (a.pc == LOOK)
                    for (uint32_t r = 0; ok && r < a.range; r++) ok = s.size[r];
                if (ok) {
                    can.push_back(i);
                    total += weight[i];
                }
            }
            if (can.empty()) return stuck(s);
            double at = total * (rng() / 4294967296.0);
            uint32_t pick = can.back();
            for (uint32_t i : can)
                if ((at -= weight[i]) < 0) {
                    pick = i;
                    break;
                }
            step(s, pick);
            steps++;
            if (!wrong.empty()) return report(steps);
        }
        if (!wrong.empty()) return report(steps);
    }
    return report(steps);
}

// Every chunk in one range, no range larger than the images, and no more ranges than groups of four chunks (which have a
// word each for their sizes), for every tensor that the kernel is launched for on a device that holds `places` small workgroups.
static int cut() {
    size_t cases = 0;
    for (uint32_t places : {64u, 128u, 512u, 1024u})
        for (uint32_t images : {32u, 48u, 64u})
            for (uint32_t step = 0; step < 1560; step++) {
                // (every size from the first one on, then sizes up to the 2^26 chunks of a tensor of 2^32 symbols)
                const uint32_t n = 4u * places + 1u + (step < 1500u ? step : (step - 1500u) * (step - 1500u) * 18000u), groups = (n + 3u) / 4u;
                const uint32_t grid = groups < 256u ? groups : 256u;
                const Ranges r = cut_ranges(n, grid, images);
                uint32_t next = 0;
                for (uint32_t q = 0; q < r.count; q++) {
                    const ChunkSpan c = range_chunks(r, q, n);
                    if (c.first != next || c.count < 1u || c.count > images || (q + 1u < r.count && c.count != r.chunks)) fail("chunks of a range", q);
                    next = c.first + c.count;
                }
                if (next != n || range_chunks(r, r.count, n).count != 0u || range_chunks(r, r.count + 300u, n).count != 0u) fail("chunks left", n);
                if (r.count > groups) fail("more ranges than words for their sizes", n);
                if (claims_another(r, grid) != (r.count > grid)) fail("claims", n);
                if (!wrong.empty()) {
                    printf("%u chunks, grid %u, %u images: ", n, grid, images);
                    return report(cases);
                }
                cases++;
            }
    return report(cases);
}

int main(int argc, char** argv) {
    if (argc == 2 && !strcmp(argv[1], "cut")) return cut();
    if (argc < 6) return 3;
    N = (uint32_t)atoi(argv[2]);
    GRID = (uint32_t)atoi(argv[3]);
    IMAGES = (uint32_t)atoi(argv[4]);
    RESIDENT = (uint32_t)atoi(argv[5]);
    by_index = !strcmp(argv[argc - 1], "index");
    if (N < 1 || GRID < 1 || IMAGES < 1 || RESIDENT < 1) return 3;
    R = cut_ranges(N, GRID, IMAGES);
    if (R.count + GRID > 60000) return 3;
    if (!strcmp(argv[1], "all")) return R.count + GRID < 100 ? all() : 3;
    return argc < 8 ? 3 : walk(atoi(argv[6]), (uint32_t)atoi(argv[7]));
}
