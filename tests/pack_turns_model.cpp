// Model of the protocol by which the wavefronts of one workgroup of the large-tensor packer share chunks, images and
// places (k_pack_stream in fmtc_coder_kernels.hip), with the rules of fmtc_pack_turns.h.  An agent's step is one access to
// what the others see; between two steps any other agent may take any number of its own, so every combination of delays is
// one order of steps.  No step repeats, so a run ends; what can go wrong is a state in which nobody can go on although
// chunks are left, or a slot that is used again too early.
//
//   pack_turns_model all  WAVES IMAGES TURNS [counter]           every order of steps
//   pack_turns_model walk WAVES IMAGES TURNS RUNS SEED [counter]  random orders, with agents of very different speed
//
// "counter": chunks dealt in plain order, whoever asks (the rule that got stuck).  Prints "ok STATES" or what went wrong.
#include <cmath>
#include <cstddef>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <random>
#include <string>
#include <unordered_set>
#include <vector>

#include "fmtc_pack_turns.h"

using namespace fmtc;

static uint32_t W, IMAGES, TURNS;
static bool counter_rule = false;
static std::string wrong;

constexpr uint32_t kMaxImages = 4;
enum Pc : uint8_t { FIRST, START, TOP, STORE_OR_PACK, ADVANCE, DRAIN, END };

struct Packer {
    uint8_t pc, early, waiting;
    uint32_t n, n_next, own_turn, own, held[kMaxImages];
};
struct Slot {
    uint32_t ticket_of, done, done_of, place_of;  // which turn's ticket / chunks / place the slot holds
};
struct State {
    uint32_t dealt, drawn, published, placed, begun;
    Slot slot[kSlots];
    Packer p[15];
};

static void fail(const char* what, uint32_t turn) {
    if (wrong.empty()) wrong = std::string(what) + ", turn " + std::to_string(turn);
}

static State initial() {
    State s;
    memset(&s, 0, sizeof s);
    for (auto& q : s.slot) q = {~0u, 0u, ~0u, ~0u};
    s.slot[0].ticket_of = 0;
    s.slot[1].ticket_of = 1;
    s.drawn = 2;
    return s;
}

static uint32_t take(State& s, Packer& a) {
    uint32_t n;
    if (counter_rule) {
        n = s.dealt++;
    } else {
        const uint32_t turn = s.dealt >> 8;
        if (a.own_turn == turn + 1 && a.own >= IMAGES) fail("a packer has had its share of both turns", turn);
        if (((s.dealt >> 4) & 15u) >= W) fail("the later turn ran out first", turn);
        const Dealt d = deal(s.dealt, a.own_turn, a.own, IMAGES, W);
        s.dealt = d.state;
        n = d.n;
    }
    const uint32_t turn = n / W;
    a.own = turn == a.own_turn ? a.own + 1 : 1;
    a.own_turn = turn;
    return n;
}

static bool have_group(State& s, uint32_t n) {
    const uint32_t turn = n / W;
    if (s.slot[turn % kSlots].ticket_of != turn) fail("ticket of another turn", turn);
    return turn < TURNS;
}

static void store(State& s, Packer& a) {
    const uint32_t turn = a.held[0] / W;
    const Slot& q = s.slot[turn % kSlots];
    if (q.ticket_of != turn || q.place_of != turn || q.done_of != turn) fail("slot used again before a store", turn);
    for (int i = 1; i < a.waiting; i++) a.held[i - 1] = a.held[i];
    a.held[--a.waiting] = 0;
}

// One step of packer i; false: it cannot go on in this state.
static bool step_packer(State& s, uint32_t i) {
    Packer& a = s.p[i];
    switch (a.pc) {
        case FIRST:  // before the barrier: one chunk of turn 0 each
            a.n = take(s, a);
            a.pc = START;
            s.begun++;
            return true;
        case START:
            if (s.begun < W) return false;
            a.pc = TOP;
            [[fallthrough]];  // (reads the ticket of n, which is known: nobody draws it again)
        case TOP:
            if (!have_group(s, a.n)) {
                a.pc = DRAIN;
                return true;
            }
            a.n_next = take(s, a);
            a.early = s.drawn > a.n_next / W;
            a.pc = STORE_OR_PACK;
            return true;
        case STORE_OR_PACK: {
            const uint32_t oldest = a.held[0] / W;
            if (stores_first(a.waiting, IMAGES, s.placed, oldest)) {
                if (s.placed <= oldest) {
                    if (!counter_rule && oldest >= a.n / W) fail("a packer waits for the turn of its own chunk", oldest);
                    return false;
                }
                store(s, a);
                return true;
            }
            const uint32_t turn = a.n / W;
            Slot& q = s.slot[turn % kSlots];
            if (q.done_of != turn) {
                if (q.done % W != 0) fail("slot used again before its turn was packed", turn);
                q.done_of = turn;
            }
            q.done++;
            a.held[a.waiting++] = a.n;
            a.pc = ADVANCE;
            return true;
        }
        case ADVANCE:
            if (!a.early && s.drawn < a.n_next / W + 1) return false;
            a.n = a.n_next;
            a.pc = TOP;
            return true;
        case DRAIN:
            if (!a.waiting) {
                a.pc = END;
                a.n = a.n_next = a.own = a.own_turn = 0;
                return true;
            }
            if (s.placed <= a.held[0] / W) return false;
            store(s, a);
            return true;
    }
    return false;
}

static bool step_publish(State& s) {
    if (s.published >= TURNS || !may_publish(s.published, s.placed)) return false;
    const Slot& q = s.slot[s.published % kSlots];
    if (q.done_of != s.published || q.done != W * (s.published / kSlots + 1)) return false;
    s.published++;
    const uint32_t next = s.published + 1;
    s.slot[next % kSlots].ticket_of = next;
    s.drawn = s.published + 2;
    return true;
}

static bool step_place(State& s) {  // (a place follows some time after the size)
    if (s.placed >= s.published) return false;
    s.slot[s.placed % kSlots].place_of = s.placed;
    s.placed++;
    return true;
}

static bool step(State& s, uint32_t agent) {
    return agent < W ? step_packer(s, agent) : agent == W ? step_publish(s) : step_place(s);
}

static bool ended(const State& s) {
    for (uint32_t i = 0; i < W; i++)
        if (s.p[i].pc != END) return false;
    return s.placed == TURNS;
}

static int report(const State& s, size_t states) {
    if (!wrong.empty()) {
        printf("%s\n", wrong.c_str());
        return 1;
    }
    (void)s;
    printf("ok %zu\n", states);
    return 0;
}

static int stuck(const State& s) {
    printf("stuck: %u turns published, %u placed, %u drawn\n", s.published, s.placed, s.drawn);
    return 2;
}

static std::string key(const State& s) {
    std::string k(reinterpret_cast<const char*>(&s), offsetof(struct State, p));
    std::vector<std::string> packers;  // (which wavefront is which makes no difference)
    for (uint32_t i = 0; i < W; i++) packers.emplace_back(reinterpret_cast<const char*>(&s.p[i]), sizeof(Packer));
    for (size_t i = 1; i < packers.size(); i++)
        for (size_t j = i; j > 0 && packers[j] < packers[j - 1]; j--) std::swap(packers[j], packers[j - 1]);
    for (auto& q : packers) k += q;
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
        for (uint32_t agent = 0; agent < W + 2; agent++) {
            State t = s;
            if (!step(t, agent)) {
                if (!wrong.empty()) return report(s, seen.size());
                continue;
            }
            if (!wrong.empty()) return report(s, seen.size());
            moved = true;
            if (seen.insert(key(t)).second) todo.push_back(t);
        }
        if (!moved && !ended(s)) return stuck(s);
    }
    return report(initial(), seen.size());
}

static int walk(int runs, uint32_t seed) {
    std::mt19937 rng(seed);
    size_t steps = 0;
    for (int run = 0; run < runs; run++) {
        State s = initial();
        double weight[17];
        auto speeds = [&]() {  // from a few to a thousand times slower than the fastest
            for (uint32_t i = 0; i < W + 2; i++) weight[i] = std::exp2(-(double)(rng() % 11));
        };
        speeds();
        while (!ended(s)) {
            if (rng() % 256 == 0) speeds();
            bool can[17];
            double total = 0;
            State next[17];
            for (uint32_t agent = 0; agent < W + 2; agent++) {
                next[agent] = s;
                can[agent] = step(next[agent], agent);
                if (!wrong.empty()) return report(s, steps);
                if (can[agent]) total += weight[agent];
            }
            if (total == 0) return stuck(s);
            double at = total * (rng() / 4294967296.0);
            uint32_t agent = 0, last = 0;
            for (; agent < W + 2; agent++)
                if (can[agent]) {
                    last = agent;
                    if ((at -= weight[agent]) < 0) break;
                }
            s = next[agent < W + 2 ? agent : last];
            steps++;
        }
    }
    return report(initial(), steps);
}

int main(int argc, char** argv) {
    if (argc < 5) return 3;
    W = (uint32_t)atoi(argv[2]);
    IMAGES = (uint32_t)atoi(argv[3]);
    TURNS = (uint32_t)atoi(argv[4]);
    counter_rule = !strcmp(argv[argc - 1], "counter");
    if (W < 1 || W > 15 || IMAGES < 2 || IMAGES > kMaxImages) return 3;
    if (!strcmp(argv[1], "all")) return all();
    return argc < 7 ? 3 : walk(atoi(argv[5]), (uint32_t)atoi(argv[6]));
}
