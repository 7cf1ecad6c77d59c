// Host emulation of one lane group (flash_group.hpp): each lane is a context of
// its own, and a cross-lane operation is a point where all of them meet.  On the
// device the lanes hold a mixture's scalars equal up to the last bit only (a
// product that is summed is fused into the first addition of the reduction); here
// the odd lanes' first partner value is moved by one unit in the last place.  The
// lanes of a group must meet at the same operations all the same and end their
// items at the same step: one that goes its own way leaves the others waiting for
// values, and the stage's loop for an item that nobody holds.
// Prints: items run, steps, decisions, decisions on which the lanes' own answers
// differed, items whose lanes parted.
#include <ucontext.h>

#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <random>
#include <vector>

static double __shfl_xor(double v, int o, int);
static double __shfl(double v, int lane, int);
static unsigned long long __ballot(bool c);
static void lane_meet();
#define __builtin_amdgcn_fence(order, scope) ((void)0)
#define __builtin_amdgcn_wave_barrier() lane_meet()

#include "flash_group.hpp"

using namespace ptf;

constexpr int NC = HOST_NC, G = NC <= 16 ? 16 : 32;
enum Op { kNone, kMeet, kXor, kRead, kBallot, kStep, kEnd };

struct Lane {
    ucontext_t ctx;
    std::vector<char> stack;
    Op op;
    int arg;
    double v;
    bool c;
    unsigned long long mask;
};
static Lane lanes[G];
static ucontext_t host;
static int cur;
static long decisions, mixed;

static void meet(Op op)
{
    lanes[cur].op = op;
    const int me = cur;
    swapcontext(&lanes[me].ctx, &host);
}
static void lane_meet() { meet(kMeet); }
static double __shfl_xor(double v, int o, int)
{
    lanes[cur].v = v;
    lanes[cur].arg = o;
    meet(kXor);
    const double w = lanes[cur].v;
    return o == 1 && (cur & 1) && std::isfinite(w) && w != 0.0 ? std::nextafter(w, INFINITY) : w;
}
static double __shfl(double v, int lane, int)
{
    lanes[cur].v = v;
    lanes[cur].arg = lane;
    meet(kRead);
    return lanes[cur].v;
}
static unsigned long long __ballot(bool c)
{
    lanes[cur].c = c;
    meet(kBallot);
    return lanes[cur].mask;
}

static void (*body)();
static void entry() { body(); meet(kEnd); }

// Runs body on every lane; false when the lanes part.
static bool run_lanes()
{
    for (int i = 0; i < G; ++i) {
        Lane &l = lanes[i];
        l.stack.resize(256 << 10);
        getcontext(&l.ctx);
        l.ctx.uc_stack.ss_sp = l.stack.data();
        l.ctx.uc_stack.ss_size = l.stack.size();
        l.ctx.uc_link = &host;
        makecontext(&l.ctx, entry, 0);
    }
    for (;;) {
        for (cur = 0; cur < G; ++cur) swapcontext(&host, &lanes[cur].ctx);
        for (int i = 1; i < G; ++i)
            if (lanes[i].op != lanes[0].op ||
                ((lanes[0].op == kXor || lanes[0].op == kRead) && lanes[i].arg != lanes[0].arg))
                return false;
        double v[G];
        unsigned long long mask = 0;
        for (int i = 0; i < G; ++i) {
            v[i] = lanes[i].v;
            mask |= (unsigned long long)lanes[i].c << i;
        }
        switch (lanes[0].op) {
        case kEnd: return true;
        case kXor:
            for (int i = 0; i < G; ++i) lanes[i].v = v[i ^ lanes[i].arg];
            break;
        case kRead:
            for (int i = 0; i < G; ++i) lanes[i].v = v[lanes[i].arg % G];
            break;
        case kBallot:
            ++decisions;
            mixed += mask != 0 && mask != (G == 64 ? ~0ull : (1ull << G) - 1);
            for (int i = 0; i < G; ++i) lanes[i].mask = mask;
            break;
        default: break;
        }
    }
}

static Ctx<NC> ctx;
static std::vector<double> lds, table;
static uint32_t item_id;
static long items, steps, parted;
static Outbox last;

template <class Item>
static void lane_body()
{
    Grp<NC, G> g;
    g.gi = cur;
    g.base = 0;
    g.act = cur < NC;
    g.row = g.act ? cur : NC;
    g.sh = lds.data();
    g.vb = g.sh + (Item::kMatrix ? GroupLds<NC, G>::V : 0);
    g.ks = table.data();
    Item it;
    bool live = it.begin(ctx, item_id, g);
    while (live) {
        if constexpr (Item::OUT != 0u) it.ob.clear();
        live = !it.step(ctx, g);
        if (cur == 0) ++steps;
        meet(kStep);
    }
    if constexpr (Item::OUT != 0u) {
        if (cur == 0) last = it.ob;
    }
}

template <class Item>
static bool run_group(uint32_t id)
{
    item_id = id;
    last.clear();
    body = lane_body<Item>;
    ++items;
    if (run_lanes()) return true;
    ++parted;
    return false;
}

template <class Item>
static bool run_item(uint32_t id, Outbox &o)
{
    Item it;
    o.clear();
    if (!it.begin(ctx, id)) return false;
    do it.ob.clear();
    while (!it.step(ctx));
    o = it.ob;
    return true;
}

int main(int, char **argv)
{
    const int n = atoi(argv[1]);
    const double tol = atof(argv[2]);
    std::mt19937_64 rng(4711 + NC);
    auto uni = [&](double a, double b) { return std::uniform_real_distribution<double>(a, b)(rng); };
    std::vector<double> Tc(NC), Pc(NC), om(NC), K(NC * NC), z(n * NC), T(n), P(n);
    for (int i = 0; i < NC; ++i) {
        Tc[i] = uni(190, 620);
        Pc[i] = uni(2e6, 5e6);
        om[i] = uni(0.01, 0.5);
        for (int j = 0; j < i; ++j) K[i * NC + j] = K[j * NC + i] = uni(0, 0.15);
    }
    for (auto &v : z) v = std::gamma_distribution<double>(0.5, 1.0)(rng) + 1e-30;
    for (auto &v : T) v = uni(200, 600);
    for (auto &v : P) v = uni(1e5, 2e7);
    std::vector<int8_t> label(n), hint(n);
    std::vector<double> beta(n), x(n * NC), y(n * NC);
    std::vector<MixRec<NC>> rec(n);
    for (int i = 0; i < n; ++i) hint[i] = i % 3 == 0 ? 1 : -1;   // a third starts as a split
    std::memset((void *)&ctx, 0, sizeof(ctx));
    FlashArgs &a = ctx.a;
    a.n = n;
    a.z = z.data();
    a.T = T.data();
    a.P = P.data();
    a.hint = hint.data();
    a.max_pre_ss = 3;
    a.max_ss = tol < 1e-12 ? 30 : 9;
    a.max_tr_sa = 20;
    a.max_tr_split = 30;
    a.max_polish = 5;
    a.dem_every = 3;
    a.tol_sa_ss = a.tol_sa_tr = a.tol_split_ss = a.tol_split_tr = tol;
    a.tol_polish = 1e-13;
    a.eps_tm = 1e-10;
    a.label = label.data();
    a.beta = beta.data();
    a.x = x.data();
    a.y = y.data();
    ctx.pr = Props{Tc.data(), Pc.data(), om.data(), K.data()};
    ctx.rec = rec.data();
    lds.assign(GroupLds<NC, G>::N, 0.0);
    const int ks = KapLds::stride<NC>();
    table.assign(NC * ks, 0.0);
    for (int i = 0; i < NC * NC; ++i) table[(i / NC) * ks + i % NC] = 1.0 - K[i];
    for (uint32_t m = 0; m < (uint32_t)n; ++m) {
        Outbox o;
        if (!run_item<FeedItem<NC, false>>(m, o)) continue;
        if (o.l0 == L_PRE) run_item<PreSsItem<NC, false>>(m, o);
        if (o.l0 == L_SA) {
            bool ok = true;
            for (uint32_t t = 0; t < 2 && ok; ++t) {
                ok = run_group<SaSsGroup<NC, false, G>>(2 * m + t);
                if (ok && last.l0 == L_SATR) ok = run_group<SaTrGroup<NC, false, G>>(2 * m + t);
            }
            if (!ok) continue;
            run_item<SaFinItem<NC, false>>(m, o);
        }
        if (o.l0 != L_SPLIT || !run_group<SpSsGroup<NC, false, G>>(m)) continue;
        if (last.l0 == L_NT || last.l0 == L_NTP) run_group<SpNtGroup<NC, false, G>>(m);
    }
    printf("%ld %ld %ld %ld %ld\n", items, steps, decisions, mixed, parted);
    return 0;
}
