// Host model of the lit kernels' loops with four lanes per ray and their per-wave queue of deferred samples, in
// both forms (test code).
//
// 64 lanes are 16 quads; lane u of a quad takes the samples k = u mod 4 of its ray.  Ballots are masks, and
// every index and decision is the kernels' own (amr_tapq_index.h):
//   loop 0: the single-camera kernel's stepped loop: a step fetches the segments of the quads that wait
//           (stepped_fetch), with checkpoints after the queue has been resolved, or takes four samples of
//           each quad that has a segment, the queue being resolved first by all lanes when it is due;
//   loop 1: the persistent kernel's per-segment loop: the quads still in their segments step together
//           and resolve the queue themselves.
//   list 0: one sample per lane when resolved, due when the samples would overfill it;
//   list 1: one tap per lane, due when the taps would overfill a wave: the samples' tap ranges must be
//           disjoint, inside the list and cover it.
// A sample whose quad mate ended the ray before it, or beyond its segment's end, is not taken.  Every
// queued sample must be resolved exactly once, a run's owners be distinct, and each lane's contributions
// arrive in its sample order.  Input (stdin): loop list ckpt nwaves, then per wave and ray (16): nseg,
// then per segment: n, then n flags (bits 0 to 5: taps pending; bit 6: the ray ends after it).
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "amr_tapq_index.h"

using namespace amr;

#define CHECK(c)                                                                                                 \
    do {                                                                                                         \
        if (!(c)) {                                                                                              \
            std::fprintf(stderr, "violated: %s (line %d, wave %d, step %ld)\n", #c, __LINE__, g_wave, g_step);   \
            std::exit(3);                                                                                        \
        }                                                                                                        \
    } while (0)

static int g_wave = 0;
static long g_step = 0;

struct Ray {
    std::vector<std::vector<int>> segs;
    size_t next = 0;
    int cur = -1, k = 0;
    bool alive = true, has = false;
    long taken = 0;
};

struct Slot {
    int owner = -1, pend = 0;
    uint32_t first = 0;
    long ord = -1;
    bool written = false;
};

struct Wave {
    std::vector<Ray> ray;                  // 16
    Slot slot[kTapQ];
    uint32_t count = 0, taps = 0;
    uint64_t b0 = 0, b1 = 0;
    long ord[64] = {}, added[64] = {};     // per lane: samples queued, contributions added
    long flushes = 0, queued = 0, resolved = 0;
    uint32_t max_count = 0, max_taps = 0;
    bool list = false;

    // the resolving lanes' work (mask act): tap list, samples, contributions
    void flush(uint64_t act) {
        CHECK(act != 0);
        const uint32_t n = count, nact = popc64(act);
        CHECK(n <= (uint32_t)kTapQ);
        flushes++;
        max_count = std::max(max_count, n);
        max_taps = std::max(max_taps, taps);
        auto dealt = [&](uint32_t m) {     // items r, r + nact, ... of the lane of rank r: each once
            std::vector<int> seen(m, 0);
            for (int lane = 0; lane < 64; lane++)
                if ((act >> lane) & 1ull)
                    for (uint32_t j = popc64(act & lanes_below(lane)); j < m; j += nact) seen[j]++;
            for (int v : seen) CHECK(v == 1);
        };
        dealt(n);
        if (list) {
            CHECK(taps <= (uint32_t)kTapList);
            std::vector<int> held(taps, 0);
            for (uint32_t j = 0; j < n; j++) {
                const uint32_t t = popc64((uint64_t)slot[j].pend);
                CHECK(t > 0 && slot[j].first + t <= taps);
                for (uint32_t i = 0; i < t; i++) held[slot[j].first + i]++;
            }
            for (int v : held) CHECK(v == 1);
            dealt(taps);
        }
        uint32_t at = 0;
        for (int w = 0; w < 2; w++) {
            uint64_t bs = w ? b1 : b0;
            while (bs) {
                const uint32_t s = 64u * w + ctz64(bs);
                bs &= bs - 1ull;
                const uint32_t e = tapq_run_end(b0, b1, s, n);
                CHECK(s == at && e > s && e <= n);
                at = e;
                uint64_t owners = 0;
                for (uint32_t j = s; j < e; j++) {
                    Slot &sl = slot[j];
                    CHECK(sl.written && sl.owner >= 0 && sl.owner < 64 && !((owners >> sl.owner) & 1ull));
                    owners |= 1ull << sl.owner;
                    CHECK(sl.ord == added[sl.owner]);
                    added[sl.owner]++;
                    resolved++;
                }
            }
        }
        CHECK(at == n);
        for (Slot &s : slot) s = Slot();
        count = taps = 0;
        b0 = b1 = 0;
    }

    // pending taps of lane's sample in this step; -1: none in its segment
    int sample(int lane) const {
        const Ray &r = ray[lane >> 2];
        const int k = r.k + (lane & 3);
        return k < (int)r.segs[r.cur].size() ? r.segs[r.cur][k] : -1;
    }

    LaneSum sums(const uint32_t (&v)[64], uint64_t act, int lane) const {
        uint64_t m[3] = {0, 0, 0};
        for (int l = 0; l < 64; l++)
            for (int b = 0; b < 3; b++)
                if (((act >> l) & 1ull) && ((v[l] >> b) & 1u)) m[b] |= 1ull << l;
        return lane_sums(m[0], m[1], m[2], lane);
    }

    // the lanes of mask act, whose quads have a segment, take a step; flushers resolve the queue before
    void step(uint64_t act, uint64_t flushers) {
        g_step++;
        uint64_t next = 0;
        uint32_t more[64] = {};
        for (int l = 0; l < 64; l++) {
            if (!((act >> l) & 1ull)) continue;
            const int f = sample(l);
            const uint32_t pend = f < 0 ? 0u : (uint32_t)f & 63u;
            if (pend) next |= 1ull << l;
            more[l] = popc64(pend);
        }
        const bool due = list ? tapq_list_full(taps, sums(more, flushers, 0).all) : tapq_full(count, next);
        if (due) flush(flushers);
        // quad_advance: what each quad takes, and where its ray ends
        uint64_t need = 0;
        uint32_t pending[64] = {};
        for (int q = 0; q < 16; q++) {
            Ray &r = ray[q];
            const uint64_t quad = 0xfull << (4 * q);
            CHECK((act & quad) == 0 || (act & quad) == quad);
            if (!(act & quad)) continue;
            CHECK(r.alive && r.has && r.k < (int)r.segs[r.cur].size());
            bool ended = false;
            for (int u = 0; u < 4; u++) {
                const int f = sample(4 * q + u);
                if (f < 0 || ended) continue;
                r.taken++;
                if (f & 63) {
                    need |= 1ull << (4 * q + u);
                    pending[4 * q + u] = popc64((uint64_t)(f & 63));
                }
                if (f & 64) ended = true;
            }
            for (int u = 0; u < 4; u++)
                if ((need >> (4 * q + u)) & 1ull) queued++;
            if (ended) r.alive = false;
        }
        if (need) {
            const uint32_t c0 = count, t0 = taps;
            for (int l = 0; l < 64; l++) {
                if (!((need >> l) & 1ull)) continue;
                const uint32_t j = tapq_slot(c0, need, l);
                CHECK(j < (uint32_t)kTapQ && !slot[j].written);
                slot[j].written = true;
                slot[j].owner = l;
                slot[j].pend = sample(l) & 63;
                slot[j].first = t0 + sums(pending, act, l).below;
                slot[j].ord = ord[l]++;
            }
            CHECK(c0 < (uint32_t)kTapQ);
            const TapqStarts b = tapq_mark(b0, b1, c0);
            b0 = b.w0;
            b1 = b.w1;
            count = tapq_count_after(c0, need);
            CHECK(count == c0 + popc64(need));
            if (list) taps = t0 + sums(pending, act, 0).all;
        }
        for (int q = 0; q < 16; q++) {
            Ray &r = ray[q];
            if (!((act >> (4 * q)) & 1ull)) continue;
            r.k += 4;
            if (!r.alive || r.k >= (int)r.segs[r.cur].size()) r.has = false;
        }
    }

    uint64_t lanes(bool (*f)(const Ray &)) const {
        uint64_t m = 0;
        for (int q = 0; q < 16; q++)
            if (f(ray[q])) m |= 0xfull << (4 * q);
        return m;
    }

    void stepped(bool ckpt) {
        while (true) {
            const uint64_t live = lanes([](const Ray &r) { return r.alive; });
            if (!live) break;
            const uint64_t waiting = lanes([](const Ray &r) { return r.alive && !r.has; });
            if (stepped_fetch(live, waiting)) {
                CHECK(waiting != 0);
                if (ckpt && count) flush(~0ull);
                for (Ray &r : ray) {
                    if (!r.alive || r.has) continue;
                    if (ckpt) CHECK(count == 0);         // the checkpoint holds every earlier sample
                    while (r.alive && !r.has) {
                        if (r.next >= r.segs.size()) {
                            r.alive = false;
                        } else {
                            r.cur = (int)r.next++;
                            r.k = 0;
                            r.has = !r.segs[r.cur].empty();
                        }
                    }
                }
                continue;
            }
            step(lanes([](const Ray &r) { return r.has; }), ~0ull);
        }
    }

    void per_segment() {
        while (true) {
            bool any = false;
            for (Ray &r : ray) {
                if (!r.alive) continue;
                if (r.next >= r.segs.size()) {
                    r.alive = false;
                    continue;
                }
                r.cur = (int)r.next++;
                r.k = 0;
                r.has = !r.segs[r.cur].empty();
                any = true;
            }
            if (!any) break;
            while (true) {
                const uint64_t act = lanes([](const Ray &r) { return r.alive && r.has; });
                if (!act) break;
                step(act, act);
            }
        }
    }
};

int main() {
    int loop, list, ckpt, nwaves;
    if (std::scanf("%d %d %d %d", &loop, &list, &ckpt, &nwaves) != 4) return 2;
    long samples = 0, queued = 0, flushes = 0;
    uint32_t max_count = 0, max_taps = 0;
    for (g_wave = 0; g_wave < nwaves; g_wave++) {
        Wave w;
        w.list = list != 0;
        w.ray.resize(16);
        std::vector<long> want(16, 0);
        for (int q = 0; q < 16; q++) {
            int nseg;
            if (std::scanf("%d", &nseg) != 1) return 2;
            bool ended = false;
            w.ray[q].segs.resize(nseg);
            for (auto &s : w.ray[q].segs) {
                int n;
                if (std::scanf("%d", &n) != 1) return 2;
                s.resize(n);
                for (int &f : s) {
                    if (std::scanf("%d", &f) != 1) return 2;
                    if (!ended) want[q]++;
                    if (f & 64) ended = true;
                }
            }
        }
        g_step = 0;
        if (loop) w.per_segment();
        else w.stepped(ckpt != 0);
        if (w.count) w.flush(~0ull);
        CHECK(w.count == 0 && w.taps == 0 && w.resolved == w.queued);
        for (int q = 0; q < 16; q++) {
            CHECK(!w.ray[q].alive && w.ray[q].taken == want[q]);
            samples += w.ray[q].taken;
        }
        for (int l = 0; l < 64; l++) CHECK(w.added[l] == w.ord[l]);
        queued += w.queued;
        flushes += w.flushes;
        max_count = std::max(max_count, w.max_count);
        max_taps = std::max(max_taps, w.max_taps);
    }
    std::printf("ok samples=%ld queued=%ld flushes=%ld max_count=%u max_taps=%u\n", samples, queued, flushes, max_count, max_taps);
    return 0;
}
