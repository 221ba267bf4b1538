// Layer loop of the hash-bucket engine (buckets.hip): breadth-first search
// by layers for generating sets closed under inverses (paper, section
// "Reminder on Cayley graphs, diameters, growth", definition of Growth).
//
// Small layers run many to a launch in one workgroup; larger ones take one
// partition (or two) and one bucket kernel each, with one read-back of the
// layer's size. Layers stay in bucket order; a layer is sorted only when the
// caller reads its states back, or when the sort path takes over (device
// memory too short for the partitions, or a partition that overruns).
#include <algorithm>
#include <cstdlib>
#include <cstring>

#include "bitmap.h"
#include "engine.h"

namespace cg {

namespace {

// Room of a run of small layers (states).
constexpr uint64_t kSmallRun = 1u << 18;

bool is_nomem(const Error &e) { return e.code == CG_E_NOMEM; }

// Most candidates a layer may have to go by hash buckets; beyond it the sort
// path takes over (CG_HASH_CANDIDATES; no limit by default).
uint64_t hash_candidates_max() {
    const char *e = std::getenv("CG_HASH_CANDIDATES");
    return e ? std::strtoull(e, nullptr, 10) : ~0ull;
}

// Growth of layers expected from one step to the next.
constexpr double kExpectSlack = 1.15;

}  // namespace

// Sets closed under inverses (two reference layers are enough), unless the
// caller asks for packed sorting or an environment tunable of the sort path
// is set. Permutations of up to 12 entries go over a rank bitmap instead, or
// by sorting where memory is too short for that (S_12 pancake: 97 ms by
// buckets of 64-bit keys, 76 by sorting 32-bit ranks, 28 over the bitmap).
// Against the sort: S_16 LRX to 2^29 states 90 ms for 184, a multiset coset of
// n = 14 9.1 for 28.6, binary LRX cosets of n = 32 44 for 82.
bool hash_layers(const JobSpec &spec) {
    if (spec.k == 0 || !spec.inverse_closed || (spec.flags & (CG_PACKED_SORT | CG_BITMASK | CG_SMALL_JOB))) return false;
    if (std::getenv("CG_CHUNK_CANDIDATES") || std::getenv("CG_RANK_FULL")) return false;
    return spec.binary || spec.n > 12 || !start_is_permutation(spec);
}

// Partitions and their counts at every frontier size up to the largest (the
// parts of small layers keep proportionally more room), three layers and
// their bucket tables, the runs of small layers.
uint64_t hash_layers_bytes(const JobSpec &spec) {
    const uint64_t orbit = spec.orbit_bound, k = (uint64_t)std::max(1, spec.k);
    const uint64_t fmax = spec.max_frontier ? std::min(orbit, spec.max_frontier) : orbit;
    const uint64_t layer = std::min(orbit, k * fmax);
    uint64_t parts = 0, tab = 0;
    for (uint64_t F = fmax; F; F /= 2)
        for (uint64_t states : {F, 2 * F + std::min(orbit, k * F)}) {
            HashPlan p;
            if (!hash_plan(F, (uint32_t)k, states, &p)) continue;
            parts = std::max(parts, p.bytes1() + p.bytes2() + 4 * (p.counts1() + p.counts2()));
            tab = std::max<uint64_t>(tab, 8ull << p.lg_q());
        }
    const double layers = 3.0 * 8.0 * kExpectSlack * (double)layer;
    return (uint64_t)(1.25 * ((double)parts + layers + 3.0 * (double)tab)) + (64ull << 20);
}

// The tags of a growth, where it can have them. (Layers that stay resident
// hold whole keys.)
HashTags make_tags(const JobSpec &spec) {
    HashTags t;
    const int n = spec.n, k = spec.k;
    const int left = 64 - (spec.binary ? n : 4 * n);
    const bool implied = !spec.binary && n >= 9 && k > left;  // entry 0 (its bits are in the high word)
    const int width = std::min({k, implied ? left + 4 : left, (int)kHashMaxTags});
    if (k < 2 || k > (int)kHashMaxTags || 2 * width < k || (spec.flags & CG_KEEP_ALL_LAYERS)) return t;
    for (int g = 0; g < k; ++g) {
        const uint8_t *a = spec.gens.data() + (size_t)g * n;
        int undo = -1;
        for (int h = 0; h < k && undo < 0; ++h) {
            const uint8_t *b = spec.gens.data() + (size_t)h * n;
            bool id = true;
            for (int i = 0; i < n && id; ++i) id = a[b[i]] == i;
            if (id) undo = h;
        }
        if (undo < 0) return HashTags();  // never, in a set closed under inverses
        if (undo < width) t.undo[g] = 1u << (32 - width + undo);
    }
    t.all = width == k;
    t.shift = (uint32_t)(32 - width);
    t.mask_hi = (1u << t.shift) - 1u;
    if (implied) {
        t.place = (uint32_t)(4 * (n - 1) - 32);
        t.mask_hi = (1u << t.place) - 1u;
        for (int i = 0; i < n; ++i) t.sum += spec.start[i];
        t.sum = 16u + t.sum % 16u;
    }
    return t;
}

// keys[0..n) sorted, there or in tmp.
uint64_t *Engine::sort_keys(const JobSpec &spec, uint64_t *keys, uint64_t *tmp, uint64_t n) {
    if (!w_.ready()) w_.init(stream_);
    sorted_ = true;
    return radix_sort(keys, tmp, n, spec.binary ? 0 : 4, spec.binary ? spec.n : 4 * spec.n, w_, spec.binary);
}

// keys[0..n) sorted, whole keys, in a or b (each n keys); keys is left as it is.
uint64_t *Engine::sorted_copy(const JobSpec &spec, const uint64_t *keys, uint64_t n, DevBuf &a, DevBuf &b) {
    a.ensure(std::max<uint64_t>(n, 1) * 8);
    b.ensure(std::max<uint64_t>(n, 1) * 8);
    if (tags_.on())
        launch_hash_strip(a.as<uint64_t>(), keys, n, tags_, stream_);
    else
        CG_HIP(hipMemcpyAsync(a.p, keys, n * 8, hipMemcpyDeviceToDevice, stream_));
    return sort_keys(spec, a.as<uint64_t>(), b.as<uint64_t>(), n);
}

// Layers d-1 and d sorted, as whole keys, each in a buffer of its own (the
// layers that stay resident: in their place). Sorted where they lie, with
// one more copy of one layer at a time, after all else is freed: memory is
// short when this runs.
void Engine::hand_to_sort(const JobSpec &spec, const HashLayer &prev, const HashLayer &cur, const Progress &p) {
    CG_HIP(hipStreamSynchronize(stream_));
    for (DevBuf *x : {&part_[0], &part_[1], &part_cnt_[0], &part_cnt_[1], &order_[0], &order_[1], &tab_[0], &tab_[1],
                      &tab_[2]})
        x->release();
    const bool keep_all = (spec.flags & CG_KEEP_ALL_LAYERS) != 0;
    DevBuf own[2], tmp;
    for (DevBuf *x : {&own[0], &own[1], &tmp}) adopt(*x);
    for (int i = 0; i < 2 && !keep_all; ++i) {
        const HashLayer &l = i ? cur : prev;
        for (DevBuf &x : lay_)
            if (l.n && x.p == l.keys) own[i].swap(x);
        if (own[i].p) continue;
        own[i].ensure(std::max<uint64_t>(l.n * 8, 64));  // (one of a run of small layers, or none)
        if (l.n) CG_HIP(hipMemcpyAsync(own[i].p, l.keys, l.n * 8, hipMemcpyDeviceToDevice, stream_));
    }
    for (DevBuf *x : {&small_[0], &small_[1], &small_[2], &lay_[0], &lay_[1], &lay_[2]}) x->release();
    for (int i = 0; i < 2; ++i) {
        const HashLayer &l = i ? cur : prev;
        if (!l.n) continue;
        uint64_t *at = keep_all ? arena_.as<uint64_t>() + p.off[p.off.size() - 3 + i] : own[i].as<uint64_t>();
        if (tags_.on()) launch_hash_strip(at, at, l.n, tags_, stream_);
        tmp.release();  // (it would grow with slack)
        tmp.ensure(l.n * 8);
        uint64_t *r = sort_keys(spec, at, tmp.as<uint64_t>(), l.n);
        uint64_t *to = keep_all ? at : tmp.as<uint64_t>();  // (the layer's own buffer may be far larger)
        if (r != to) CG_HIP(hipMemcpyAsync(to, r, l.n * 8, hipMemcpyDeviceToDevice, stream_));
        if (!keep_all) own[i].swap(tmp);
    }
    CG_HIP(hipStreamSynchronize(stream_));
    tmp.release();
    if (keep_all) return;
    for (int i = 0; i < 2; ++i) lay_[i].swap(own[i]);
    // The sort path's chunks take the largest free block: a layer that lies
    // between two moves where a smaller one holds it.
    for (int pass = 0; pass < 2; ++pass)
        for (int i = 0; i < 2; ++i) {
            const size_t bytes = lay_[i].bytes, largest = device_bytes_available();
            if (bytes < (1u << 30)) continue;
            DevBuf moved;
            adopt(moved);
            try {
                moved.ensure(bytes);
            } catch (const Error &e) {
                if (!is_nomem(e)) throw;
                continue;
            }
            if (moved.in_arena && device_bytes_available() == largest) {
                CG_HIP(hipMemcpyAsync(moved.p, lay_[i].p, bytes, hipMemcpyDeviceToDevice, stream_));
                CG_HIP(hipStreamSynchronize(stream_));
                lay_[i].swap(moved);
            }
            moved.release();
        }
}

bool Engine::run_hashed(const JobSpec &spec, cg_result_t *res, uint64_t key0, Progress &p) {
    const int n = spec.n;
    const uint32_t k = (uint32_t)spec.k;
    const bool keep_all = (spec.flags & CG_KEEP_ALL_LAYERS) != 0;
    uint64_t *sizes = res->layer_sizes;

    // One upload: the start key, then the generators.
    std::vector<uint8_t> up(64);
    std::memcpy(up.data(), &key0, 8);
    auto append = [&](const void *x, size_t bytes) {
        const size_t at = up.size();
        up.resize(at + (bytes + 63) / 64 * 64);
        std::memcpy(up.data() + at, x, bytes);
        return at;
    };
    size_t at_sel = 0, at_term = 0, at_first = 0;
    if (spec.binary) {
        std::vector<BitTerm> terms;
        std::vector<uint32_t> first;
        make_bit_terms(n, spec.gens.data(), spec.k, terms, first);
        at_term = append(terms.data(), terms.size() * sizeof(BitTerm));
        at_first = append(first.data(), first.size() * sizeof(uint32_t));
    } else {
        std::vector<GenSel> sel(k);
        for (uint32_t g = 0; g < k; ++g) sel[g] = make_gensel(n, spec.gens.data() + (size_t)g * n);
        at_sel = append(sel.data(), sel.size() * sizeof(GenSel));
    }
    gsel_.ensure(up.size());
    const void *up_from = up.data();
    if (up.size() <= kHostSmallBytes) {
        std::memcpy(host_small_, up.data(), up.size());
        up_from = host_small_;
    }
    CG_HIP(hipMemcpyAsync(gsel_.p, up_from, up.size(), hipMemcpyHostToDevice, stream_));
    HashGens gens;
    gens.binary = spec.binary;
    gens.k = k;
    gens.sel = reinterpret_cast<const GenSel *>(gsel_.as<uint8_t>() + at_sel);
    gens.term = reinterpret_cast<const BitTerm *>(gsel_.as<uint8_t>() + at_term);
    gens.first = reinterpret_cast<const uint32_t *>(gsel_.as<uint8_t>() + at_first);
    tags_ = make_tags(spec);

    // two sets of counters: a step clears the other one's
    hctr_.ensure(2 * kHashCounterStride * 8);
    launch_clear(nullptr, 0, hctr_.as<uint64_t>(), 2 * kHashCounterStride, stream_);
    uint32_t set = 0;
    // small-layer results: two words of state, then the sizes
    ssz_.ensure(8 + kSmallMaxLayers * 8);
    static_assert(8 + kSmallMaxLayers * 8 <= kHostSmallBytes, "small-layer results fit the pinned buffer");

    HashLayer prev, cur;
    cur.keys = gsel_.as<uint64_t>();
    cur.n = 1;
    if (keep_all) {
        // the whole orbit when it fits comfortably, else grow on demand
        size_t free_b = 0, total_b = 0;
        CG_HIP(hipMemGetInfo(&free_b, &total_b));
        uint64_t first = std::min<uint64_t>(spec.orbit_bound, 1ull << 20);
        if (spec.orbit_bound <= (uint64_t)(free_b / 4 / sizeof(uint64_t))) first = spec.orbit_bound;
        arena_.ensure(first * 8);
        CG_HIP(hipMemcpyAsync(arena_.p, gsel_.p, 8, hipMemcpyDeviceToDevice, stream_));
        cur.keys = arena_.as<uint64_t>();
        p.off = {0, 1};
    }
    if (spec.layers_out) {
        if (spec.layers_out_cap) std::memcpy(spec.layers_out, spec.start, (size_t)n);
        p.written = 1;
    }
    // keep_all: room for `more` states behind the recorded ones (the arena
    // may move: the layers' addresses are taken afresh)
    auto arena_room = [&](uint64_t more) {
        const uint64_t need = (p.total + more) * 8;
        if (need <= arena_.bytes) return;
        size_t want = std::max<size_t>(need, (size_t)(arena_.bytes * 1.5));
        want = std::min<size_t>(want, std::max<size_t>(need, spec.orbit_bound * 8));
        DevBuf bigger;
        adopt(bigger);
        bigger.ensure(want);
        CG_HIP(hipMemcpyAsync(bigger.p, arena_.p, p.total * 8, hipMemcpyDeviceToDevice, stream_));
        CG_HIP(hipStreamSynchronize(stream_));
        arena_.swap(bigger);
        cur.keys = arena_.as<uint64_t>() + p.off[p.off.size() - 2];
        if (prev.n) prev.keys = arena_.as<uint64_t>() + p.off[p.off.size() - 3];
    };
    int lay_at = 0, tab_at = 0;    // lay_[lay_at], tab_[tab_at] take the next layer
    const uint64_t most_candidates = hash_candidates_max();
    uint64_t states_try = 0;       // larger table estimate of a layer that is done again
    bool small_ok = true;          // false: the next layer did not fit one workgroup
    for (;;) {
        if (spec.max_frontier && p.F > spec.max_frontier) {
            p.status = CG_TRUNCATED;
            return true;
        }
        if (p.layers >= spec.max_layers) {
            p.status = CG_TRUNCATED;
            return true;
        }
        const uint64_t C = p.F * (uint64_t)k;
        const uint64_t room = spec.orbit_bound > p.total ? spec.orbit_bound - p.total : 0;

        if (small_ok && C <= most_candidates && p.np + p.F <= kSmallStates && C <= kSmallMaxCand) {
            HashSmallArgs a{};
            a.prev = prev.keys;
            a.cur = cur.keys;
            a.np = (uint32_t)p.np;
            a.nc = (uint32_t)p.F;
            a.k = k;
            const uint64_t left = (uint64_t)(spec.max_layers - p.layers);
            a.max_new = (uint32_t)std::min<uint64_t>(left, kSmallMaxLayers - 1);
            a.max_new_is_rule = a.max_new == left;
            a.max_frontier = spec.max_frontier;
            uint64_t *out;
            if (keep_all) {
                // the kernel wants room for a whole table of states, also
                // where the orbit has fewer left; where memory has not, the
                // layer takes a step of its own, which wants less
                try {
                    arena_room(std::max<uint64_t>(kSmallStates, std::min<uint64_t>(room, kSmallRun)));
                } catch (const Error &e) {
                    if (!is_nomem(e)) throw;
                    small_ok = false;
                    continue;
                }
                a.prev = prev.keys;
                a.cur = cur.keys;
                out = arena_.as<uint64_t>() + p.total;
                a.out_cap = arena_.bytes / 8 - p.total;
            } else {
                // a buffer that holds neither layer d-1 nor layer d
                DevBuf *b = nullptr;
                for (DevBuf &x : small_)
                    if (!x.holds(prev.keys) && !x.holds(cur.keys)) b = &x;
                b->ensure((kSmallRun + kSmallStates) * 8);
                out = b->as<uint64_t>();
                a.out_cap = kSmallRun + kSmallStates;
            }
            a.out = out;
            a.state = ssz_.as<uint32_t>();
            a.sizes = ssz_.as<uint64_t>() + 1;
            launch_hash_small(a, gens, tags_, w_);
            CG_HIP(hipMemcpyAsync(host_small_, ssz_.p, 8 + kSmallMaxLayers * 8, hipMemcpyDeviceToHost, stream_));
            CG_HIP(hipStreamSynchronize(stream_));
            if (prof_.on) prof_.collect();
            const uint32_t made = ((const uint32_t *)host_small_)[0], code = ((const uint32_t *)host_small_)[1];
            const uint64_t *hs = host_small_ + 1;
            if (made > a.max_new) throw Error(CG_E_DEVICE, "small-layer count out of range (device error)");
            uint64_t used = 0;
            uint32_t filled = 0;
            for (uint32_t i = 0; i < made; ++i) {
                res->states_expanded += p.F;
                res->candidates += p.F * (uint64_t)k;
                const uint64_t N = hs[i];
                if (N > kSmallStates || p.total + N > spec.orbit_bound)
                    throw Error(CG_E_DEVICE, "layer size out of range (device error)");
                if (!N) break;
                prev = cur;
                cur = HashLayer{out + used, N, nullptr, 0, false};
                used += N;
                ++filled;
                sizes[p.layers++] = N;
                p.total += N;
                if (keep_all) p.off.push_back(p.total);
                p.np = p.F;
                p.F = N;
            }
            if (spec.layers_out && filled) {
                if (p.written < spec.layers_out_cap) launch_hash_sort_small(out, a.sizes, filled, stream_);
                export_layer(spec, out, used, p.written);
            }
            if (code == kSmallDone) {
                p.status = CG_OK;
                return true;
            }
            small_ok = made != 0 && code != kSmallFull;
            continue;  // the rules above, then the next run or a larger layer
        }

        // expected new states: layers grow by less and less
        uint64_t expect = std::min(C, room);
        if (p.np) {
            const double e = kExpectSlack * (double)p.F * (double)p.F / (double)p.np + 4096.0;
            if (e < (double)expect) expect = (uint64_t)e;
        }
        // (CG_EXPECT_FACTOR: times that, for tests of layers larger than expected)
        expect = std::max<uint64_t>((uint64_t)((double)expect * plan_factor("CG_EXPECT_FACTOR")), 1);
        const uint64_t most = p.np + p.F + std::min(C, room);
        const bool all_tags = cur.tagged && tags_.all;
        const uint64_t states = std::max(states_try, (all_tags ? 0 : p.np) + p.F + expect);
        HashPlan plan;
        bool ok = C <= most_candidates && hash_plan(p.F, all_tags ? k - 1 : k, states, &plan);
        HashBufs hb{};
        uint64_t *out = nullptr, out_cap = 0;
        DevBuf &out_buf = lay_[lay_at];
        if (ok) {
            try {
                part_[0].ensure(plan.bytes1());
                part_cnt_[0].ensure(plan.counts1() * 4);
                if (plan.lg2) {
                    part_[1].ensure(plan.bytes2());
                    part_cnt_[1].ensure(plan.counts2() * 4);
                }
                tab_[tab_at].ensure(8ull << plan.lg_q());
                if (keep_all) {
                    arena_room(std::min(expect, room));
                    out = arena_.as<uint64_t>() + p.total;
                    out_cap = arena_.bytes / 8 - p.total;
                } else {
                    out_buf.ensure(expect * 8);
                    out = out_buf.as<uint64_t>();
                    out_cap = out_buf.bytes / 8;
                }
            } catch (const Error &e) {
                if (!is_nomem(e)) throw;
                ok = false;
            }
        }
        uint64_t N = 0;
        if (ok) {
            uint64_t *ctr = hctr_.as<uint64_t>() + set * kHashCounterStride;
            set ^= 1u;
            hb = {part_[0].as<uint64_t>(),     part_[1].as<uint64_t>(), part_cnt_[0].as<uint32_t>(),
                  part_cnt_[1].as<uint32_t>(), ctr,                     hctr_.as<uint64_t>() + set * kHashCounterStride};
            launch_hash_partition(plan, gens, tags_, cur, hb, w_);
            uint64_t flags = 0;
            for (int attempt = 0;; ++attempt) {
                launch_hash_buckets(plan, prev, cur, hb, tags_, out, out_cap, tab_[tab_at].as<uint64_t>(), w_);
                CG_HIP(hipMemcpyAsync(host_small_, ctr, kHashCounters * 8, hipMemcpyDeviceToHost, stream_));
                CG_HIP(hipStreamSynchronize(stream_));
                N = host_small_[kHashCount];
                flags = host_small_[kHashFlags];
                if (flags || N <= out_cap) break;
                if (N > C || N > room || attempt) throw Error(CG_E_DEVICE, "layer size out of range (device error)");
                // more new states than expected: the buckets once more into
                // a larger buffer
                try {
                    if (keep_all) {
                        arena_room(N);
                        out = arena_.as<uint64_t>() + p.total;
                        out_cap = arena_.bytes / 8 - p.total;
                    } else {
                        out_buf.ensure(N * 8);
                        out = out_buf.as<uint64_t>();
                        out_cap = out_buf.bytes / 8;
                    }
                } catch (const Error &e) {
                    if (!is_nomem(e)) throw;
                    ok = false;
                    break;
                }
                launch_clear(nullptr, 0, ctr, kHashCounters, stream_);
            }
            if (prof_.on) prof_.collect();
            if (flags & kHashFlagPart) ok = false;
            else if (flags & kHashFlagTable) {
                if (states < most) {
                    states_try = std::min(most, 2 * states);
                    continue;
                }
                ok = false;
            }
        }
        if (!ok) {
            hand_to_sort(spec, prev, cur, p);
            return false;
        }
        states_try = 0;
        if (N > C || N > room) throw Error(CG_E_DEVICE, "layer size out of range (device error)");
        if (spec.layers_out && N) {
            try {
                if (p.written < spec.layers_out_cap)
                    export_layer(spec, sorted_copy(spec, out, N, order_[0], order_[1]), N, p.written);
                else
                    p.written += N;
            } catch (const Error &e) {
                // no room for the copies: the sort path, whose layers are
                // in order, makes the layer again
                if (!is_nomem(e)) throw;
                hand_to_sort(spec, prev, cur, p);
                return false;
            }
        }
        res->states_expanded += p.F;
        res->candidates += C;
        if (!N) {
            p.status = CG_OK;
            return true;
        }
        // (the candidates of tagged layers are counted as if each state had one
        // way back: an upper bound of what the kernels move)
        if (prof_.on) prof_.bytes[K_BUCKET] += 8.0 * (double)N;
        sizes[p.layers++] = N;
        const HashLayer next{out, N, tab_[tab_at].as<uint64_t>(), plan.lg_q(), tags_.on()};
        p.total += N;
        if (keep_all) p.off.push_back(p.total);
        prev = cur;
        cur = next;
        if (!keep_all) lay_at = (lay_at + 1) % 3;
        tab_at = (tab_at + 1) % 3;
        p.np = p.F;
        p.F = N;
        small_ok = true;
    }
}

}  // namespace cg
