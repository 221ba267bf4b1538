// Layer loop of the rank-bitmap engine (rankbits.hip): breadth-first search
// by layers of permutations of up to 12 entries (paper, section "Reminder on
// Cayley graphs, diameters, growth", definition of Growth).
#include <algorithm>
#include <cstdlib>
#include <cstring>

#include "bitmap.h"
#include "engine.h"
#include "rankbits.h"

namespace cg {

namespace {

// Candidates from which a layer takes a large step. S_10 with six random
// generators: a layer of 9e6 neighbours takes 336 us tested in memory; two
// launches and a read-back of their own cost about 30 us.
constexpr uint64_t kRbLargeCandidates = 1u << 20;
// States a chain of steps may add where the layer array grows on demand.
constexpr uint64_t kRbChainStates = 1u << 22;
// Room the layer array starts with (whole orbits up to n = 10).
constexpr uint64_t kRbFirstStates = 1u << 22, kRbFirstStates12 = 1u << 20;
// States from which a growth on S_11 that no stop rule cuts is taken to reach
// the whole group: the array is reserved at once (319 MB), chains need not
// heed its length.
constexpr uint64_t kRbWholeFrom = 4096;

// States a growth can record before a stop rule ends it.
uint64_t most_states(const JobSpec &spec) {
    const uint64_t orbit = spec.orbit_bound, k = (uint64_t)spec.k;
    uint64_t total = 1, F = 1;
    for (uint64_t left = (uint64_t)spec.max_layers - 1; left && total < orbit; --left) {
        const uint64_t next = std::min(orbit, k * (spec.max_frontier ? std::min(F, spec.max_frontier) : F));
        if (next == F) return std::min(orbit, total + left * next);
        total += next;
        F = next;
    }
    return std::min(total, orbit);
}
bool takes_whole(const JobSpec &spec) {
    return spec.n <= 11 && !spec.max_frontier && most_states(spec) == spec.orbit_bound;
}

}  // namespace

// The layer array (while it grows: the old one beside the new), the bitmaps and
// the partition at every frontier size. (Queued jobs read no layers back.)
uint64_t rank_layers_bytes(const JobSpec &spec) {
    const uint64_t orbit = spec.orbit_bound, k = (uint64_t)std::max(1, spec.k), most = most_states(spec);
    const uint64_t fmax = spec.max_frontier ? std::min(orbit, spec.max_frontier) : orbit;
    const uint64_t room = most + kSmallStates;
    uint64_t b = 8 * room;
    if (spec.n > 10) b += takes_whole(spec) ? 8 * (kRbFirstStates + kSmallStates) : 8 * room;
    b += (spec.n >= kRbLargeMinN ? 2 : 1) * 4 * rb_bitmap_words(spec.n);
    uint64_t parts = 0;
    for (uint64_t F = std::min(fmax, most); spec.n >= kRbLargeMinN && F * k >= kRbLargeCandidates; F /= 2) {
        const RbPlan p = rb_plan(F, (uint32_t)k);
        parts = std::max(parts, p.bytes() + 4 * p.parts());
    }
    b += parts + parts / 2;
    return b + (64ull << 20);
}

bool rank_layers(const JobSpec &spec) {
    if (spec.k == 0 || spec.binary || spec.n > kRbMaxN || !start_is_permutation(spec)) return false;
    if (spec.flags & (CG_PACKED_SORT | CG_BITMASK | CG_SMALL_JOB)) return false;
    return !std::getenv("CG_CHUNK_CANDIDATES") && !std::getenv("CG_RANK_FULL");
}

// Reads the states of every layer back, in order: layers are sorted first
// (small ones all in one launch, in place).
void Engine::export_ranked(const JobSpec &spec, const uint64_t *sizes, int layers) {
    uint64_t off = 0, written = 0;
    uint64_t *all = arena_.as<uint64_t>();
    ssz_.ensure((size_t)layers * 8);
    CG_HIP(hipMemcpyAsync(ssz_.p, sizes, (size_t)layers * 8, hipMemcpyHostToDevice, stream_));
    for (int d = 0; d < layers && written < spec.layers_out_cap;) {
        int e = d;
        uint64_t run = 0;
        while (e < layers && sizes[e] <= kSmallSortStates) run += sizes[e++];
        if (e > d) {
            launch_hash_sort_small(all + off, ssz_.as<uint64_t>() + d, (uint32_t)(e - d), stream_);
            export_layer(spec, all + off, run, written);
        } else {
            run = sizes[d];
            e = d + 1;
            const uint64_t *sorted;
            try {
                sorted = sorted_copy(spec, all + off, run, order_[0], order_[1]);
            } catch (const Error &e) {
                // one copy less, where the layer lies (not on whole lines:
                // 0.1 ms more for 3e6 states)
                if (e.code != CG_E_NOMEM) throw;
                order_[1].release();
                order_[0].ensure(run * 8);
                sorted = sort_keys(spec, all + off, order_[0].as<uint64_t>(), run);
            }
            export_layer(spec, sorted, run, written);
        }
        off += run;
        d = e;
    }
}

void Engine::run_ranked(const JobSpec &spec, cg_result_t *res, uint64_t key0, Progress &p) {
    const int n = spec.n;
    const uint32_t k = (uint32_t)spec.k;
    uint64_t *sizes = res->layer_sizes;
    const uint64_t orbit = spec.orbit_bound;

    // one upload: the start key, then the generators
    const size_t bytes = 64 + 2 * k * sizeof(GenSel);  // and their inverses
    std::vector<uint8_t> up(bytes);
    std::memcpy(up.data(), &key0, 8);
    for (uint32_t g = 0; g < k; ++g) {
        const uint8_t *row = spec.gens.data() + (size_t)g * n;
        uint8_t inv[16] = {0};
        for (int i = 0; i < n; ++i) inv[row[i]] = (uint8_t)i;
        const GenSel s[2] = {make_gensel(n, row), make_gensel(n, inv)};
        std::memcpy(up.data() + 64 + g * sizeof(GenSel), &s[0], sizeof(GenSel));
        std::memcpy(up.data() + 64 + (k + g) * sizeof(GenSel), &s[1], sizeof(GenSel));
    }
    gsel_.ensure(bytes);
    const void *from = up.data();
    if (bytes <= kHostSmallBytes) {
        std::memcpy(host_small_, up.data(), bytes);
        from = host_small_;
    }
    CG_HIP(hipMemcpyAsync(gsel_.p, from, bytes, hipMemcpyHostToDevice, stream_));

    RbArgs a{};
    a.sel = reinterpret_cast<const GenSel *>(gsel_.as<uint8_t>() + 64);
    a.k = k;
    a.max_frontier = spec.max_frontier;
    // room for `states` states in all; what is there is kept
    const uint64_t cut = most_states(spec);
    const bool whole_ok = takes_whole(spec);
    auto room_for = [&](uint64_t states) {
        states = std::min(states, cut) + kSmallStates;
        if (states * 8 > arena_.bytes) {
            DevBuf bigger;
            adopt(bigger);
            bigger.ensure(std::max<uint64_t>(states * 8, std::min<uint64_t>((cut + kSmallStates) * 8,
                                                                           arena_.bytes + arena_.bytes / 2)));
            if (p.total > 1 || a.all) {
                CG_HIP(hipMemcpyAsync(bigger.p, arena_.p, p.total * 8, hipMemcpyDeviceToDevice, stream_));
                CG_HIP(hipStreamSynchronize(stream_));
            }
            arena_.swap(bigger);
        }
        a.all = arena_.as<uint64_t>();
        a.cap = arena_.bytes / 8;
    };
    bool marked = false;         // `seen` and the counters are set up
    bool unused_marked = false;  // bit numbers of no rank are marked in it
    const uint64_t words = rb_bitmap_words(n);
    bool large_ok = n >= kRbLargeMinN;
    room_for(n <= 10 ? kRbFirstStates : kRbFirstStates12);
    CG_HIP(hipMemcpyAsync(a.all, gsel_.p, 8, hipMemcpyDeviceToDevice, stream_));
    bool small_ok = spec.inverse_closed;
    for (;;) {
        if (spec.max_frontier && p.F > spec.max_frontier) {
            p.status = CG_TRUNCATED;
            break;
        }
        if (p.layers >= spec.max_layers) {
            p.status = CG_TRUNCATED;
            break;
        }
        const uint64_t C = p.F * (uint64_t)k;
        if (small_ok && p.np + p.F <= kSmallStates && C <= kSmallMaxCand) {
            // small layers in one workgroup, straight behind the last one
            ssz_.ensure(8 + kSmallMaxLayers * 8);
            room_for(p.total + (1u << 18));
            HashSmallArgs s{};
            s.cur = a.all + p.total - p.F;
            s.prev = a.all + p.total - p.F - p.np;
            s.np = (uint32_t)p.np;
            s.nc = (uint32_t)p.F;
            s.k = k;
            const uint64_t left = (uint64_t)(spec.max_layers - p.layers);
            s.max_new = (uint32_t)std::min<uint64_t>(left, kSmallMaxLayers - 1);
            s.max_new_is_rule = s.max_new == left;
            s.max_frontier = spec.max_frontier;
            s.out = a.all + p.total;
            s.out_cap = a.cap - p.total;
            s.state = ssz_.as<uint32_t>();
            s.sizes = ssz_.as<uint64_t>() + 1;
            HashGens gens;
            gens.k = k;
            gens.sel = a.sel;
            launch_hash_small(s, gens, HashTags(), w_);
            CG_HIP(hipMemcpyAsync(host_small_, ssz_.p, 8 + kSmallMaxLayers * 8, hipMemcpyDeviceToHost, stream_));
            CG_HIP(hipStreamSynchronize(stream_));
            if (prof_.on) prof_.collect();
            const uint32_t made = ((const uint32_t *)host_small_)[0], code = ((const uint32_t *)host_small_)[1];
            if (made > s.max_new) throw Error(CG_E_DEVICE, "small-layer count out of range (device error)");
            for (uint32_t i = 0; i < made; ++i)
                if (!take_layer(spec, res, host_small_[1 + i], p)) break;
            marked = false;
            if (code == kSmallDone) {
                p.status = CG_OK;
                break;
            }
            small_ok = made != 0 && code != kSmallFull;
            continue;
        }
        // a large layer takes a step of its own; smaller ones a chain of
        // steps, as long as they are expected to stay small, whose sizes
        // are read back together
        bool large = large_ok && C >= kRbLargeCandidates;
        const bool pull = large && pull_is_less(orbit - p.total, p.F, p.np, k);
        RbPlan plan;
        uint32_t chain = 1;
        uint64_t most = p.F, sum = std::min(orbit, C);
        const bool whole = n <= 10 || (whole_ok && p.total >= kRbWholeFrom);
        if (!large) {
            const uint32_t longest = (uint32_t)std::min<int>(kRbChain, spec.max_layers - p.layers);
            const double grow = std::min((double)k, p.np ? 1.25 * (double)p.F / (double)p.np : (double)k);
            double c = (double)C * grow;
            // a shrinking growth is about to end
            const uint32_t enough = p.F < p.np ? 4 : longest;
            uint64_t last = sum;  // states of the chain's last layer at most
            while (chain < std::min(longest, enough) && (!large_ok || c < (double)kRbLargeCandidates)) {
                last = std::min(orbit, k * (spec.max_frontier ? std::min(last, spec.max_frontier) : last));
                if (!whole && sum + last > kRbChainStates) break;
                sum = std::min(orbit, sum + last);
                c *= std::max(grow, 0.5);
                ++chain;
            }
        } else if (!pull) {
            plan = rb_plan(p.F, k);
            try {
                part_[0].ensure(plan.bytes());
                part_cnt_[0].ensure(plan.parts() * 4);
            } catch (const Error &e) {
                if (e.code != CG_E_NOMEM) throw;
                part_[0].release();
                large = large_ok = false;
            }
        }
        room_for(whole ? orbit : p.total + sum);
        if (!marked) {
            vis_[0].ensure(words * 4);
            hctr_.ensure((2 * kRbWindow * kRbStride + 16) * 8);
            a.seen = vis_[0].as<uint32_t>();
            a.cnt = hctr_.as<uint64_t>() + 16;
            a.off = a.cnt + kRbWindow * kRbStride;
            a.flags = hctr_.as<uint32_t>();
            CG_HIP(hipMemsetAsync(a.seen, 0, words * 4, stream_));
            launch_rb_begin(n, a, (uint32_t)(p.layers - 1), p.total - p.F, p.F, stream_);
            marked = true;
            unused_marked = false;
        }
        if (pull) {
            vis_[1].ensure(words * 4);
            if (!unused_marked) launch_rb_mark_unused(n, a.seen, stream_);
            unused_marked = true;
            uint32_t *to = a.seen == vis_[0].as<uint32_t>() ? vis_[1].as<uint32_t>() : vis_[0].as<uint32_t>();
            launch_rb_pull(n, a, (uint32_t)(p.layers - 1), p.total - p.F, p.F, a.sel + k, to, w_);
            a.seen = to;
        } else if (large)
            launch_rb_large(n, a, (uint32_t)(p.layers - 1), p.total - p.F, p.F, plan, part_[0].as<uint32_t>(),
                            part_cnt_[0].as<uint32_t>(), w_);
        for (uint32_t i = 0; !large && i < chain; ++i) {
            launch_rb_step(n, a, (uint32_t)(p.layers - 1) + i, most, w_);
            most = std::min(orbit, most * k);
        }
        const size_t span = (16 + kRbWindow * kRbStride) * 8;
        static_assert((16 + kRbWindow * kRbStride) * 8 <= kHostSmallBytes, "counters fit the pinned buffer");
        CG_HIP(hipMemcpyAsync(host_small_, hctr_.p, span, hipMemcpyDeviceToHost, stream_));
        CG_HIP(hipStreamSynchronize(stream_));
        if (prof_.on) prof_.collect();
        const uint32_t flags = *(const uint32_t *)host_small_;
        if (flags & kRbFlagRoom) throw Error(CG_E_DEVICE, "layer larger than its room (device error)");
        if (flags & kRbFlagPart) {
            // a part overran: some neighbours are missing. What was found
            // is marked as seen, so the bitmap is built again from the
            // layers, and no further layer goes this way.
            large_ok = marked = false;
            continue;
        }
        const uint32_t d0 = (uint32_t)(p.layers - 1);
        bool ended = false;
        for (uint32_t i = 0; i < chain && !ended; ++i) {
            if (spec.max_frontier && p.F > spec.max_frontier) break;  // it was not expanded
            const uint64_t N = host_small_[16 + ((d0 + i + 1) % kRbWindow) * kRbStride];
            if (prof_.on) prof_.bytes[large && !pull ? K_BUCKET : K_STEP] += 8.0 * (double)N;
            ended = !take_layer(spec, res, N, p);
        }
        if (ended) {
            p.status = CG_OK;
            break;
        }
        small_ok = false;
    }
    if (spec.layers_out) export_ranked(spec, sizes, p.layers);
}

// Books the expansion of layer d, which found N new states. False when none.
bool Engine::take_layer(const JobSpec &spec, cg_result_t *res, uint64_t N, Progress &p) {
    res->states_expanded += p.F;
    res->candidates += p.F * (uint64_t)spec.k;
    if (p.total + N > spec.orbit_bound) throw Error(CG_E_DEVICE, "layer size out of range (device error)");
    if (!N) return false;
    res->layer_sizes[p.layers++] = N;
    p.total += N;
    p.np = p.F;
    p.F = N;
    return true;
}

}  // namespace cg
