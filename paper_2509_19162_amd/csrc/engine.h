// Single-job growth engine: the layer loop of the breadth-first search.
#pragma once

#include <vector>

#include "../../include/cayleygrowth.h"
#include "buckets.h"
#include "internal.h"

namespace cg {

// A validated job (generators deduplicated, identity dropped).
struct JobSpec {
    int n = 0;
    int k = 0;                  // distinct non-identity generators
    std::vector<uint8_t> gens;  // k rows of n bytes
    bool inverse_closed = true;
    bool binary = false;        // one bit per entry (0/1 start vector, n <= 64)
    uint8_t start[64] = {0};
    int max_layers = 1;
    uint64_t max_frontier = 0;
    uint32_t flags = 0;
    uint8_t *layers_out = nullptr;
    uint64_t layers_out_cap = 0;
    uint64_t orbit_bound = 1;  // n! / prod(mult!) of the start's entries
};

// Validates and canonicalises a job; throws Error(CG_E_INVAL / _UNSUPPORTED).
JobSpec canonicalize(const cg_job_t &job, bool batch);

// Whether a job's layers go by hash buckets (Engine::run_hashed).
bool hash_layers(const JobSpec &spec);
// Whether they go over a rank bitmap (Engine::run_ranked).
bool rank_layers(const JobSpec &spec);
// Upper bounds of the device bytes a job by either makes an engine hold.
uint64_t rank_layers_bytes(const JobSpec &spec);
uint64_t hash_layers_bytes(const JobSpec &spec);

double now_seconds();

// Sets the calling thread's cg_last_error() string.
void set_last_error(const std::string &msg);

class Engine {
public:
    explicit Engine(hipStream_t user_stream);
    ~Engine();
    Engine(const Engine &) = delete;
    Engine &operator=(const Engine &) = delete;

    // Runs the job to completion; fills res (layer_sizes must hold
    // spec.max_layers entries). Throws Error on failure.
    void run(const JobSpec &spec, cg_result_t *res);

    // Where a growth stands between layers: L_{d-1} has np states, L_d F.
    struct Progress {
        uint64_t np = 0, F = 1, total = 1, written = 0;
        int layers = 1, status = CG_OK;
        std::vector<uint64_t> off;  // keep_all: offsets of the layers in arena_
    };
    PipeWork &work() { return w_; }
    hipStream_t stream() const { return stream_; }
    // Reads back one u64 counter and the kernel error flag (synchronises).
    uint64_t read_counter();
    // Device bytes the engine's buffers hold now (they are kept between
    // runs; release_buffers() frees them), and the most they held at once in
    // the last run.
    uint64_t device_bytes();
    uint64_t peak_bytes() const { return held_.peak; }
    // Raises the error flag of the sort kernels (tests).
    void raise_error_flag();
    void release_buffers();

private:
    // Layers by hash buckets (buckets.hip). True when the growth ended;
    // false when the sort path has to go on from `p`: L_{d-1} and L_d are
    // then sorted in lay_[0] and lay_[1] (keep_all: in arena_).
    bool run_hashed(const JobSpec &spec, cg_result_t *res, uint64_t key0, Progress &p);
    // Layers over a rank bitmap (rankbits.hip): permutations of up to 12
    // entries.
    void run_ranked(const JobSpec &spec, cg_result_t *res, uint64_t key0, Progress &p);
    bool take_layer(const JobSpec &spec, cg_result_t *res, uint64_t N, Progress &p);
    // As before the first layer, with no buffer held.
    void start_over(const JobSpec &spec, cg_result_t *res, Progress &p);
    void export_ranked(const JobSpec &spec, const uint64_t *sizes, int layers);
    void run_sorted(const JobSpec &spec, cg_result_t *res, uint64_t key0, Progress &p, bool resume);
    void hand_to_sort(const JobSpec &spec, const HashLayer &prev, const HashLayer &cur, const Progress &p);
    uint64_t *sort_keys(const JobSpec &spec, uint64_t *keys, uint64_t *tmp, uint64_t n);
    uint64_t *sorted_copy(const JobSpec &spec, const uint64_t *keys, uint64_t n, DevBuf &a, DevBuf &b);
    // a buffer of this engine: its stream, counted
    void adopt(DevBuf &b) {
        b.stream = stream_;
        b.held = &held_;
    }
    // every device buffer beside the pipeline's own (w_)
    std::vector<DevBuf *> buffers();
    void export_layer(const JobSpec &spec, const uint64_t *d_keys, uint64_t count,
                      uint64_t &written);
    uint64_t forced_chunk(uint64_t C);
    uint64_t chunk_capacity(uint64_t C, size_t key_bytes);
    bool binary_ = false;  // the current run's states are binary (one bit per entry)
    uint64_t run_chunked(bool ranked, int n, const uint64_t *Ld, uint64_t F, const uint64_t *Ra, uint64_t na,
                         const uint64_t *Rb, uint64_t nb, int k, uint64_t cap, int rank_bits, int bit_lo, int bit_hi,
                         uint64_t *dst, uint64_t out_cap, uint64_t room, int in);

    hipStream_t stream_ = nullptr;
    HeldBytes held_;
    PipeWork w_;
    Profiler prof_;
    DevBuf gsel_, cand0_, cand1_, lay_[3], arena_, stage_, chunk_hist_, vis_[2];
    DevBuf rk_[3];  // ranked runs: 32-bit ranks of layers d-1, d, d+1
    // hash buckets: both partitions and their counts, the layers' bucket
    // tables, runs of small layers, counters and small-layer sizes, sort
    // space of layers that are read back
    DevBuf part_[2], part_cnt_[2], tab_[3], small_[3], hctr_, ssz_, order_[2];
    class WgRunner *wg_ = nullptr;  // small-job engine (created on first use)
    static constexpr size_t kHostSmallBytes = 16384;
    bool sorted_ = false;             // a layer of the current run was sorted beside the sort path
    HashTags tags_;                   // of the layers that hash buckets hold now
    HostKit kit_;
    uint64_t *host_small_ = nullptr;  // of the kit: counters read back, inputs uploaded
};

void fill_kstats(const Profiler &p, cg_result_t *res);

}  // namespace cg
