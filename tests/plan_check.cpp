// The planner of csrc/qlin.cpp on the host, for tests/test_planner.py: plans of
// handles that own no device memory.  The kernel launches are empty here; no
// function of this file calls the HIP runtime.
#include "../paper_2607_04244_amd/csrc/qlin.cpp"

namespace qlin {
hipError_t launch_repack(const uint32_t *, const uint16_t *, const uint16_t *, uint4 *, void *, int, int, bool, bool,
                         hipStream_t) { return hipSuccess; }
hipError_t launch_forward(int, int, int, bool, Route, int, size_t, const FwdArgs &, hipStream_t) { return hipSuccess; }
hipError_t launch_unpack(const uint4 *, uint8_t *, int, int, hipStream_t) { return hipSuccess; }
hipError_t launch_dequant(int, const uint4 *, const void *, bool, bool, uint16_t *, int, int, hipStream_t) {
    return hipSuccess;
}
hipError_t prepare_kernels() { return hipSuccess; }
hipError_t launch_quantize(const uint16_t *, const uint16_t *, const uint16_t *, uint32_t *, int, int, hipStream_t) {
    return hipSuccess;
}
hipError_t launch_tiled(bool, Route, TiledShape, const TiledArgs &, int, hipStream_t) { return hipSuccess; }
hipError_t launch_stream_read(const void *, size_t, int, uint32_t *, hipStream_t) { return hipSuccess; }
const char *kernel_name(int, int, int, bool) { return ""; }
hipError_t static_scratch_setup(int, hipStream_t) { return hipSuccess; }
void *static_scratch(int) { return nullptr; }
}  // namespace qlin

namespace {

// A group of n linears of K x N[i] on a device of 256 compute units.
struct Group {
    qlin_s h[kMaxMembers];
    Target t;
    Group(int n, const int *N, int K, int symmetric, int64_t ws) {
        for (int i = 0; i < n; ++i) {
            h[i].K = K;
            h[i].N = N[i];
            h[i].Kb = K / kGroup;
            h[i].Nt = N[i] / kTileN;
            h[i].num_cu = 256;
            h[i].device = 0;
            h[i].symmetric = symmetric != 0;
            h[i].cap_rows = capacity_rows(h[i].Kb);
        }
        qlin_t hs[kMaxMembers];
        for (int i = 0; i < n; ++i) hs[i] = &h[i];
        group_target_ws(n, hs, ws, &t);
    }
};

}  // namespace

extern "C" {

struct PlanOut {
    int64_t kern, S, Gn, TnMax, rows, ws_bytes;
};

// Status of the plan for a workspace of ws bytes (< 0: no limit), and the plan.
int pc_plan(int n, const int *N, int K, int symmetric, int path, int64_t split, int64_t M, int64_t ws, PlanOut *out) {
    Group g(n, N, K, symmetric, ws);
    if (check_path_rows(path, M) != QLIN_OK) return last_status();
    Plan p;
    const int rc = make_plan(g.t, path, split, M, &p);
    if (rc == QLIN_OK) *out = PlanOut{p.kern, p.S, p.Gn, p.TnMax, p.rows, (int64_t)plan_ws_bytes(p)};
    return rc;
}

// Workgroups of a decode launch of this plan whose chunk and range, as the
// kernels compute them, are not the quotient and remainder (-1: no such plan).
int64_t pc_wrong_work(int n, const int *N, int K, int path, int64_t split, int64_t M, int64_t ws) {
    Group g(n, N, K, 0, ws);
    Plan p;
    if (make_plan(g.t, path, split, M, &p) != QLIN_OK || p.kern == kKernTiled) return -1;
    uint16_t *ys[kMaxMembers] = {};
    const FwdArgs a = fwd_args(g.t, p, std::min<int64_t>(M, p.rows), nullptr, ys, nullptr, 0, 0);
    int64_t wrong = 0;
    for (int b = 0; b < p.grid; ++b) {
        const int c = gn_chunk(b, a.Gn, a.inv_gn, a.gn_shift);
        wrong += c != b / a.Gn || c >= a.S;
    }
    return wrong;
}

// The same for Gn ranges and S chunks whatever their plan: the last workgroups
// of every chunk, where a reciprocal that is too large errs first.
int64_t pc_wrong_chunks(int Gn, int64_t S) {
    uint32_t inv;
    int shift;
    gn_reciprocal(Gn, &inv, &shift);
    int64_t wrong = 0;
    for (int64_t c = 0; c < S; ++c)
        for (int64_t b : {c * Gn, c * Gn + Gn / 2, c * Gn + Gn - 1}) wrong += gn_chunk((int)b, Gn, inv, shift) != c;
    return wrong;
}

// The route of a launch over n members, bit i of f16 the route of member i.
int pc_route(int n, unsigned f16) {
    qlin_s h[kMaxMembers];
    Target t;
    t.nmem = n;
    for (int i = 0; i < n; ++i) {
        h[i].f16 = (f16 >> i) & 1u;
        t.mem[i] = &h[i];
    }
    return route_of(t);
}

// Most 16-byte units on one LDS bank group (of 16) among 16 lanes in a row, for
// the matrix cores' results (lane l: quarter l >> 4 of row l & 15) and for reads
// in row order, over rows rows.
int pc_sums_conflicts(int rows) {
    int worst = 0;
    for (int first = 0; first < rows * 4; first += 16)
        for (int order = 0; order < 2; ++order) {
            int n[16] = {};
            for (int i = first; i < first + 16; ++i) {
                const int u = order ? sums_unit(i >> 2, i & 3) : sums_unit(first / 64 * 16 + i % 16, first / 16 % 4);
                worst = std::max(worst, ++n[u & 15]);
            }
        }
    return worst;
}

}  // extern "C"
