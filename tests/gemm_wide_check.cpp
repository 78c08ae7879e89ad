// Host-side check of the launches that plan_wide adds to the square tiles and
// plan_few to the GEMV: over the projections of several widths and ragged row
// counts from 1 to 2048, every output tile is covered by exactly its K ranges
// (each stage or K tile once), partials fit the workspace, and the shapes are
// ones the launcher knows; 1 and 2 rows and unaligned operands stay the GEMV's,
// and no launch of up to 8 rows is a plain tile.
// Test infrastructure: builds the library's planning header for the host.
#include "gemm_plan.h"

#include <cstdio>
#include <cstdlib>
#include <map>
#include <string>
#include <vector>

namespace {

int failures = 0;
long launches = 0;
std::map<std::string, int> seen;

#define CHECK(cond, what)                                                                                     \
    do {                                                                                                      \
        if (!(cond)) {                                                                                        \
            if (++failures <= 20) std::printf("FAIL %s M=%d N=%d K=%d %dx%d/%d\n", what, p.M, p.N, p.K1, w.bm, \
                                              w.bn, w.splits);                                                \
            return;                                                                                           \
        }                                                                                                     \
    } while (0)

template <int BM, int BN, int BKE>
void check_stream(const pb::GemmParams& p, const pb::WidePlan& w) {
    const int nbm = (p.M + BM - 1) / BM, nbn = p.N / BN, nk = p.K1 / BKE, grid = nbm * nbn * w.splits;
    const int kst = w.splits > 1 ? w.kt * pb::BK / BKE : nk;
    CHECK(p.N % BN == 0 && p.K1 % BKE == 0, "divisibility");
    std::vector<int> cover((size_t)nbm * nbn * nk, 0);
    std::vector<char> part((size_t)nbm * nbn * w.splits, 0);
    for (int b = 0; b < grid; ++b) {
        const pb::StreamJob j = pb::stream_job<BM, BN, BKE>(p, kst, b, grid);
        CHECK(w.splits == 1 || (j.t0 * BKE == j.split * w.kt * pb::BK && w.kt * pb::BK % BKE == 0), "split ranges");
        CHECK(j.m0 >= 0 && j.m0 < p.M && j.m0 % BM == 0 && j.n0 >= 0 && j.n0 < p.N && j.n0 % BN == 0, "corner");
        CHECK(j.split >= 0 && j.split < w.splits && j.n >= 1 && j.t0 >= 0 && j.t0 + j.n <= nk, "range");
        const size_t t = (size_t)(j.m0 / BM) * nbn + j.n0 / BN;
        CHECK(!part[t * w.splits + j.split], "split twice");
        part[t * w.splits + j.split] = 1;
        for (int k = j.t0; k < j.t0 + j.n; ++k) ++cover[t * nk + k];
    }
    for (int c : cover) CHECK(c == 1, "stage coverage");
}

template <int BM, int BN>
void check_tiles(const pb::GemmParams& p, const pb::GemmWorkspace& ws, const pb::WidePlan& w) {
    const pb::TileGeometry g = pb::tile_geometry<BM, BN>(p, ws, w.splits, 0);
    const int nbm = (p.M + BM - 1) / BM, nbn = p.N / BN, nk = p.K1 / pb::BK;
    CHECK(p.N % BN == 0 && p.group % BN == 0, "divisibility");
    std::vector<int> cover((size_t)nbm * nbn * nk, 0);
    for (int b = 0; b < g.grid; ++b) {
        const pb::TileJob j = pb::tile_job<BM, BN>(p, g.sa, b, g.grid);
        CHECK(j.m0 >= 0 && j.m0 < p.M && j.m0 % BM == 0 && j.n0 >= 0 && j.n0 < p.N && j.n0 % BN == 0, "corner");
        CHECK(j.nk >= 1 && j.partial == (g.sa.splits > 1), "range");
        const size_t t = (size_t)(j.m0 / BM) * nbn + j.n0 / BN;
        for (int k = j.t_begin; k < j.t_begin + j.nk && k < nk; ++k) ++cover[t * nk + k];
    }
    for (int c : cover) CHECK(c == 1, "K coverage");
}

void run(int role, int M, int N, int K, int group, bool ln, size_t ws_bytes) {
    pb::GemmParams p{};
    p.M = M; p.N = N; p.K1 = K; p.group = group;
    static char dummy;
    if (ln) p.ln_out = &dummy;
    const pb::GemmWorkspace ws{ws_bytes ? (void*)0x40000000 : nullptr, ws_bytes};
    p.ldx = p.ldw = K;
    const bool few = M <= pb::GEMV_MAX_ROWS;
    const pb::TilePlan base = pb::plan_for_role(role, p, ws);
    const pb::WidePlan w = few ? pb::plan_few(p, ws) : pb::plan_wide(p, ws, base);
    if (few) {
        CHECK(pb::plan_wide(p, ws, base).kind == pb::WIDE_NONE, "few rows in a tile");
        CHECK(w.kind == pb::WIDE_NONE || (w.kind == pb::WIDE_STREAM && w.bm == 32), "kernel of few rows");
        CHECK(M > 2 || w.kind == pb::WIDE_NONE, "1 and 2 rows");
        pb::GemmParams q = p;
        q.X = (const void*)0x1002;
        CHECK(pb::plan_few(q, ws).kind == pb::WIDE_NONE, "unaligned X");
        q = p;
        q.W = (const void*)0x1008;
        CHECK(pb::plan_few(q, ws).kind == pb::WIDE_NONE, "unaligned W");
    }
    ++launches;
    char key[48];
    std::snprintf(key, sizeof key, "%d:%dx%dk%d/%d", w.kind, w.bm, w.bn, w.bk, w.splits);
    ++seen[key];
    if (w.kind == pb::WIDE_NONE) return;
    if (!few) {  // the sum's K ranges are the base's
        const pb::SplitArgs sa = pb::make_split(p, ws, base.splits);
        CHECK(base.ragged_tail == 0 && (w.splits == 1 || pb::make_split(p, ws, w.splits).kt_split == sa.kt_split),
              "ranges");
        CHECK(w.kind == pb::WIDE_STREAM ? w.kt == sa.kt_split : w.splits == base.splits, "order of the sum");
    }
    CHECK(w.splits == 1 || (ws.ws && (double)w.splits * M * N * 4 <= (double)ws_bytes), "workspace");
    if (w.kind == pb::WIDE_STREAM) {
        if (w.bm == 128 && w.bn == 64 && w.bk == 128) check_stream<128, 64, 128>(p, w);
        else if (w.bm == 64 && w.bn == 64 && w.bk == 128) check_stream<64, 64, 128>(p, w);
        else if (w.bm == 32 && w.bn == 32 && w.bk == 128) check_stream<32, 32, 128>(p, w);
        else if (w.bm == 32 && w.bn == 64 && w.bk == 256) check_stream<32, 64, 256>(p, w);
        else if (w.bm == 32 && w.bn == 64 && w.bk == 128) check_stream<32, 64, 128>(p, w);
        else CHECK(false, "unknown stream shape");
    } else if (w.kind == pb::WIDE_RING) {
        CHECK((w.bn == 128 && w.bm == 192) || (w.bn == 256 && w.bm == 256), "unknown ring shape");
        if (w.bm == 256) check_tiles<256, 256>(p, ws, w);
        else check_tiles<192, 128>(p, ws, w);
    } else {
        CHECK(w.bn == 256 && (w.bm == 192 || w.bm == 128), "unknown ping-pong shape");
        if (w.bm == 192) check_tiles<192, 256>(p, ws, w);
        else check_tiles<128, 256>(p, ws, w);
    }
}

}  // namespace

// the plan of one product of more than GEMV_MAX_ROWS rows: kernel, block and its
// K elements per stage, K ranges launched, K tiles per range of the sum
void print_plan(int M, int N, int K, size_t ws_bytes) {
    pb::GemmParams p{};
    p.M = M; p.N = N; p.K1 = K; p.group = N; p.ldx = p.ldw = K;
    const pb::GemmWorkspace ws{ws_bytes ? (void*)0x40000000 : nullptr, ws_bytes};
    const pb::TilePlan base = pb::plan_tiles(p, ws);
    const pb::WidePlan w = pb::plan_wide(p, ws, base);
    const char* kinds[] = {"tile", "stream", "ring", "pingpong"};
    if (w.kind == pb::WIDE_NONE)
        std::printf("tile %d %d 64 %d %d%s\n", base.tile, base.tile, base.splits,
                    pb::make_split(p, ws, base.splits).kt_split, base.ragged_tail ? " ragged" : "");
    else
        std::printf("%s %d %d %d %d %d\n", kinds[w.kind], w.bm, w.bn, w.kind == pb::WIDE_STREAM ? w.bk : 64, w.splits,
                    pb::make_split(p, ws, base.splits).kt_split);
}

int main(int argc, char** argv) {
    if (argc == 5) {
        print_plan(std::atoi(argv[1]), std::atoi(argv[2]), std::atoi(argv[3]), std::strtoull(argv[4], nullptr, 10));
        return 0;
    }
    for (int d : {128, 256, 384, 2048, 2176, 4096, 5120, 9216})
        for (int F : {4 * d, 4 * d + 64})
            for (int M : {1, 2, 3, 4, 5, 8, 9, 16, 31, 32, 33, 61, 64, 65, 100, 128, 129, 200, 256, 257, 333, 385, 512, 513, 700, 1000, 2000,
                          2048, 2049})
                for (size_t ws : {(size_t)0, (size_t)16 << 20, (size_t)1 << 30}) {
                    run(0, M, 3 * d, d, d, false, ws);
                    run(0, M, d, d, d, false, ws);
                    run(1, M, d, d, d, true, ws);
                    run(2, M, F, d, F, false, ws);
                    run(3, M, d, F, d, true, ws);
                    run(3, M, d, F, d, false, ws);
                }
    std::printf("%ld launches, %d failures;", launches, failures);
    for (const auto& kv : seen) std::printf(" [%s] %d", kv.first.c_str(), kv.second);
    std::printf("\n");
    return failures ? 1 : 0;
}
