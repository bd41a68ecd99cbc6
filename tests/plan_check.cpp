// CPU check of the launch plans (Alg. 6 over tile anti-diagonals, as built
// by csrc/api.hip): every (source, target) tile pair farther than knear apart
// is applied exactly once, by a node push whose sources are solved before it
// and whose targets are solved after it; side-stream pushes are released after
// their sources, waited for before any main op that writes their targets, and
// never run while a main op writes the same tiles; the host enqueue order
// respects every wait.  The launch functions are stubbed out: only the host
// planning code runs.  Exit status = number of failing cases.
#include <functional>
#include "api.hip"
#include <cstdio>
#include <map>
#include <set>
#include <tuple>
int check(int mt, int nt, int knear, int b_ident, bool defer) {
    bk::Plan plan; std::vector<int4> items;
    build_plan(mt, nt, knear, b_ident, defer, plan, items);
    const int Q = mt + nt - 1;
    std::vector<int> seg_pos(Q, -1);
    for (int i = 0; i < (int)plan.ops.size(); ++i)
        if (plan.ops[i].kind == 0) for (int D = plan.ops[i].K; D < plan.ops[i].L; ++D) seg_pos[D] = i;
    for (int D = 0; D < Q; ++D) if (seg_pos[D] < 0) { printf("diag %d unsolved\n", D); return 1; }
    // first main op that waits for side op c
    std::vector<int> first_wait(plan.side.size(), (int)plan.ops.size());
    for (int i = (int)plan.ops.size() - 1; i >= 0; --i)
        for (int c = 0; c < plan.ops[i].need_side; ++c) first_wait[c] = i;
    std::map<std::tuple<int,int,int,int>, int> cnt;
    int bad = 0;
    // lo < pos < hi in main-op time: source segment <= lo, target segment >= hi
    auto apply = [&](int lo, int hi, const bk::PlanOp& op, int4 it) {
        const int I0 = it.x, J0 = it.y, kind = it.z & 1, klo = it.z >> 1, khi = it.w, MT = op.macro;
        for (int a = 0; a < MT; ++a) for (int b = 0; b < MT; ++b) {
            int I = I0 + a, J = J0 + b;
            if (I >= mt || J >= nt || I + J < op.tlo || I + J >= op.thi) continue;
            for (int kt = klo; kt < khi; ++kt) {
                int sd;
                if (kind == 0) { if (!(kt <= I - knear - 1) || !(kt + J >= op.K && kt + J < op.Mid)) continue; sd = kt + J; }
                else { if (!(kt <= J - knear - 1) || !(I + kt >= op.K && I + kt < op.Mid)) continue; sd = I + kt; }
                if (b_ident && kind == 0) continue;
                cnt[{kind, I, J, kt}]++;
                if (!(seg_pos[sd] <= lo) || !(hi <= seg_pos[I + J])) {
                    if (bad < 5) printf("order error kind %d tgt (%d,%d) src %d lo %d hi %d sp %d tp %d\n", kind, I, J, kt, lo, hi, seg_pos[sd], seg_pos[I + J]);
                    ++bad;
                }
            }
        }
    };
    for (int i = 0; i < (int)plan.ops.size(); ++i) {
        const bk::PlanOp& op = plan.ops[i];
        if (op.kind == 1)
            for (int j = 0; j < op.item_cnt; ++j) apply(i - 1, i + 1, op, items[op.item_off + j]);
        // a main op never runs before the side ops its targets need
        for (int c = 0; c < (int)plan.side.size(); ++c) {
            const bk::PlanOp& so = plan.side[c];
            const bool overlap = op.tlo < so.thi && so.tlo < op.thi;
            if (overlap && i > so.rel && i < first_wait[c]) { if (bad < 5) printf("race: main %d with side %d\n", i, c); ++bad; }
        }
    }
    for (int c = 0; c < (int)plan.side.size(); ++c) {
        const bk::PlanOp& so = plan.side[c];
        if (!plan.ops[so.rel].rec_rel) { printf("side %d: release not recorded\n", c); ++bad; }
        for (int j = 0; j < so.item_cnt; ++j) apply(so.rel, first_wait[c], so, items[so.item_off + j]);
    }
    // enqueue order: every side op after its release op, main ops in order
    {
        std::vector<int> seen_main;
        int last_main = -1;
        for (auto& o : plan.order) {
            if (o.first == 0) { if (o.second != last_main + 1) { printf("main order\n"); ++bad; } last_main = o.second; }
            else if (plan.side[o.second].rel > last_main) { printf("side %d enqueued before its release\n", o.second); ++bad; }
        }
        // every waited side op is enqueued before the waiting main op
        std::vector<int> pos_side(plan.side.size(), -1), pos_main(plan.ops.size(), -1);
        for (int k = 0; k < (int)plan.order.size(); ++k) (plan.order[k].first ? pos_side : pos_main)[plan.order[k].second] = k;
        for (int i = 0; i < (int)plan.ops.size(); ++i)
            for (int c = 0; c < plan.ops[i].need_side; ++c)
                if (pos_side[c] > pos_main[i]) { printf("main %d waits for side %d enqueued later\n", i, c); ++bad; }
    }
    long missing = 0, dup = 0, expected = 0, extra = 0;
    for (int I = 0; I < mt; ++I) for (int J = 0; J < nt; ++J) {
        for (int kt = 0; kt < I - knear; ++kt) { if (b_ident) break; ++expected; auto c = cnt[{0, I, J, kt}]; if (c == 0) ++missing; if (c > 1) ++dup; }
        for (int kt = 0; kt < J - knear; ++kt) { ++expected; auto c = cnt[{1, I, J, kt}]; if (c == 0) ++missing; if (c > 1) ++dup; }
    }
    for (auto& kv : cnt) { auto [kind, I, J, kt] = kv.first; if (kind == 0 ? kt > I - knear - 1 : kt > J - knear - 1) ++extra; }
    int nnode = 0; for (auto& op : plan.ops) nnode += op.kind == 1;
    if (missing || dup || extra || bad || (mt == 128 && nt == 128 && knear == 8))
        printf("mt %d nt %d knear %d bident %d defer %d: main %zu (nodes %d) side %zu; far pairs %ld missing %ld dup %ld extra %ld errors %d\n",
               mt, nt, knear, b_ident, (int)defer, plan.ops.size(), nnode, plan.side.size(), expected, missing, dup, extra, bad);
    return (missing || dup || extra || bad) ? 1 : 0;
}
int main() {
    int fails = 0;
    int small[][2] = {{1,1},{2,3},{7,10},{10,7},{6,6},{9,5},{40,40},{70,33},{33,90}};
    for (auto& sh : small) for (int k : {0, 1, 3, 8}) for (int bi : {0, 1}) for (int d : {0, 1})
        fails += check(sh[0], sh[1], k, bi, d);
    for (int k : {1, 8}) for (int d : {0, 1}) fails += check(128, 128, k, 0, d);   // the 4096^2 layer
    // the library's choice on 256 CUs against the faster plan measured on
    // MI355X for each shape (tiles of 32; solve ms with one stream / two):
    // 1 = two streams, 0 = one stream, -1 = within 1% (either is accepted)
    int shapes[][3] = {
        {32, 32, 0},      // 1024 x 1024:   0.73 / 0.79
        {47, 47, 0},      // 1500 x 1500:   1.17 / 1.27
        {64, 64, 0},      // 2048 x 2048:   1.59 / 1.69
        {96, 96, -1},     // 3072 x 3072:   2.78 / 2.79
        {128, 96, 0},     // 4096 x 3072:   3.31 / 3.47
        {128, 128, -1},   // 4096 x 4096:   3.95 / 3.96
        {160, 160, 0},    // 5120 x 5120:   5.91 / 9.79
        {192, 192, 0},    // 6144 x 6144:   7.88 / 19.13
        {256, 64, 0},     // 8192 x 2048:   5.28 / 9.20
        {64, 256, 0},     // 2048 x 8192:   5.28 / 9.19
        {256, 128, 0},    // 8192 x 4096:   7.49 / 11.81
        {128, 256, 0},    // 4096 x 8192:   7.52 / 13.40
        {344, 128, 0},    // 11008 x 4096: 10.18 / 16.24
        {128, 344, 0},    // 4096 x 11008: 10.17 / 19.16
        {448, 128, 0},    // 14336 x 4096: 13.62 / 22.74
        {128, 448, 0},    // 4096 x 14336: 13.63 / 26.75
        {896, 256, 0},    // 28672 x 8192: the widest segment needs every CU
    };
    for (auto& sh : shapes) {
        bk::Plan p0, p1; std::vector<int4> it;
        build_plan(sh[0], sh[1], 8, 0, false, p0, it);
        const int R = side_split(p0, 256);
        bool two = false;
        if (R > 0) {
            build_plan(sh[0], sh[1], 8, 0, true, p1, it);
            two = use_two_streams(p0, p1, R, 256, 2);
        }
        printf("%dx%d tiles: %s stream plan\n", sh[0], sh[1], two ? "two" : "one");
        if (sh[2] >= 0 && two != (sh[2] != 0)) {
            printf("cost model picks the slower plan for %dx%d tiles\n", sh[0], sh[1]);
            ++fails;
        }
    }
    // a shape that the model gives to two streams (by 1%), so that its first solve times both
    {
        bk::Plan p0, p1; std::vector<int4> it;
        build_plan(69, 75, 8, 0, false, p0, it);
        build_plan(69, 75, 8, 0, true, p1, it);
        if (!use_two_streams(p0, p1, side_split(p0, 256), 256, 2)) { printf("2208 x 2400 is not timed\n"); ++fails; }
    }
    // after a timing: two streams only where they are more than 3% faster
    if (keep_two_streams(3.95f, 3.96f) || keep_two_streams(4.0f, 4.0f) || keep_two_streams(4.10f, 4.0f) ||
        !keep_two_streams(4.13f, 4.0f)) {
        printf("keep_two_streams\n");
        ++fails;
    }
    printf("fails %d\n", fails);
    return fails;
}
namespace bk {
void factor_ops(std::vector<std::function<hipError_t()>>&, hipStream_t, hipStream_t, hipEvent_t, hipEvent_t, const float*, int64_t, double, double*, double*, double*, double*, int*, int64_t*, float*, int64_t) {}
hipError_t pack_identity(hipStream_t, int64_t, float*) { return hipSuccess; }
hipError_t unpack_factor(hipStream_t, const float*, int64_t, float*) { return hipSuccess; }
int plan_timed_launches(const Plan&) { return 0; }
hipError_t fill_words(hipStream_t, void*, int64_t, uint32_t) { return hipSuccess; }
hipError_t check_scales(hipStream_t, const float*, int64_t, int*) { return hipSuccess; }
size_t gptq_workspace_floats(int64_t, int64_t) { return 0; }
hipError_t run_gptq(hipStream_t, const float*, int64_t, int64_t, const float*, float*, const QuantArgs&, int8_t*, float*, float*, int) { return hipSuccess; }
hipError_t run_plan(hipStream_t, hipStream_t, const Plan&, const float*, int64_t, int64_t, int, int, const Workspace&, const float*, const float*, int, const QuantArgs&, int8_t*, float*, float*, int, int, int, const int4*, hipEvent_t*, hipEvent_t*, hipEvent_t*) { return hipSuccess; }
hipError_t run_antidiag(hipStream_t, const float*, int64_t, int64_t, float*, float*, const float*, const float*, const QuantArgs&, int8_t*, float*, float*) { return hipSuccess; }
}
