// What a call is planned to take, from the headers and sources that the library's host side is built from: a line of "kind M K N R nnz" in,
// a line of "name=value" out.  linear, codes: with the workspace for the fastest path.
#include <cstdio>
#include <cstring>

#include "salr.h"
#include "salr_backward.hip"   // (host code only: its plan is the file's own)

using namespace salr;

static void row_tiled(int64_t M, int64_t K, int64_t N, int64_t R, size_t room) {
    const RowtilePlan p = rowtile_plan_in(M, K, N, R, room);
    std::printf("kernel=rowtile parts=%d slices=%d t_slices=%d t_first=%d handed=%d\n", p.parts, p.ksplit, p.t_slices, (int)(R > 0 && !p.partial),
                (int)(R > 0 && rowtile_hands_over(M, K, N, R, p, room)));
}

static void small_batch(const char* kernel, int64_t M, int64_t K, int64_t N, int64_t R, size_t room) {
    const bool shares = shares_t(M, K, N, R) && room >= shared_t_bytes(M, N, R);
    std::printf("kernel=%s shared=%s\n", kernel, !shares ? "no" : (N + 15) / 16 + shared_t_blocks(R) <= 256 ? "own" : "beside");
}

int main() {
    char kind[16];
    long long M, K, N, R, nnz;
    while (std::scanf("%15s %lld %lld %lld %lld %lld", kind, &M, &K, &N, &R, &nnz) == 6) {
        if (!std::strcmp(kind, "linear")) {
            const size_t room = linear_workspace_bytes_fastest(M, K, N, R);
            if (linear_takes_rowtile(M, K, N, R, room)) row_tiled(M, K, N, R, room);
            else if (linear_slice_takes(M, K, N)) std::printf("kernel=slice\n");
            else if (M <= kStreamMaxM) small_batch("stream", M, K, N, R, room);
            else std::printf("kernel=large\n");
        } else if (!std::strcmp(kind, "codes")) {
            const size_t room = salr_qsalr_linear_workspace_bytes_fastest(M, K, N, R, nnz);
            if (qsalr_takes_rowtile(M, K, N, R, nnz)) row_tiled(M, K, N, R, room);
            else if (linear_nf4_takes(M, K, N, nnz)) small_batch(K <= 4096 ? "codes" : "codes, long slices", M, K, N, R, room);
            else std::printf("kernel=large\n");
        } else if (!std::strcmp(kind, "2of4")) {
            const bool stream = uses_2of4_stream(M, K, N);
            if (stream) small_batch("2of4", M, K, N, R, salr_linear_2of4_workspace_bytes(M, K, N, R));
            else std::printf("kernel=%s\n", uses_2of4_kernel(M, K, N) ? "2of4, row tiles" : "large");
        } else {   // backward: the matrix stage of dX, [M, N] x [N, K]
            const BackwardPlan b = backward_plan(M, K, N, R, true, true);
            const GemmPlan g = gemm_plan(M, N + b.Rpad, K, b.y_room);
            RowProducts p{};
            p.C[0] = K; p.C[1] = N; p.M = M; p.R = (int)R; p.Rpad = b.Rpad; p.ksplit = b.ks_tn;
            std::printf("mt=%d nt=%d split=%d beside=%d slices=%d\n", g.mt, g.nt, g.ksplit, (int)(b.words && gradients_beside(M, N, K, g, p)),
                        b.ks_tn < kBesideSlices ? b.ks_tn : kBesideSlices);
        }
    }
    return 0;
}
