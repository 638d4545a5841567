// Backward pass of the SALR layer  Y = X What^T + (X A_cat) B_cat  (the layer of paper Sec. 3.2 / 3.3; fine-tuning,
// whose throughput Sec. 4 compares, runs it every step).  The pruned base weight is frozen, the adapters train:
//     dX = dY What + (dY B_cat^T) A_cat^T        [M, K]
//     dA = X^T (dY B_cat^T)                      [K, R]
//     dB = (X A_cat)^T dY                        [R, N]
// Two launches (three where the matrix stage splits its contraction), or four:
//     the transposed weight in MFMA operand order, A_cat's rank blocks behind it (decode_transposed_frags_kernel), and in the same
//     launch's first workgroups T' = dY B_cat^T and T = X A_cat, both as they are [M, Rpad] and transposed (a launch of their own,
//     backward_t_kernel, where the weight is not wanted, R is no multiple of 8 or the chains are long and many);
//     dX: the large-batch matrix stage on dY and that weight, T' riding along as its adapter steps (salr_gemm.hip);
//     dA, dB: products that contract over the rows of X and dY against T'^T and T^T (salr_row_products.hpp), in workgroups beside the matrix
//     stage's where those leave room on a CU and the stage is long enough (gradients_beside), or in a launch of their own
//     and one that sums their slices.
// As in the forward pass T and T' are rounded to bf16 once; sums are fp32; outputs bf16.  The sixteen slices of T and T' interleave
// (every sixteenth step of 64 columns, whichever launch forms them), so a sum can differ from one over contiguous slices in its last
// bits, and where it sits on a rounding boundary by one bf16 step: about 2e-4 of dA and dB in the 2-norm against such a sum;
// against fp64 both are off by 2.35e-3, the two roundings.
#include "salr_internal.hpp"

namespace salr {

struct BackwardPlan {
    int Rpad, ks_tn;
    size_t off_wf, off_tp, off_tt, off_tp_t, off_tt_t, off_tn, off_words, off_ypart, y_room, total;
    bool words;   // there is room for the gradients' slices to meet
};

// What the call tells its callers to bring: the sizes of two dense copies of the weight, row-padded factors, the intermediates in
// both orders and split sums.  The plan below needs less for the weight and keeps its splits inside what is left; a few KB
// more on layers that are narrower than their rank.
static size_t backward_room(int64_t M, int64_t K, int64_t N, int64_t R, bool want_dx, bool want_dadb) {
    const size_t Rpad = (size_t)adapter_rank_padded(R);
    size_t o = 0, part = 0;
    if (want_dx) o += 2 * round_up_256((size_t)N * K * 2);
    o += round_up_256(M * Rpad * 2) + round_up_256(K * Rpad * 2) + round_up_256(N * Rpad * 2);
    if (R > 0) part = (size_t)adapter_ksplit(M, N) * M;
    if (want_dadb && R > 0) {
        o += round_up_256(M * Rpad * 2) + round_up_256(2 * M * Rpad * 2);
        const size_t c[3] = {(size_t)adapter_ksplit(M, K) * M, (size_t)tn_ksplit(K, M) * K, (size_t)tn_ksplit(N, M) * N};
        for (size_t v : c) part = v > part ? v : part;
    }
    o += round_up_256(part * Rpad * sizeof(float));
    const int ks_y = want_dx ? dense_ksplit(M, N, K) : 1;
    return o + (ks_y > 1 ? round_up_256((size_t)ks_y * M * K * sizeof(float)) : 0);
}

static BackwardPlan backward_plan(int64_t M, int64_t K, int64_t N, int64_t R, bool want_dx, bool want_dadb) {
    BackwardPlan p{};
    p.Rpad = (int)adapter_rank_padded(R);
    const bool grads = want_dadb && R > 0;
    const size_t room = backward_room(M, K, N, R, want_dx, want_dadb), t_bytes = (size_t)M * p.Rpad * sizeof(uint16_t);
    p.ks_tn = grads ? tn_ksplit(K, M, N) : 1;   // dA: columns of X, dB: columns of dY; both contract over M
    for (;; p.ks_tn /= 2) {
        size_t o = 0;
        auto take = [&](size_t bytes) { const size_t at = o; o += round_up_256(bytes); return at; };
        p.off_wf = take(want_dx ? frag_weight_bytes(N, K, R) : 0);
        p.off_tp = take(t_bytes);
        p.off_tt = take(grads ? t_bytes : 0);
        p.off_tp_t = take(grads ? t_bytes : 0);
        p.off_tt_t = take(grads ? t_bytes : 0);
        p.off_tn = take(grads ? (size_t)p.ks_tn * (K + N) * p.Rpad * sizeof(float) : 0);
        const size_t words = grads && want_dx ? (size_t)((K + 63) / 64 + (N + 63) / 64) * p.ks_tn * sizeof(uint64_t) : 0;
        p.words = words > 0 && o + round_up_256(words) <= room;
        p.off_words = take(p.words ? words : 0);
        p.off_ypart = o;
        if (o <= room || p.ks_tn == 1) break;
    }
    p.y_room = room > p.off_ypart ? room - p.off_ypart : 0;
    p.total = p.off_ypart + p.y_room;
    return p;
}

size_t linear_backward_workspace_bytes(int64_t M, int64_t K, int64_t N, int64_t R, bool want_dx, bool want_dadb) {
    return backward_plan(M, K, N, R, want_dx, want_dadb).total;
}

hipError_t launch_linear_backward(const uint16_t* x, const uint16_t* dy, int64_t M, int64_t K, int64_t N,
                                  const uint32_t* bitmap, const uint16_t* values, const uint32_t* row_offsets,
                                  const uint16_t* a_cat, const uint16_t* b_cat, int64_t R64, uint16_t* dx, uint16_t* da,
                                  uint16_t* db, void* workspace, hipStream_t stream) {
    const bool want_dx = dx != nullptr, want_dadb = (da != nullptr || db != nullptr);
    const BackwardPlan p = backward_plan(M, K, N, R64, want_dx, want_dadb);
    const int R = (int)R64;
    char* ws = static_cast<char*>(workspace);
    auto at = [&](size_t offset) { return reinterpret_cast<uint16_t*>(ws + offset); };

    // T' is needed by dX and dA, T by dB: in the launch that decodes the weight where there is one
    const LowRankJob none{nullptr, nullptr, 0, nullptr, nullptr};
    LowRankJob dy_b = none, x_a = none;
    if (R > 0 && (want_dx || da != nullptr)) dy_b = {dy, b_cat, N, at(p.off_tp), da != nullptr ? at(p.off_tp_t) : nullptr};
    if (R > 0 && db != nullptr) x_a = {x, a_cat, K, at(p.off_tt), at(p.off_tt_t)};
    // (A launch of their own, four times the waves to a chain of steps, where the chains are long and there are many of them for the
    // weight's size.  Own launch / in the decode launch, us a call: 3392 x 19072 x 576 rank 64 263 / 275, 4096 x 8192 x 512 rank 128
    // 215 / 223, 4096 x 10240 x 1024 rank 64 197 / 203; 3392 x 6144 x 1024 rank 128 196 / 192, 2048 x 1024 x 10240 rank 64 126 / 115,
    // 2048 x 4096 x 14336 rank 32 313 / 287.)
    const bool short_chains = K <= 6144 && N <= 6144, few = M * (K + N) * ((p.Rpad + 31) / 32) <= 6 * N * K;
    const bool with_decode = want_dx && R % 8 == 0 && (short_chains || few);
    if (R > 0 && !with_decode) launch_backward_t(dy_b, x_a, M, R, stream);
    const bool beside = p.words && handover_aligned(workspace);
    RowProducts products{{x, dy}, {at(p.off_tp_t), at(p.off_tt_t)}, {da != nullptr ? K : 0, db != nullptr ? N : 0}, {da, db}, M, R, p.Rpad, p.ks_tn,
                         reinterpret_cast<float*>(ws + p.off_tn), reinterpret_cast<uint64_t*>(ws + p.off_words), beside ? next_handover_tag() : 0};
    bool gradients_done = false;
    if (want_dx) {
        const hipError_t e = launch_decode_transposed_frags(bitmap, values, row_offsets, N, K, a_cat, R, at(p.off_wf), with_decode ? dy_b : none,
                                                            with_decode ? x_a : none, M, stream);
        if (e != hipSuccess) return e;
        const TimingEvents none;
        gradients_done = launch_frag_gemm(dy, M, N, K, at(p.off_wf), at(p.off_tp), p.Rpad, dx, reinterpret_cast<float*>(ws + p.off_ypart), p.y_room,
                                          none, stream, beside ? &products : nullptr);
    }
    if (want_dadb && R > 0 && !gradients_done) {
        products.words = nullptr;
        launch_row_products(products, stream);
    }
    return hipGetLastError();
}

}  // namespace salr
