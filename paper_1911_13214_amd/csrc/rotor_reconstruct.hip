// Algorithm 2 (OptRec) of Beaumont et al. (arXiv 1911.13214): rebuild the
// optimal persistent sequence of the whole chain from the decision table.
//
// The recursion is unrolled into a walk with an explicit stack kept in LDS,
// one wave per requested budget.  It is a chain of dependent reads of the
// decision table, so the wave reads ahead: 32 lanes take a frame (s, t, m) and
// the frames (s + 1, t, m - w_abar^s), (s + 2, t, ...), ... that follow it as
// long as the decisions are C_2, and find the first that is not (the frame's
// event); the other 32 do the same for a second frame.  A C_1 split reads both
// its parts at once, so a walk waits once per C_1 split instead of once per
// frame.  Measured on MI355X: ten budgets of a chain of L = 339, M = 500 (31 to
// 66 C_1 splits and about 400 frames each) 231 -> 99 us.
// Pending items always cover disjoint stage ranges (a split leaves [s, s'-1]
// pending while [s', t] is walked; the F_all^s of a run leave their B^s pending
// while what follows the run is walked), so the stack never holds more than L
// frames.
#include "rotor_internal.h"

namespace rotor {
namespace {

constexpr int kAhead = 32;  // frames read ahead, a half wave
// What ends a run of C_2 decisions: a split s' > 0, or
constexpr int kLeaf = 0, kNegative = -1, kOutOfBudget = -2, kNoEvent = -3;

// A pending item: B^{s + run - 1} .. B^s (backward), or a sub-chain whose
// first `run` decisions are C_2 and whose event comes next, at stage s + run
// with budget m.  m < 2^28, s and t < 2^13.
struct Frame {
    int s, t, run, event, m;
    bool backward;
};
__device__ inline void push(uint64_t *lo, int32_t *hi, int top, const Frame &f)
{
    lo[top] = ((uint64_t)f.backward << 63) | ((uint64_t)f.s << 50) | ((uint64_t)f.t << 37) | (uint32_t)f.m;
    hi[top] = (f.event << 16) | f.run;
}
__device__ inline Frame pop(const uint64_t *lo, const int32_t *hi, int top)
{
    const uint64_t v = lo[top];
    const int32_t h = hi[top];
    Frame f;
    f.backward = v >> 63;
    f.s = (int)((v >> 50) & 0x1fff);
    f.t = (int)((v >> 37) & 0x1fff);
    f.m = (int)(uint32_t)v;
    f.event = h >> 16;
    f.run = h & 0xffff;
    return f;
}

__global__ __launch_bounds__(64) void walk_kernel(const int64_t *__restrict__ params, int L, int M, int64_t pitch,
                                                  const int16_t *__restrict__ dec,
                                                  const int64_t *__restrict__ budgets, int64_t cap,
                                                  rotor_op *__restrict__ ops, int64_t *__restrict__ count,
                                                  int32_t *__restrict__ status)
{
    // two words per frame, then the prefix sums of w_abar and w_a (both clamped
    // to M + 1), the sums modulo 2^32: a run's first budget below 0 shows exactly, since its sum
    // passes M < 2^28 by at most 2^28; later ones may wrap and are not read
    // outside [0, M]
    extern __shared__ __align__(8) uint64_t stack[];
    int32_t *const stack_hi = (int32_t *)(stack + L + 1);
    uint32_t *const kept = (uint32_t *)(stack_hi + L + 1);
    int32_t *const wa_l = (int32_t *)(kept + L + 1);
    const int lane = threadIdx.x;
    const int b = blockIdx.x;
    const int64_t *wa = params + (int64_t)ROTOR_ROW_WA * L;
    const int64_t *wabar = params + (int64_t)ROTOR_ROW_WABAR * L;
    // a table filled from parameters outside the domain is unspecified and is
    // not walked
    const bool in_domain = chain_in_domain(params, L, lane);
    const int64_t m0 = budgets[b];
    if (!in_domain || m0 < 0 || m0 > M) {
        if (lane == 0) {
            count[b] = 0;
            status[b] = in_domain ? ROTOR_EINVAL : ROTOR_EDOMAIN;
        }
        return;
    }
    uint32_t sum = 0;
    for (int l0 = 0; l0 < L; l0 += 64) {
        const int l = l0 + lane;
        uint32_t v = l < L ? (uint32_t)min(wabar[l], (int64_t)M + 1) : 0u;
        for (int off = 1; off < 64; off *= 2) {
            const uint32_t up = __shfl_up(v, off);
            v += lane >= off ? up : 0u;
        }
        if (l < L) {
            kept[l + 1] = sum + v;
            wa_l[l] = (int32_t)min(wa[l], (int64_t)M + 1);
        }
        sum += __shfl(v, 63);
    }
    if (lane == 0)
        kept[0] = 0;
    __syncthreads();

    rotor_op *const out = ops + (int64_t)b * cap;
    int64_t n = 0;
    // `len` operations from place n on, the one at place i being op(i)
    auto emit = [&](int len, auto &&op) {
        for (int i = lane; i < len; i += 64)
            if (n + i < cap)
                out[n + i] = op(i);
        n += len;
    };
    const int i = lane & (kAhead - 1);
    const bool second = lane >= kAhead;
    // the runs and events of two frames (s, t, m) at once (the second: s > t
    // for none)
    auto look = [&](Frame &f, Frame &g) {
        const int s = second ? g.s : f.s, t = second ? g.t : f.t;
        const int si = s + i;
        int event = kNoEvent, mi = 0;
        // one lane past a run's last frame carries on with its budget
        if (si <= t) {
            mi = (int)((uint32_t)(second ? g.m : f.m) - (kept[si - 1] - kept[s - 1]));
            if (mi < 0 || mi > M) {
                event = kOutOfBudget;
            } else {
                const int dv = dec[row_of(L, si, t) * pitch + mi];
                event = dv < 0 ? kNegative : si == t ? kLeaf : dv > 0 ? dv : kNoEvent;
            }
        }
        const uint64_t found = __ballot(event != kNoEvent);
        auto take = [&](Frame &x, int half) {
            const uint32_t bits = (uint32_t)(found >> (half * kAhead));
            x.run = bits ? __ffs((int)bits) - 1 : kAhead;
            const int at = half * kAhead + min(x.run, kAhead - 1);
            x.event = bits ? __builtin_amdgcn_readlane(event, at) : kNoEvent;
            x.m = bits ? __builtin_amdgcn_readlane(mi, at) : (int)((uint32_t)x.m - (kept[x.s + kAhead - 1] - kept[x.s - 1]));
        };
        take(f, 0);
        if (g.s <= g.t)
            take(g, 1);
    };
    Frame f{1, L, 0, 0, (int)m0, false}, none{1, 0, 0, 0, 0, false};
    look(f, none);
    int32_t st = f.run == 0 && f.event == kNegative ? ROTOR_INFEASIBLE : ROTOR_OK;
    int top = 0;
    while (st == ROTOR_OK) {
        if (f.backward) {
            const int last = f.s + f.run - 1;
            emit(f.run, [&](int k) { return rotor_op{ROTOR_B, last - k}; });
        } else {
            const int s = f.s + f.run, t = f.t, m = f.m;
            if (f.run > 0) {
                emit(f.run, [&](int k) { return rotor_op{ROTOR_F_ALL, f.s + k}; });
                if (top + 1 > L) {
                    st = ROTOR_ECORRUPT;
                    break;
                }
                push(stack, stack_hi, top++, Frame{f.s, 0, f.run, 0, 0, true});
            }
            if (f.event == kNoEvent) {
                // more C_2 than the half wave reads; m may be below 0, which
                // the next look finds
                f = Frame{s, t, 0, 0, m, false};
                look(f, none);
                continue;
            }
            if (f.event == kLeaf) {
                emit(2, [&](int k) { return rotor_op{k == 0 ? ROTOR_F_ALL : ROTOR_B, s}; });
            } else if (f.event < 0) {
                st = ROTOR_ECORRUPT;
                break;
            } else {
                // F_ck^s, F_none^{s+1..s'-1}, then [s', t] with a^{s'-1} stored,
                // then [s, s'-1]
                const int sp = f.event;
                if (sp <= s || sp > t) {
                    st = ROTOR_ECORRUPT;
                    break;
                }
                const int mr = m - wa_l[sp - 2];
                if (mr < 0 || mr > M || top + 1 > L) {
                    st = ROTOR_ECORRUPT;
                    break;
                }
                emit(sp - s, [&](int k) { return rotor_op{k == 0 ? ROTOR_F_CK : ROTOR_F_NONE, s + k}; });
                Frame left{s, sp - 1, 0, 0, m, false};
                f = Frame{sp, t, 0, 0, mr, false};
                look(f, left);
                push(stack, stack_hi, top++, left);
                continue;
            }
        }
        if (top == 0)
            break;
        f = pop(stack, stack_hi, --top);
    }
    if (st == ROTOR_OK && n > cap)
        st = ROTOR_ECAPACITY;
    if (lane == 0) {
        count[b] = (st == ROTOR_OK || st == ROTOR_ECAPACITY) ? n : 0;
        status[b] = st;
    }
}

}  // namespace

hipError_t launch_reconstruct(const int64_t *params, int L, int M, int64_t pitch, int64_t rows,
                              const int16_t *dec_chain, int n_budgets, const int64_t *budgets, int64_t cap,
                              rotor_op *ops, int64_t *count, int32_t *status, hipStream_t stream)
{
    (void)rows;
    (void)hipGetLastError();  // an error the caller's earlier calls left behind is not this launch's
    const size_t lds = (sizeof(uint64_t) + sizeof(int32_t) + sizeof(uint32_t) + sizeof(int32_t)) * (size_t)(L + 1);
    walk_kernel<<<dim3(n_budgets), 64, lds, stream>>>(params, L, M, pitch, dec_chain, budgets, cap, ops, count,
                                                      status);
    return hipGetLastError();
}

}  // namespace rotor
