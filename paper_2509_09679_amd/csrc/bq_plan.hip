// Plan build: cos/sin twiddles and the scale-deferred coefficient tables, all derived from theta.
// (Paper: "pre-computed cos/sin twiddle factors stored in a lookup table", section "Inference
// Efficiency"; kept in float32 here, evaluated in double and rounded once.)
#include "bq_internal.h"

namespace bq {

// Marks the buffer as a plan of this shape and clears the flags that plan_table_kernel raises behind it.
__global__ void plan_header_kernel(PlanHeader *hdr, int n, int heads, int k)
{
    if (threadIdx.x == 0) {
        hdr->magic = kPlanMagic;
        hdr->n = n;
        hdr->heads = heads;
        hdr->k = k;
        hdr->fast_bad_fwd = 0;
        hdr->fast_bad_inv = 0;
    }
}

// The tables, in groups of elements that are independent of each other.  The scale D of an element before layer i is
// the product of the cosines of the layers in front of it, so a group needs from outside only the cosines its
// own elements meet there.  The k layers are split into the low kl and the high kh = k - kl:
//   low group  g: elements g 2^kl + l (l < 2^kl); layers 1 .. kl pair them among each other
//   high group g: elements l 2^kl + g (l < 2^kh); layers kl + 1 .. k pair them among each other
// A workgroup takes one group of one head: it evaluates the cosines and tangents of the group's own layers (one per
// pair) and the cosines of the other layers (one per element), then runs both directions over the own layers, the
// forward cascade in threads 0 .. 127 and the transposed one in threads 128 .. 255, partners' scales exchanged through
// LDS.  At n = 4096 that is 128 workgroups of 576 evaluations each (1.5 times the angles there are).  Bound by the
// latency of the double-precision sine and cosine.  One workgroup per head and direction walking
// all layers with a barrier each, which this replaces, evaluated every angle four times on two compute units.
// A high group's elements are 2^kl apart, so neighbouring groups share the cache lines they read and write: workgroups
// (dealt to the eight dies in turn) are numbered so that neighbouring groups are on the same die, whose L2 then puts the lines
// together.  In launch order many heads were slower than the kernel this replaces: 512 heads of 4096 396 us before, 606
// in launch order, 321 this way; 512 heads of 8192 897, 1209, 672.  One head, both launches, back to back: n = 4096
// 80 -> 7.2 us, n = 8192 163 -> 8.1, n = 16384 342 -> 9.4.
constexpr int kPlanThreads = 256, kPlanMaxThreads = 1024;  // of a workgroup (launch_plan_build)
constexpr int kPlanMaxGroup = 128;  // elements of a group: k <= 7 has one group per head, k <= 14 groups of <= 2^7

struct PlanTableArgs {
    const float *theta;
    int n, k, kl, low_groups, high_groups;
    float2 *cs;
    float *fg[2], *fd[2];
    float *fw;  // transposed cascade only
    float *fm;  // forward cascade only
    int *bad[2];
};

__global__ __launch_bounds__(kPlanMaxThreads) void plan_table_kernel(PlanTableArgs A)
{
    __shared__ double own_c[7][kPlanMaxGroup / 2], own_t[7][kPlanMaxGroup / 2];  // own layers, per pair
    __shared__ double other_c[7][kPlanMaxGroup];                                // the other layers, per element
    __shared__ double D[2][kPlanMaxGroup];
    const int n = A.n, k = A.k, kl = A.kl, kh = k - kl;
    const int groups = A.low_groups + A.high_groups;
    const int die = blockIdx.x & 7, each = gridDim.x >> 3, extra = gridDim.x & 7;
    const int place = die * each + (die < extra ? die : extra) + (int)(blockIdx.x >> 3);
    const int head = place / groups;
    int g = place % groups;
    const bool low = g < A.low_groups;
    if (!low) g -= A.low_groups;
    const int own = low ? kl : kh, first = low ? 0 : kl;     // own layers first + 1 .. first + own
    const int others = k - own, ofirst = low ? kl : 0;        // the other layers ofirst + 1 .. ofirst + others
    const int size = 1 << own, pairs = size >> 1;
    const int shift = low ? 0 : kl;  // own layer j (0-based) pairs l with l ^ (1 << j), element e = base | l << shift
    const int base = low ? g << kl : g;
    const float *th = A.theta + (size_t)head * k * (n / 2);
    const int tid = threadIdx.x;

    for (int q = tid; q < own * pairs + others * size; q += blockDim.x) {
        const bool mine = q < own * pairs;
        const int r = mine ? q : q - own * pairs;
        const int j = mine ? r >> (own - 1) : r >> own;       // layer inside its set
        int l = mine ? r & (pairs - 1) : r & (size - 1);
        if (mine) l = ((l >> j) << (j + 1)) | (l & ((1 << j) - 1));  // lower element of the pair
        const int i = (mine ? first : ofirst) + j + 1;
        const int e = base | (l << shift);
        const int p = ((e >> i) << (i - 1)) | (e & ((1 << (i - 1)) - 1));
        const size_t at = (size_t)(i - 1) * (n / 2) + p;
        const double t = (double)th[at];
        if (mine) {
            double s, c;
            sincos(t, &s, &c);
            own_c[j][r & (pairs - 1)] = c;
            own_t[j][r & (pairs - 1)] = s / c;
            A.cs[(size_t)head * k * (n / 2) + at] = make_float2((float)c, (float)s);
        } else {
            other_c[j][l] = cos(t);
        }
    }
    __syncthreads();
    const int inverse = tid >= kPlanMaxGroup, l = tid & (kPlanMaxGroup - 1);
    const bool live = l < size && tid < 2 * kPlanMaxGroup;
    const int e = base | (l << shift);
    float *fgh = A.fg[inverse] + (size_t)head * k * n;
    // scale in front of the group's own layers: the other layers' cosines in cascade order, if they come first
    double Dself = 1.0;
    if (live && (low ? inverse : !inverse))
        for (int j = 0; j < others; ++j) Dself *= other_c[inverse ? others - 1 - j : j][l];
    int bad = 0;
    const double lo_d = 0x1p-60, hi_d = 0x1p60, lo_c = 0x1p-100, hi_c = 0x1p100;
    for (int step = 0; step < own; ++step) {
        const int j = inverse ? own - 1 - step : step;
        const int i = first + j + 1;
        if (live) D[inverse][l] = Dself;
        __syncthreads();
        if (live) {
            const double Dpart = D[inverse][l ^ (1 << j)];
            const int pr = ((l >> (j + 1)) << j) | (l & ((1 << j) - 1));
            const double c = own_c[j][pr];
            double tt = own_t[j][pr];
            if (inverse) tt = -tt;
            // lower element: u_a -= t (D_b / D_a) u_b ; upper element: u_b += t (D_a / D_b) u_a
            double coef = tt * Dpart / Dself;
            if (!(l & (1 << j))) coef = -coef;
            const double nd = c * Dself;
            fgh[(size_t)(i - 1) * n + e] = (float)coef;
            if (inverse) A.fw[((size_t)head * k + (i - 1)) * n + e] = (float)Dself;  // scale before this layer
            if (!inverse && i == k) {
                const double m = Dself / c;
                A.fm[(size_t)head * n + e] = (float)m;
                if (!(fabs(m) > lo_d && fabs(m) < hi_d)) bad = 1;
            }
            const double ac = fabs(coef), ad = fabs(nd);
            if (!(ad > lo_d && ad < hi_d)) bad = 1;
            if (!(ac == 0.0 || (ac > lo_c && ac < hi_c))) bad = 1;
            Dself = nd;
        }
        __syncthreads();
    }
    // the group that holds the cascade's last layer has the output scales
    if (live && (inverse ? low : (!low || kh == 0))) A.fd[inverse][(size_t)head * n + e] = (float)Dself;
    if (bad) atomicOr(A.bad[inverse], 1);
}

hipError_t launch_plan_build(const float *theta, int n, int heads, int k, void *plan, hipStream_t stream)
{
    PlanLayout L = plan_layout(n, heads, k);
    char *p = (char *)plan;
    PlanHeader *hdr = (PlanHeader *)p;
    hipLaunchKernelGGL(plan_header_kernel, dim3(1), dim3(64), 0, stream, hdr, n, heads, k);
    PlanTableArgs F{};
    F.theta = theta;
    F.n = n;
    F.k = k;
    F.kl = k <= 7 ? k : (k + 1) / 2;
    F.low_groups = n >> F.kl;
    F.high_groups = k > F.kl ? n >> (k - F.kl) : 0;
    F.cs = (float2 *)(p + L.cs);
    F.fg[0] = (float *)(p + L.fg_fwd);
    F.fg[1] = (float *)(p + L.fg_inv);
    F.fd[0] = (float *)(p + L.fd_fwd);
    F.fd[1] = (float *)(p + L.fd_inv);
    F.fw = (float *)(p + L.fw_inv);
    F.fm = (float *)(p + L.fm_fwd);
    F.bad[0] = &hdr->fast_bad_fwd;
    F.bad[1] = &hdr->fast_bad_inv;
    // A plan that leaves compute units free: as many threads as evaluations, up to the workgroup's limit, because the rounds are one
    // behind the other (one head, both launches, 256 threads, sine and cosine apart / as it is: 4096 7.45 / 7.2 us, 8192 8.6 / 8.1, 16384 10.2 / 9.4).  Many
    // heads: 256, so that the units are not held by waves that wait (512 heads of 4096 321 us, with 576 threads 522).
    const int64_t workgroups = (int64_t)heads * (F.low_groups + F.high_groups);
    int threads = kPlanThreads;
    if (workgroups <= 256) {
        const int kh = k - F.kl;
        const int low = (F.kl << (F.kl - 1)) + (kh << F.kl), high = kh > 0 ? (kh << (kh - 1)) + (F.kl << kh) : 0;
        const int evals = low > high ? low : high, rounds = (evals + kPlanMaxThreads - 1) / kPlanMaxThreads;
        threads = ((evals + rounds - 1) / rounds + 63) & ~63;
        if (threads < kPlanThreads) threads = kPlanThreads;
    }
    hipLaunchKernelGGL(plan_table_kernel, dim3((unsigned)workgroups), dim3((unsigned)threads), 0, stream, F);
    return hipGetLastError();
}

}  // namespace bq
