// PPO update of the trainable policy / value heads on cached encoder outputs (Sec. 3.1 Eq. 1,
// Sec. 3.2, Appendix hyper-parameter table), and the generalised advantage estimate.
//
// The backbone is frozen, so a rollout stores h_t once and the update touches only the two small
// MLPs: every mini-batch is a forward pass of both heads, the clipped-surrogate / entropy / value
// gradients at their outputs, back-propagation, one global gradient-norm clip and an Adam step.
// The products are tiny (64 x 2560 x 256), so a step is latency: it is laid out as four kernels
// (first layer of both heads; everything between the first layer's outputs and its deltas, one
// workgroup per sample; all weight gradients; gradient norm and Adam), of which the last takes the
// next step's first along where it can, the two large contractions
// on the fp64 matrix cores, every sum in fp64 in a fixed order: results do not depend on scheduling.
// Parameters and optimiser state are fp32 in one flat buffer each (policy W_1, b_1, ..., W_L, b_L,
// then the value head likewise); activations, deltas and gradients of a step live in fp64 scratch.
#include "mlp_f64.hpp"

#include <cmath>
#include <cstring>

namespace brl {

namespace {

constexpr int PPO_MAX_LAYERS = 8;

struct HeadShape {
    int n;                           // layers
    int dims[PPO_MAX_LAYERS + 1];
    size_t w_off[PPO_MAX_LAYERS];    // offsets into the flat parameter buffer
    size_t b_off[PPO_MAX_LAYERS];
};

struct Layout {
    HeadShape head[2];               // 0 policy, 1 value
    size_t n_params, n_policy;
};

int make_layout(const brl_ppo_config* c, Layout& L) {
    BRL_REQUIRE(c != nullptr, "ppo: null config");
    BRL_REQUIRE(c->policy_dims && c->value_dims, "ppo: null layer sizes");
    BRL_REQUIRE(c->policy_layers >= 1 && c->policy_layers <= PPO_MAX_LAYERS && c->value_layers >= 1 &&
                    c->value_layers <= PPO_MAX_LAYERS,
                "ppo: 1..%d layers per head", PPO_MAX_LAYERS);
    BRL_REQUIRE(c->act == BRL_ACT_TANH || c->act == BRL_ACT_RELU, "ppo: unknown activation %d", c->act);
    size_t off = 0;
    for (int hd = 0; hd < 2; ++hd) {
        HeadShape& H = L.head[hd];
        H.n = hd == 0 ? c->policy_layers : c->value_layers;
        const int* dims = hd == 0 ? c->policy_dims : c->value_dims;
        for (int i = 0; i <= H.n; ++i) {
            BRL_REQUIRE(dims[i] >= 1 && dims[i] <= (1 << 20), "ppo: layer size %d", dims[i]);
            H.dims[i] = dims[i];
        }
        for (int l = 0; l < H.n; ++l) {
            H.w_off[l] = off;
            off += (size_t)H.dims[l + 1] * H.dims[l];
            H.b_off[l] = off;
            off += (size_t)H.dims[l + 1];
        }
        if (hd == 0) L.n_policy = off;
    }
    L.n_params = off;
    BRL_REQUIRE(L.head[0].dims[0] == L.head[1].dims[0], "ppo: the heads disagree on the input width");
    BRL_REQUIRE(L.head[1].dims[L.head[1].n] == 1, "ppo: the value head must end in one output");
    BRL_REQUIRE(L.head[0].dims[L.head[0].n] <= 1024, "ppo: at most 1024 actions");
    return BRL_OK;
}

// ---- kernels ---------------------------------------------------------------------------------

// adv[e, t], ret[e, t] for E independent rollouts of T steps, backwards in fp64:
// delta = r + gamma V' (1 - done) - V;  A = delta + gamma lambda (1 - done) A'
// The recurrence A_t = delta_t + c_t A_{t+1} is a composition of affine maps.  Each of a rollout's threads composes the
// maps of a contiguous stretch of steps, a suffix scan over them (in a fixed order) gives every stretch the value that
// enters it from the right, and a second walk writes the results.  A rollout has as many threads as stretches of eight
// steps, at most a workgroup's; a workgroup takes as many rollouts as fit.  One thread per rollout walked 2048 dependent
// steps in 303 us, this takes 5 us; a workgroup per rollout took 89 us for 65536 rollouts of 16 steps (6 us here).
// SHIFT: log2 of a rollout's threads, or -1 for the argument (a whole workgroup's scan unrolled: 2048 steps 4.0 us, 4.4).
constexpr int GAE_THREADS = 256, GAE_STRETCH = 8;
template <int SHIFT>
__global__ __launch_bounds__(GAE_THREADS) void gae_kernel(const float* __restrict__ rewards, const float* __restrict__ values,
                                                          const float* __restrict__ dones, const float* __restrict__ last_value,
                                                          int E, int T, int per, int shift_arg, double gamma, double lam,
                                                          float* __restrict__ adv, float* __restrict__ ret) {
    __shared__ double sm[2][GAE_THREADS], sa[2][GAE_THREADS];       // composed maps x -> sm x + sa, ping-pong
    const int shift = SHIFT >= 0 ? SHIFT : shift_arg;
    const int threads = 1 << shift, tid = threadIdx.x, rt = tid & (threads - 1);      // threads and thread of a rollout
    const int e = (int)((blockIdx.x * GAE_THREADS + tid) >> shift), steps = e < E ? T : 0;
    const size_t row = (size_t)min(e, E - 1) * T;
    const int t0 = min(steps, rt * per), t1 = min(steps, t0 + per);  // steps t0 .. t1 - 1
    const double v_after = t1 < steps ? (double)values[row + t1] : (double)last_value[min(e, E - 1)];
    double m = 1.0, a = 0.0, nxt = v_after;
#pragma unroll 8
    for (int t = t1 - 1; t >= t0; --t) {
        const double live = 1.0 - (double)dones[row + t], v = (double)values[row + t];
        const double delta = (double)rewards[row + t] + gamma * nxt * live - v, c = gamma * lam * live;
        a = delta + c * a;
        m = c * m;
        nxt = v;
    }
    sm[0][tid] = m;
    sa[0][tid] = a;
    __syncthreads();
    // suffix composition: afterwards sa[tid] is the value at t0 of thread tid (nothing enters after the last step)
    int cur = 0;
    for (int off = 1; off < threads; off <<= 1) {
        double mm = sm[cur][tid], aa = sa[cur][tid];
        if (rt + off < threads) {
            aa = aa + mm * sa[cur][tid + off];
            mm = mm * sm[cur][tid + off];
        }
        sm[cur ^ 1][tid] = mm;
        sa[cur ^ 1][tid] = aa;
        cur ^= 1;
        __syncthreads();
    }
    double A = rt + 1 < threads ? sa[cur][tid + 1] : 0.0;
    nxt = v_after;
#pragma unroll 8
    for (int t = t1 - 1; t >= t0; --t) {
        const double live = 1.0 - (double)dones[row + t], v = (double)values[row + t];
        const double delta = (double)rewards[row + t] + gamma * nxt * live - v;
        A = delta + gamma * lam * live * A;
        adv[row + t] = (float)A;
        ret[row + t] = (float)(A + v);
        nxt = v;
    }
}

// Rollout indices and actions are caller data read on the device: they are clamped into range so that a bad
// entry can never address memory outside the rollout or the logits (its result is then meaningless, not a fault).
__device__ inline int clamp_index(int v, int n) { return v < 0 ? 0 : (v >= n ? n - 1 : v); }

typedef double v2d_u __attribute__((ext_vector_type(2), aligned(8)));      // rows of the flat buffers start anywhere

// ---- first layer of both heads: z[b, o] = sum_i W[o, i] h[rows[b], i], columns of the policy head first (mlp_f64.hpp)
// One more workgroup computes the mean and deviation of the mini-batch's advantages.
struct FirstArgs {
    const float* h;
    const int32_t* rows;
    const float* W[2];
    int out_dim[2], tiles[2];        // output units and their tiles of 16, per head
    int B, T, d, splits, btiles;
    double* z;                       // [splits][B][out_dim[0] + out_dim[1]]
    const float* adv;
    double adv_eps;
    int normalize_adv;
    double* scal;                    // [0] mean, [1] 1 / (deviation + eps)
};

// by the first 256 threads of a workgroup (the others keep step)
__device__ void minibatch_scale(const float* adv, const int32_t* rows, int B, int T, double eps, int normalize, double* scal) {
    __shared__ double red[256];
    if (!normalize) {
        if (threadIdx.x == 0) { scal[0] = 0.0; scal[1] = 1.0; }
        return;
    }
    const int tid = (int)threadIdx.x, first = tid < 256 ? tid : B;
    auto total = [&](double part) {                      // fixed tree
        if (tid < 256) red[tid] = part;
        __syncthreads();
        for (int st = 128; st >= 1; st >>= 1) {
            if (tid < st) red[tid] += red[tid + st];
            __syncthreads();
        }
        const double r = red[0];
        __syncthreads();
        return r;
    };
    double part = 0.0;
    for (int b = first; b < B; b += 256) part += (double)adv[clamp_index(rows[b], T)];
    const double mean = total(part) / (double)B;
    part = 0.0;
    for (int b = first; b < B; b += 256) {
        const double d = (double)adv[clamp_index(rows[b], T)] - mean;
        part += d * d;
    }
    const double ss = total(part);
    if (threadIdx.x == 0) {
        const double sd = B > 1 ? sqrt(ss / (double)(B - 1)) : 0.0;
        scal[0] = mean;
        scal[1] = 1.0 / (sd + eps);
    }
}

// ALL: a workgroup takes all of its tile's inputs (a.splits is 1)
template <bool ALL>
__global__ __launch_bounds__(256, 3) void ppo_first_layer_kernel(FirstArgs a) {
    __shared__ FirstLayerSums<ALL, 4> part;
    const int tiles = a.tiles[0] + a.tiles[1];
    if ((int)blockIdx.x == tiles * a.splits * a.btiles) {
        minibatch_scale(a.adv, a.rows, a.B, a.T, a.adv_eps, a.normalize_adv, a.scal);
        return;
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int split = blockIdx.x % a.splits, tile = (blockIdx.x / a.splits) % tiles, bt = blockIdx.x / (a.splits * tiles);
    const int hd = tile >= a.tiles[0] ? 1 : 0;
    const int o0 = (tile - (hd ? a.tiles[0] : 0)) * 16;
    const float* hrow[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) hrow[q] = a.h + (size_t)clamp_index(a.rows[min(bt * 64 + q * 16 + (lane & 15), a.B - 1)], a.T) * a.d;
    double sum[4];
    first_layer_sums<ALL, 4>(a.W[hd] + (size_t)min(o0 + (lane & 15), a.out_dim[hd] - 1) * a.d, hrow, a.d, split, part, sum);
    const int ncol = a.out_dim[0] + a.out_dim[1];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int b = bt * 64 + u * 16 + 4 * wave + (lane >> 4), o = o0 + (lane & 15);
        if (b < a.B && o < a.out_dim[hd])
            a.z[((size_t)split * a.B + b) * ncol + (hd ? a.out_dim[0] : 0) + o] = sum[u];
    }
}

// ---- from the first layer's sums to every delta, one workgroup per sample ---------------------------------------
// The layers above the first are small (256 -> 18, 256 -> 1): one workgroup runs the rest of both heads forward, the
// clipped surrogate (Eq. 1), the entropy bonus and the value error with their gradients, and both heads backward on
// activations and deltas in its LDS.  One launch (8.6 us, a chain of L2 and fp64 exp / log / tanh latencies) for what were
// three (second layer 6 us, loss 14 us, deltas 5 us).  Used wherever the units fit the LDS, whatever weights every
// workgroup then reads: a step at 64 samples of 2560 inputs 39 us against 73 with the level kernels below for hidden 256,
// 64 / 158 for 256, 256 (136 k weights above the first layers), 149 / 257 for 480, 480 (470 k), 220 / 360 for a policy head
// of 1000, 1000 (1 M); at 8 samples 35 / 56, 63 / 127, 149 / 200, 218 / 309, at 1024 three times ahead.
constexpr int TAIL_MAX_UNITS = 2048;          // layer outputs of both heads together: activations and deltas in 32 KB of LDS
constexpr int TAIL_THREADS = 512;             // (256: 1.5 us more at 512 first-layer units: every loop over units has two rounds)
struct TailArgs {
    const double* z;                 // first-layer sums [splits][B][..]
    int splits, B, A, T, act;
    int n[2];
    int dims[2][PPO_MAX_LAYERS + 1];
    const float* W[2][PPO_MAX_LAYERS];
    const float* bias[2][PPO_MAX_LAYERS];
    double* acts[2][PPO_MAX_LAYERS];     // [B, dims[l + 1]], hidden layers
    double* delta[2][PPO_MAX_LAYERS];    // [B, dims[l + 1]]
    const int32_t* rows;
    const int32_t* actions;
    const float* logp_old;
    const float* adv;
    const float* returns;
    const double* scal;
    double clip_eps, ent_coef;
    double* row_terms;               // [4, B]
};

// Clipped surrogate of one sample (Eq. 1): the term, whether its gradient flows, and its derivative by log pi(action)
struct Surrogate {
    double term, active, coef;
    __device__ Surrogate(double logp, double logp_old, double adv, double clip_eps) {
        const double ratio = exp(logp - logp_old);
        const double surr1 = ratio * adv;
        const double surr2 = fmin(fmax(ratio, 1.0 - clip_eps), 1.0 + clip_eps) * adv;
        term = fmin(surr1, surr2);
        active = surr1 <= surr2 ? 1.0 : 0.0;
        coef = -(active * adv * ratio);
    }
};
// derivative of a sample's loss by one logit of log-probability lp, entropy ent
__device__ inline double logit_slope(double coef, bool taken, double lp, double ent, double ent_coef, int B) {
    const double p = exp(lp);
    return (coef * ((taken ? 1.0 : 0.0) - p) + ent_coef * p * (lp + ent)) / (double)B;
}

__device__ inline double act_slope(double a, int act) { return act == BRL_ACT_RELU ? (a > 0.0 ? 1.0 : 0.0) : 1.0 - a * a; }

__global__ __launch_bounds__(TAIL_THREADS) void ppo_tail_kernel(TailArgs a) {
    __shared__ double out[TAIL_MAX_UNITS], del[TAIL_MAX_UNITS];      // layer outputs / deltas, policy head first
    const int tid = threadIdx.x, b = blockIdx.x;
    const int ncol = a.dims[0][1] + a.dims[1][1];
    const int r = clamp_index(a.rows[b], a.T);
    // the loss terms' inputs are requested ahead of the layers
    const double adv_r = ((double)a.adv[r] - a.scal[0]) * a.scal[1];
    const double logp_old = (double)a.logp_old[r], ret = (double)a.returns[r];
    const int action = clamp_index(a.actions[r], a.A);
    int off1 = 0;                                                    // where the value head's units start
    for (int l = 0; l < a.n[0]; ++l) off1 += a.dims[0][l + 1];

    for (int c = tid; c < ncol; c += TAIL_THREADS) {
        const int hd = c >= a.dims[0][1] ? 1 : 0, o = c - (hd ? a.dims[0][1] : 0);
        double v = first_layer_total(a.z + (size_t)b * ncol + c, a.splits, (size_t)a.B * ncol) + (double)a.bias[hd][0][o];
        if (a.n[hd] > 1) {
            v = activate(v, a.act);
            a.acts[hd][0][(size_t)b * a.dims[hd][1] + o] = v;
        }
        out[(hd ? off1 : 0) + o] = v;
    }
    __syncthreads();
    // the layers above, level by level for both heads: eight lanes per output unit
    constexpr int LG = 8, GROUPS = TAIL_THREADS / LG;
    const int depth = max(a.n[0], a.n[1]);
    int in0[2] = {0, off1};
    for (int l = 1; l < depth; ++l) {
        const int od0 = l < a.n[0] ? a.dims[0][l + 1] : 0, od1 = l < a.n[1] ? a.dims[1][l + 1] : 0, total = od0 + od1;
        for (int u = tid / LG; u < (total + GROUPS - 1) / GROUPS * GROUPS; u += GROUPS) {
            const int uc = min(u, total - 1), hd = uc >= od0 ? 1 : 0, o = uc - (hd ? od0 : 0);
            const int id = a.dims[hd][l], od = a.dims[hd][l + 1];
            double v = group_dot<LG>(a.W[hd][l] + (size_t)o * id, out + in0[hd], id);
            if (tid % LG == 0 && u < total) {
                v += (double)a.bias[hd][l][o];
                if (l + 1 < a.n[hd]) {
                    v = activate(v, a.act);
                    a.acts[hd][l][(size_t)b * od + o] = v;
                }
                out[in0[hd] + id + o] = v;
            }
        }
        in0[0] += od0 ? a.dims[0][l] : 0;
        in0[1] += od1 ? a.dims[1][l] : 0;
        __syncthreads();
    }
    const int lp0 = off1 - a.A;                                      // logits
    int lv = off1;                                                   // value
    for (int l = 0; l + 1 < a.n[1]; ++l) lv += a.dims[1][l + 1];
    if (tid < 64) {                                                  // one wavefront, a lane per action (and every 64th on)
        const double* z = out + lp0;
        double m = z[0];
        for (int k = tid; k < a.A; k += 64) m = fmax(m, z[k]);
        m = wave_reduce(m, [](double a, double b) { return fmax(a, b); });
        double se = 0.0;
        for (int k = tid; k < a.A; k += 64) se += exp(z[k] - m);
        const double lse = m + log(wave_sum(se));
        const Surrogate sg(z[action] - lse, logp_old, adv_r, a.clip_eps);
        double ent = 0.0;
        for (int k = tid; k < a.A; k += 64) {
            const double lp = z[k] - lse;
            ent -= exp(lp) * lp;
        }
        ent = wave_sum(ent);
        for (int k = tid; k < a.A; k += 64) {
            const double d = logit_slope(sg.coef, k == action, z[k] - lse, ent, a.ent_coef, a.B);
            del[lp0 + k] = d;
            a.delta[0][a.n[0] - 1][(size_t)b * a.A + k] = d;
        }
        if (tid == 0) {
            const double diff = out[lv] - ret, dv = diff / (double)a.B;
            del[lv] = dv;
            a.delta[1][a.n[1] - 1][b] = dv;
            a.row_terms[0 * a.B + b] = sg.term;
            a.row_terms[1 * a.B + b] = ent;
            a.row_terms[2 * a.B + b] = diff * diff;
            a.row_terms[3 * a.B + b] = 1.0 - sg.active;
        }
    }
    __syncthreads();
    // backward, level by level for both heads: a thread per unit of the layer below
    int at0 = lp0, at1 = lv;                                         // deltas of the level above
    for (int t = 0; t < depth - 1; ++t) {
        const int l0 = a.n[0] - 1 - t, l1 = a.n[1] - 1 - t;
        const int id0 = l0 >= 1 ? a.dims[0][l0] : 0, id1 = l1 >= 1 ? a.dims[1][l1] : 0;
        for (int u = tid; u < id0 + id1; u += TAIL_THREADS) {
            const int hd = u >= id0 ? 1 : 0, l = hd ? l1 : l0, i = u - (hd ? id0 : 0), id = hd ? id1 : id0;
            const int od = a.dims[hd][l + 1], up = hd ? at1 : at0, in = up - id;
            const float* w = a.W[hd][l] + i;
            double v = 0.0;
            int o = 0;
            for (; o + 16 <= od; o += 16) {
                float wv[16];
#pragma unroll
                for (int q = 0; q < 16; ++q) wv[q] = w[(size_t)(o + q) * id];
#pragma unroll
                for (int q = 0; q < 16; ++q) v += del[up + o + q] * (double)wv[q];
            }
            for (; o < od; ++o) v += del[up + o] * (double)w[(size_t)o * id];
            v *= act_slope(out[in + i], a.act);
            del[in + i] = v;
            a.delta[hd][l - 1][(size_t)b * id + i] = v;
        }
        at0 -= id0;
        at1 -= id1;
        __syncthreads();
    }
}

// ---- heads too wide for that: one launch per layer level forward and backward, one for the loss ------------------
constexpr int FB = 4;        // samples per workgroup
constexpr int FO = 4;        // output units per workgroup
// out[b, o] = act(sum_i W[o, i] in(b, i) + bias[o]); a workgroup takes FO output units for FB consecutive
// samples (weight rows and inputs are read once for all of them); its four wavefronts take a quarter of the
// inputs each, sum in fp64 in lane order, fold, and the four parts are added in order.
// in(b, i) = in64[b, i], or for the first layer the cached encoder output h[rows[b], i].
// One launch runs the same layer level of both heads (they read the same rows of h and depend on nothing of
// each other): the workgroups of problem 0 come first, then those of problem 1.
struct FwdProblem {
    const double* in64;      // null: first layer, inputs are rows of h
    const float* W;
    const float* bias;
    double* out;
    int in_dim, out_dim, last;
    unsigned blocks;
};
struct FwdArgs {
    FwdProblem p[2];
    int n;                   // 1 or 2 problems
    const float* h;
    const int32_t* rows;
    int B, act, T;
};
__global__ __launch_bounds__(256) void ppo_forward_kernel(FwdArgs a) {
    const int which = (a.n > 1 && blockIdx.x >= a.p[0].blocks) ? 1 : 0;
    const unsigned block = blockIdx.x - (which ? a.p[0].blocks : 0u);
    const double* __restrict__ in64 = which ? a.p[1].in64 : a.p[0].in64;
    const float* __restrict__ W = which ? a.p[1].W : a.p[0].W;
    const float* __restrict__ bias = which ? a.p[1].bias : a.p[0].bias;
    double* __restrict__ out = which ? a.p[1].out : a.p[0].out;
    const int in_dim = which ? a.p[1].in_dim : a.p[0].in_dim;
    const int out_dim = which ? a.p[1].out_dim : a.p[0].out_dim;
    const int last = which ? a.p[1].last : a.p[0].last;
    const float* __restrict__ h = a.h;
    const int32_t* __restrict__ rows = a.rows;
    const int B = a.B, act = a.act;
    // a lane's weights and inputs are each loaded once and meet in FO * FB accumulators
    __shared__ double part[4][FO][FB];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int ogroups = (out_dim + FO - 1) / FO;
    const int bg = (int)(block / ogroups), og = (int)(block % ogroups);
    const float* w[FO];
#pragma unroll
    for (int u = 0; u < FO; ++u) w[u] = W + (size_t)min(og * FO + u, out_dim - 1) * in_dim;   // clamped duplicates are not stored
    const float* hrow[FB];
    const double* drow[FB];
#pragma unroll
    for (int q = 0; q < FB; ++q) {
        const int b = min(bg * FB + q, B - 1);
        hrow[q] = in64 ? nullptr : h + (size_t)clamp_index(rows[b], a.T) * in_dim;
        drow[q] = in64 ? in64 + (size_t)b * in_dim : nullptr;
    }
    const int quarter = (in_dim + 3) / 4;
    const int i_end = min(in_dim, (wave + 1) * quarter);
    double acc[FO][FB];
#pragma unroll
    for (int u = 0; u < FO; ++u)
#pragma unroll
        for (int q = 0; q < FB; ++q) acc[u][q] = 0.0;
#pragma unroll 2
    for (int i = wave * quarter + lane; i < i_end; i += 64) {
        double wi[FO], xi[FB];
#pragma unroll
        for (int u = 0; u < FO; ++u) wi[u] = (double)w[u][i];
#pragma unroll
        for (int q = 0; q < FB; ++q) xi[q] = in64 ? drow[q][i] : (double)hrow[q][i];
#pragma unroll
        for (int u = 0; u < FO; ++u)
#pragma unroll
            for (int q = 0; q < FB; ++q) acc[u][q] += wi[u] * xi[q];
    }
#pragma unroll
    for (int u = 0; u < FO; ++u)
#pragma unroll
        for (int q = 0; q < FB; ++q) {
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) acc[u][q] += __shfl_xor(acc[u][q], off, 64);
        }
    if (lane == 0) {
#pragma unroll
        for (int u = 0; u < FO; ++u)
#pragma unroll
            for (int q = 0; q < FB; ++q) part[wave][u][q] = acc[u][q];
    }
    __syncthreads();
    if (threadIdx.x < FO * FB) {
        const int u = threadIdx.x / FB, q = threadIdx.x % FB;
        const int b = bg * FB + q, o = og * FO + u;
        if (b < B && o < out_dim) {
            double z = ((part[0][u][q] + part[1][u][q]) + part[2][u][q]) + part[3][u][q] + (double)bias[o];
            if (!last) z = (act == BRL_ACT_RELU) ? fmax(z, 0.0) : tanh(z);
            out[(size_t)b * out_dim + o] = z;
        }
    }
}

struct LossArgs {
    const double* logits;     // [B, A]
    const double* v;          // [B]
    const int32_t* rows;      // [B] indices into the rollout
    const int32_t* actions;
    const float* logp_old;
    const float* adv;
    const float* returns;
    int B, A, T;
    double clip_eps, ent_coef, adv_eps;
    int normalize_adv;
    double* dlogits;          // [B, A]
    double* dv;               // [B]
    double* row_terms;        // [4, B] scratch
};

// One workgroup: advantage normalisation over the mini-batch, then a few lanes per sample for the
// clipped surrogate (Eq. 1), the entropy bonus and the value error, and their gradients at the heads' outputs.
__global__ __launch_bounds__(256) void ppo_loss_kernel(LossArgs a) {
    __shared__ double scal[2];                      // mean and scale of the advantages
    minibatch_scale(a.adv, a.rows, a.B, a.T, a.adv_eps, a.normalize_adv, scal);
    __syncthreads();
    // LG adjacent lanes share a sample: each takes every LG-th action; maxima and sums meet by butterfly
    constexpr int LG = 4;
    const int part = threadIdx.x % LG;
    for (int b0 = 0; b0 < a.B; b0 += 256 / LG) {
        const int b = b0 + (int)threadIdx.x / LG;
        const bool live = b < a.B;
        const int bc = live ? b : a.B - 1;              // idle lanes shadow the last sample and store nothing
        const int r = clamp_index(a.rows[bc], a.T);
        const double A = ((double)a.adv[r] - scal[0]) * scal[1];
        const double* z = a.logits + (size_t)bc * a.A;
        double m = z[0];
        for (int k = part; k < a.A; k += LG) m = fmax(m, z[k]);
#pragma unroll
        for (int off = 1; off < LG; off <<= 1) m = fmax(m, __shfl_xor(m, off, 64));
        double se = 0.0;
        for (int k = part; k < a.A; k += LG) se += exp(z[k] - m);
#pragma unroll
        for (int off = 1; off < LG; off <<= 1) se += __shfl_xor(se, off, 64);
        const double lse = m + log(se);
        const int act = clamp_index(a.actions[r], a.A);
        const Surrogate sg(z[act] - lse, (double)a.logp_old[r], A, a.clip_eps);
        double ent = 0.0;
        for (int k = part; k < a.A; k += LG) {
            const double lp = z[k] - lse;
            ent -= exp(lp) * lp;
        }
#pragma unroll
        for (int off = 1; off < LG; off <<= 1) ent += __shfl_xor(ent, off, 64);
        if (live) {
            for (int k = part; k < a.A; k += LG) a.dlogits[(size_t)b * a.A + k] = logit_slope(sg.coef, k == act, z[k] - lse, ent, a.ent_coef, a.B);
            if (part == 0) {
                const double diff = a.v[b] - (double)a.returns[r];
                a.dv[b] = diff / (double)a.B;
                a.row_terms[0 * a.B + b] = sg.term;
                a.row_terms[1 * a.B + b] = ent;
                a.row_terms[2 * a.B + b] = diff * diff;
                a.row_terms[3 * a.B + b] = 1.0 - sg.active;
            }
        }
    }
}

// ---- weight gradients of every layer of both heads: dW[o, i] = sum_b delta[b, o] in(b, i), db[o] = sum_b delta[b, o] --
// A wavefront takes 16 output units x 64 inputs on the fp64 matrix cores: a lane reads four consecutive inputs of a
// sample, one for each of four result tiles, so that its results are four consecutive inputs again (32-byte stores).
// The squares of its gradients are summed (fixed tree) to one slot of partial[] for the global norm.
// 2 x 256 x 2560 from 64 samples: 29 us + 17 us for the second layers with vector FMAs and a launch per level, 11.8 us
// here for all of them (1292 wavefronts on 1024 SIMDs; one round of gathered reads, then 64 MFMAs each).
struct GradProblem {
    const double* delta;     // [B, out_dim]
    const double* in64;      // [B, in_dim]; null: first layer, inputs are rows of h
    double* gW;
    double* gb;
    int in_dim, out_dim, ichunks;
    int first;               // first wavefront of the problem
};
struct GradArgs {
    GradProblem p[2 * PPO_MAX_LAYERS];
    int n, waves;
    const float* h;
    const int32_t* rows;
    int B, T;
    double* partial;         // [waves]
};
// The sums over the samples, 64 samples' loads in flight (32 for fp64 inputs).  IN: 0 rows of h read 16 bytes at a time
// (in_dim a multiple of 4), 1 rows of h of any width, 2 fp64 activations.  Every load is unconditional with a clamped
// address and nothing is converted before all are requested: inputs past the row's end only reach results that are
// never stored, and under a branch each load would be waited for before the next (18.4 us that way, 11.8 us this).
template <int IN>
__device__ __forceinline__ void weight_grad_sums(const GradProblem& P, const GradArgs& a, int lane, int oc, bool o_ok, int i,
                                                 v4d (&acc)[4], double& db) {
    constexpr int NS = IN == 2 ? 8 : 16;             // groups of four samples requested together
    const int in_dim = P.in_dim, out_dim = P.out_dim, kk = lane >> 4;
    int at[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) at[e] = min(IN == 0 ? min(i, in_dim - 4) + e : i + e, in_dim - 1);
    for (int bb = 0; bb < a.B; bb += 64) {
        const int my_row = clamp_index(a.rows[min(bb + lane, a.B - 1)], a.T);
        const int b_end = min(a.B, bb + 64);
        for (int b0 = bb; b0 < b_end; b0 += 4 * NS) {
            double d[NS];
            v4f_u xf[IN == 2 ? 1 : NS];
            v4d xd[IN == 2 ? NS : 1];
#pragma unroll
            for (int u = 0; u < NS; ++u) {           // (sample past the end: any row, its delta counts as zero)
                const int bc = min(b0 + 4 * u + kk, a.B - 1);
                d[u] = P.delta[(size_t)bc * out_dim + oc];
                if constexpr (IN == 2) {
                    const double* row = P.in64 + (size_t)bc * in_dim;
#pragma unroll
                    for (int e = 0; e < 4; ++e) xd[u][e] = row[at[e]];
                } else {
                    const float* row = a.h + (size_t)__shfl(my_row, (4 * u + kk + b0 - bb) & 63, 64) * in_dim;
                    if constexpr (IN == 0) {
                        xf[u] = *reinterpret_cast<const v4f_u*>(row + at[0]);
                    } else {
#pragma unroll
                        for (int e = 0; e < 4; ++e) xf[u][e] = row[at[e]];
                    }
                }
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < NS; ++u) {
                if (b0 + 4 * u >= b_end) break;
                const double dv = (o_ok && b0 + 4 * u + kk < b_end) ? d[u] : 0.0;
                db += dv;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    double x;
                    if constexpr (IN == 2) x = xd[u][e];
                    else x = (double)xf[u][e];
                    acc[e] = __builtin_amdgcn_mfma_f64_16x16x4f64(dv, x, acc[e], 0, 0, 0);
                }
            }
        }
    }
}

__global__ __launch_bounds__(256) void ppo_weight_grad_kernel(GradArgs a) {
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * 4 + (threadIdx.x >> 6)));
    if (w >= a.waves) return;
    int pi = 0;
    while (pi + 1 < a.n && w >= a.p[pi + 1].first) ++pi;
    const GradProblem& P = a.p[pi];
    const int in_dim = P.in_dim, out_dim = P.out_dim;
    const int ot = (w - P.first) / P.ichunks, ic = (w - P.first) % P.ichunks;
    const int o = ot * 16 + (lane & 15), i = ic * 64 + 4 * (lane & 15), kk = lane >> 4;
    const bool o_ok = o < out_dim;
    const int oc = min(o, out_dim - 1);
    v4d acc[4] = {};
    double db = 0.0;
    if (P.in64) weight_grad_sums<2>(P, a, lane, oc, o_ok, i, acc, db);
    else if (in_dim % 4 == 0) weight_grad_sums<0>(P, a, lane, oc, o_ok, i, acc, db);
    else weight_grad_sums<1>(P, a, lane, oc, o_ok, i, acc, db);
    double sq = 0.0;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int oo = ot * 16 + 4 * v + kk;
        if (oo >= out_dim) continue;
        double* g = P.gW + (size_t)oo * in_dim + i;
        if (i + 4 <= in_dim) {
            *reinterpret_cast<v2d_u*>(g) = v2d_u{acc[0][v], acc[1][v]};
            *reinterpret_cast<v2d_u*>(g + 2) = v2d_u{acc[2][v], acc[3][v]};
#pragma unroll
            for (int e = 0; e < 4; ++e) sq += acc[e][v] * acc[e][v];
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (i + e < in_dim) {
                    g[e] = acc[e][v];
                    sq += acc[e][v] * acc[e][v];
                }
        }
    }
    if (ic == 0) {
        db += __shfl_xor(db, 16, 64);
        db += __shfl_xor(db, 32, 64);
        if (lane < 16 && o_ok) {
            P.gb[o] = db;
            sq += db * db;
        }
    }
    sq = wave_sum(sq);
    if (lane == 0) a.partial[w] = sq;
}

// delta_prev[b, i] = (sum_o delta[b, o] W[o, i]) * act'(a[b, i]), a = the activated output of the layer below
struct DeltaProblem {
    const double* delta;
    const float* W;
    const double* a_prev;
    double* delta_prev;
    int in_dim, out_dim;
    unsigned blocks;
};
struct DeltaArgs {
    DeltaProblem p[2];
    int n, B, act;
};
__global__ __launch_bounds__(256) void ppo_delta_kernel(DeltaArgs a) {
    const int which = (a.n > 1 && blockIdx.x >= a.p[0].blocks) ? 1 : 0;
    const unsigned block = blockIdx.x - (which ? a.p[0].blocks : 0u);
    const double* __restrict__ delta = which ? a.p[1].delta : a.p[0].delta;
    const float* __restrict__ W = which ? a.p[1].W : a.p[0].W;
    const double* __restrict__ a_prev = which ? a.p[1].a_prev : a.p[0].a_prev;
    double* __restrict__ delta_prev = which ? a.p[1].delta_prev : a.p[0].delta_prev;
    const int in_dim = which ? a.p[1].in_dim : a.p[0].in_dim;
    const int out_dim = which ? a.p[1].out_dim : a.p[0].out_dim;
    const int B = a.B, act = a.act;
    const size_t idx = (size_t)block * 256 + threadIdx.x;
    if (idx >= (size_t)B * in_dim) return;
    const int b = (int)(idx / in_dim), i = (int)(idx % in_dim);
    double acc = 0.0;
    for (int o = 0; o < out_dim; ++o) acc += delta[(size_t)b * out_dim + o] * (double)W[(size_t)o * in_dim + i];
    const double av = a_prev[idx];
    delta_prev[idx] = acc * (act == BRL_ACT_RELU ? (av > 0.0 ? 1.0 : 0.0) : 1.0 - av * av);
}

// ---- global gradient norm and Adam ------------------------------------------------------------------------------
// Up to ADAM_OWN_NORM partial sums every workgroup adds them itself, in one fixed order (thread t takes partials t,
// t + 256, ..., then a fixed tree): the same norm everywhere, and no launch of its own.  Beyond, where that work would grow
// with the square of the heads' size, a launch ahead leaves their total and the workgroups read one value.  Then Adam with bias correction on the clipped
// gradient, p -= lr (m / c1) / (sqrt(v / c2) + eps), scale min(1, max_norm / (norm + 1e-6)).  1.3 M parameters: 10.4 us
// for 42 MB, against 7 us for the norm alone in its own launch and 8.6 us for Adam (12.2 us with the partial sums read one
// after the other and three divisions per parameter).
struct AdamArgs {
    float* p;
    float* m;
    float* v;
    const double* g;
    size_t n, n_policy;
    const double* partial;
    int n_partials, B;
    double max_norm, step_policy, step_value, b1, b2, inv_c2, eps, ent_coef;   // steps: learning rate / (1 - b1^t)
    const double* row_terms;
    float* stats;            // [5]: policy loss, value loss, entropy, clip fraction, gradient norm; or null
};
constexpr int ADAM_PER_THREAD = 4;
// (64 samples, 2560 inputs, a step with the workgroups' own sums / with the launch, us: hidden 256 (1292 partials) 38.0 /
// 40.4, 384 (1938) 46.5 / 49.1, 640 (3230) 68.1 / 68.0, 1000 (5088) 92.5 / 89.7, 2048 (10336) 325 / 302, 4096 and 2048
// (36960) 2109 / 1650)
constexpr int ADAM_OWN_NORM = 3072;

// sum of the partials, in a fixed order
constexpr int NORM_THREADS = 1024;
__global__ __launch_bounds__(NORM_THREADS) void ppo_norm_kernel(const double* __restrict__ partial, int n, double* __restrict__ total) {
    __shared__ double red[NORM_THREADS / 64];
    double s = 0.0;
    for (int i0 = 0; i0 < n; i0 += NORM_THREADS * 8) {
        double t[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) t[u] = partial[min(i0 + u * NORM_THREADS + (int)threadIdx.x, n - 1)];
#pragma unroll
        for (int u = 0; u < 8; ++u) s += i0 + u * NORM_THREADS + (int)threadIdx.x < n ? t[u] : 0.0;
    }
    s = wave_sum(s);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < NORM_THREADS / 64; ++w) s += red[w];
        *total = s;
    }
}

// min(1, max_norm / (norm + 1e-6)) from the partial sums, by a whole workgroup; the norm itself to `norm`.  The
// order of the sum is that of 256 threads whatever the workgroup's size.
template <int NT>
__device__ inline double adam_scale(const AdamArgs& a, double (&red)[NT], double& norm) {
    const int tid = (int)threadIdx.x;
    double s = 0.0;
    if (tid < 256) {
        for (int i0p = 0; i0p < a.n_partials; i0p += 256 * 8) {      // eight of a thread's partial sums in flight
            double t[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) t[u] = a.partial[min(i0p + u * 256 + tid, a.n_partials - 1)];
#pragma unroll
            for (int u = 0; u < 8; ++u) s += i0p + u * 256 + tid < a.n_partials ? t[u] : 0.0;
        }
        red[tid] = s;
    }
    __syncthreads();
    // ((t + 128) first, then the pair's 64: the tree of a halving reduction)
    const int l = tid & 63;
    norm = sqrt(wave_sum((red[l] + red[l + 128]) + (red[l + 64] + red[l + 192])));
    return fmin(1.0, a.max_norm / (norm + 1e-6));
}

__device__ inline void adam_element(const AdamArgs& a, double scale, double step, double g, float& p, float& m, float& v) {
    const double gi = g * scale;
    const double mi = a.b1 * (double)m + (1.0 - a.b1) * gi;
    const double vi = a.b2 * (double)v + (1.0 - a.b2) * gi * gi;
    m = (float)mi;
    v = (float)vi;
    p = (float)((double)p - step * mi / (sqrt(vi * a.inv_c2) + a.eps));
}

// four neighbouring parameters with their state and gradients; the buffers may start at any element, so the accesses ask
// for no more.  n: how many of the four there are (the others are neither read nor written).
struct AdamQuad {
    float p[4], m[4], v[4];
    double g[4];
    __device__ __forceinline__ void load_all(const AdamArgs& a, size_t i) {
        const v4f_u pv = *reinterpret_cast<const v4f_u*>(a.p + i), mv = *reinterpret_cast<const v4f_u*>(a.m + i);
        const v4f_u vv = *reinterpret_cast<const v4f_u*>(a.v + i);
        const v2d_u g0 = *reinterpret_cast<const v2d_u*>(a.g + i), g1 = *reinterpret_cast<const v2d_u*>(a.g + i + 2);
        p[0] = pv.x; p[1] = pv.y; p[2] = pv.z; p[3] = pv.w;
        m[0] = mv.x; m[1] = mv.y; m[2] = mv.z; m[3] = mv.w;
        v[0] = vv.x; v[1] = vv.y; v[2] = vv.z; v[3] = vv.w;
        g[0] = g0.x; g[1] = g0.y; g[2] = g1.x; g[3] = g1.y;
    }
    __device__ __forceinline__ void load(const AdamArgs& a, size_t i, int n) {
        if (n >= 4) { load_all(a, i); return; }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const bool in = e < n;
            p[e] = in ? a.p[i + e] : 0.f; m[e] = in ? a.m[i + e] : 0.f; v[e] = in ? a.v[i + e] : 0.f;
            g[e] = in ? a.g[i + e] : 0.0;
        }
    }
    __device__ __forceinline__ void store(const AdamArgs& a, size_t i, int n) const {
        if (n >= 4) {
            *reinterpret_cast<v4f_u*>(a.p + i) = v4f_u{p[0], p[1], p[2], p[3]};
            *reinterpret_cast<v4f_u*>(a.m + i) = v4f_u{m[0], m[1], m[2], m[3]};
            *reinterpret_cast<v4f_u*>(a.v + i) = v4f_u{v[0], v[1], v[2], v[3]};
            return;
        }
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (e < n) { a.p[i + e] = p[e]; a.m[i + e] = m[e]; a.v[i + e] = v[e]; }
    }
};

// the five statistics of an update, by one wavefront
__device__ inline void adam_stats(const AdamArgs& a, double norm) {
    double t[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        double x = 0.0;
        for (int b = threadIdx.x; b < a.B; b += 64) x += a.row_terms[(size_t)k * a.B + b];
        t[k] = wave_sum(x);
    }
    if (threadIdx.x == 0) {
        const double n = (double)a.B;
        a.stats[0] = (float)(-t[0] / n - a.ent_coef * t[1] / n);
        a.stats[1] = (float)(0.5 * t[2] / n);
        a.stats[2] = (float)(t[1] / n);
        a.stats[3] = (float)(t[3] / n);
        a.stats[4] = (float)norm;
    }
}

// four parameters a thread, by a whole workgroup; returns the norm
template <int NT>
__device__ inline double adam_quad(const AdamArgs& a, size_t i0, int n, const double (&step)[4], double (&red)[NT]) {
    AdamQuad q;                                      // requested ahead of the norm
    q.load(a, i0, n);
    double norm;
    const double scale = adam_scale(a, red, norm);
#pragma unroll
    for (int e = 0; e < 4; ++e) adam_element(a, scale, step[e], q.g[e], q.p[e], q.m[e], q.v[e]);
    q.store(a, i0, n);
    return norm;
}
__global__ __launch_bounds__(256) void ppo_adam_kernel(AdamArgs a) {
    __shared__ double red[256];
    const size_t i0 = ((size_t)blockIdx.x * 256 + threadIdx.x) * ADAM_PER_THREAD;
    const int n = i0 < a.n ? (int)min((size_t)4, a.n - i0) : 0;
    double step[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) step[e] = i0 + e < a.n_policy ? a.step_policy : a.step_value;
    const double norm = adam_quad(a, i0, n, step, red);
    if (blockIdx.x == 0 && a.stats && threadIdx.x < 64) adam_stats(a, norm);
}

// ---- one update's Adam and the next mini-batch's first layer in one launch ---------------------------------------
// The first layers hold almost all parameters, and a workgroup of their contraction can be the only reader of its tile of
// weights (16 units, a group of inputs): it updates the tile itself (neighbouring threads neighbouring parameters), keeps
// the new weights in LDS and contracts them with all samples, 64 at a time.  Two wavefronts share a range of inputs, 32
// samples each, so that a SIMD has two chains of fp64 instructions to alternate between; the samples' inputs are requested
// ahead of everything else, the next samples' under the matrix instructions.  Further workgroups update the other
// parameters, which only later launches read.  The arithmetic and its order are those of the two kernels by themselves.
// Bound by the 42 MB of parameters, state and gradients (2 x 256 x 2560) and a chain of latencies: 13.8 us for 8.4 + 10.4 and
// a launch; Adam's arithmetic shows with 0.4 us of it, the contraction's with 1.7.
constexpr int FUSED_THREADS = 512;
constexpr int FUSED_MAX_CHUNKS = 6;                  // chunks of 16 inputs per range: 3072 inputs, 25 KB of weights in LDS
struct FusedArgs {
    FirstArgs f;                                     // of the next mini-batch
    AdamArgs a;                                      // of this one
    size_t w0[2];                                    // where the first layers' weights start in the flat buffers
    size_t rest0[2], rest_n[2];                      // the parameters behind them, per head
    int tile_blocks, rest_blocks[2];                 // workgroups of the tiles, of each head's other parameters
};
// ROUNDS: quads of parameters per thread, half the chunks per range
template <int ROUNDS>
__global__ __launch_bounds__(FUSED_THREADS, 4) void ppo_adam_first_kernel(FusedArgs t) {
    constexpr int LD = ROUNDS * 2 * 64 + 4;
    constexpr int REQUEST_AT = ROUNDS > 2 ? ROUNDS - 2 : 0;              // (before, they would not fit the registers)
    __shared__ double part[4][16][64];               // the ranges' sums
    __shared__ double red[FUSED_THREADS];
    __shared__ __attribute__((aligned(16))) float fresh[16][LD];
    const AdamArgs& a = t.a;
    const FirstArgs& f = t.f;
    const int block = (int)blockIdx.x, tid = (int)threadIdx.x;
    if (block >= t.tile_blocks) {
        int rb = block - t.tile_blocks;
        if (rb == t.rest_blocks[0] + t.rest_blocks[1]) {
            minibatch_scale(f.adv, f.rows, f.B, f.T, f.adv_eps, f.normalize_adv, f.scal);
            return;
        }
        const int hd = rb >= t.rest_blocks[0] ? 1 : 0;
        if (hd) rb -= t.rest_blocks[0];
        const size_t k0 = ((size_t)rb * FUSED_THREADS + tid) * ADAM_PER_THREAD;
        const int n = k0 < t.rest_n[hd] ? (int)min((size_t)4, t.rest_n[hd] - k0) : 0;
        const double step = hd ? a.step_value : a.step_policy;
        const double norm = adam_quad(a, t.rest0[hd] + k0, n, {step, step, step, step}, red);
        if (hd == 0 && rb == 0 && a.stats && tid < 64) adam_stats(a, norm);
        return;
    }
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), kk = lane >> 4;
    const int range = wave & 3, half = wave >> 2;
    const int split = block % f.splits, tile = block / f.splits;
    const int hd = tile >= f.tiles[0] ? 1 : 0;
    const int o0 = (tile - (hd ? f.tiles[0] : 0)) * 16, units = min(16, f.out_dim[hd] - o0);
    const int d = f.d, chunks = d / 16, per = first_layer_range_chunks(d);

    // inputs of the wavefront's samples, NC chunks at a time; past the last chunk some other, whose results are not used
    constexpr int NC = ROUNDS < 3 ? 2 * ROUNDS : ROUNDS;     // (one or two batches)
    const int c0 = (split * 4 + range) * per, nc = max(0, min(chunks, c0 + per) - c0);
    v4f_u next[NC][2];
    const float* hrow[2];
    auto rows_of = [&](int bt) {
#pragma unroll
        for (int q = 0; q < 2; ++q)
            hrow[q] = f.h + (size_t)clamp_index(f.rows[min(bt * 64 + (half * 2 + q) * 16 + (lane & 15), f.B - 1)], f.T) * d;
    };
    auto request = [&](int cb) {
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int q = 0; q < 2; ++q)
                next[c][q] = *reinterpret_cast<const v4f_u*>(hrow[q] + min(c0 + cb + c, chunks - 1) * 16 + 4 * kk);
    };
    rows_of(0);

    // the tile's parameters: 16 rows of 16 per quads
    AdamQuad aq[ROUNDS];
    unsigned at[ROUNDS];                             // (at most 2048 units of 4096 inputs)
    int slot[ROUNDS];                                // in fresh, or -1
    const int k_group = split * 64 * per;
#pragma unroll
    for (int i = 0; i < ROUNDS; ++i) {
        const int j = tid + i * FUSED_THREADS, r = j / (16 * per), c = 4 * (j - r * 16 * per);
        const bool live = r < units && k_group + c < d;
        at[i] = (unsigned)t.w0[hd] + (unsigned)((o0 + min(r, units - 1)) * d + min(k_group + c, d - 4));
        slot[i] = live ? r * LD + c : -1;
        aq[i].load_all(a, at[i]);
    }
    double norm;
    const double scale = adam_scale(a, red, norm), step = hd ? a.step_value : a.step_policy;
#pragma unroll
    for (int i = 0; i < ROUNDS; ++i) {
        AdamQuad& q = aq[i];
        if (i == REQUEST_AT) request(0);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int e = 0; e < 4; ++e) adam_element(a, scale, step, q.g[e], q.p[e], q.m[e], q.v[e]);
        if (slot[i] >= 0) {
            *reinterpret_cast<float4*>(&fresh[0][0] + slot[i]) = make_float4(q.p[0], q.p[1], q.p[2], q.p[3]);
            q.store(a, at[i], 4);
        }
    }
    __syncthreads();

    const int ncol = f.out_dim[0] + f.out_dim[1];
    const float* wrow = &fresh[lane & 15][range * 16 * per + 4 * kk];
    for (int bt = 0; bt < f.btiles; ++bt) {
        v4d acc[2] = {};
        for (int cb = 0; cb < max(nc, 1); cb += NC) {
            v4f_u x[NC][2];
#pragma unroll
            for (int c = 0; c < NC; ++c)
#pragma unroll
                for (int q = 0; q < 2; ++q) x[c][q] = next[c][q];
            if (cb + NC < nc) {
                request(cb + NC);
            } else if (bt + 1 < f.btiles) {
                rows_of(bt + 1);
                request(0);
            }
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                if (cb + c >= nc) break;
                const float4 wv = *reinterpret_cast<const float4*>(wrow + 16 * (cb + c));
                const float w[4] = {wv.x, wv.y, wv.z, wv.w};
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int q = 0; q < 2; ++q)
                        acc[q] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)x[c][q][e], (double)w[e], acc[q], 0, 0, 0);
            }
        }
        if (bt) __syncthreads();                     // the block before has been read
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int v = 0; v < 4; ++v) part[range][(half * 2 + q) * 4 + v][lane] = acc[q][v];
        __syncthreads();
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int qv = wave * 2 + u, b = bt * 64 + (qv >> 2) * 16 + 4 * (qv & 3) + kk, o = o0 + (lane & 15);
            if (b < f.B && o < f.out_dim[hd])
                f.z[((size_t)split * f.B + b) * ncol + (hd ? f.out_dim[0] : 0) + o] =
                    ((part[0][qv][lane] + part[1][qv][lane]) + part[2][qv][lane]) + part[3][qv][lane];
        }
    }
}

// ---- workspace ---------------------------------------------------------------------------------

struct PpoWs {
    size_t act_off[2][PPO_MAX_LAYERS];   // layer outputs [batch, dims[l+1]] fp64
    size_t delta_off[2][PPO_MAX_LAYERS]; // their deltas
    size_t z_off, grad_off, partial_off, scal_off, rows_off, total;
    int grad_waves;
    int grad_first[2][PPO_MAX_LAYERS];   // first wavefront of each layer's weight gradients
    int splits, btiles;                  // of the first layer's contraction
    bool tail;                           // both heads above their first layers fit one workgroup per sample
};

constexpr size_t PPO_ALIGN = 256;

PpoWs ppo_ws_layout(const Layout& L, int batch) {
    PpoWs W;
    memset(&W, 0, sizeof(W));
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t at = off;
        off += round_up_sz(bytes, PPO_ALIGN);
        return at;
    };
    size_t units = 0;
    for (int hd = 0; hd < 2; ++hd)
        for (int l = 0; l < L.head[hd].n; ++l) {
            W.act_off[hd][l] = take((size_t)batch * L.head[hd].dims[l + 1] * 8);
            W.delta_off[hd][l] = take((size_t)batch * L.head[hd].dims[l + 1] * 8);
            units += (size_t)L.head[hd].dims[l + 1];
        }
    W.tail = units <= TAIL_MAX_UNITS;
    const int ncol = L.head[0].dims[1] + L.head[1].dims[1];
    const int tiles = (L.head[0].dims[1] + 15) / 16 + (L.head[1].dims[1] + 15) / 16;
    W.btiles = (batch + 63) / 64;
    W.splits = first_layer_splits(tiles, W.btiles, L.head[0].dims[0]);
    W.z_off = W.tail ? take(first_layer_rows(tiles, batch, L.head[0].dims[0]) * ncol * 8) : 0;
    W.grad_off = take(L.n_params * 8);
    int nw = 0;
    for (int hd = 0; hd < 2; ++hd)
        for (int l = 0; l < L.head[hd].n; ++l) {
            W.grad_first[hd][l] = nw;
            nw += ((L.head[hd].dims[l + 1] + 15) / 16) * ((L.head[hd].dims[l] + 63) / 64);
        }
    W.grad_waves = nw;
    W.partial_off = take((size_t)nw * 8);
    W.scal_off = take(3 * 8);            // mean and scale of the advantages, total of the partial sums
    W.rows_off = take((size_t)4 * batch * 8);
    W.total = off;
    return W;
}

}  // namespace

}  // namespace brl

using namespace brl;

extern "C" {

size_t brl_ppo_param_count(const brl_ppo_config* cfg) {
    Layout L;
    if (make_layout(cfg, L) != BRL_OK) return 0;
    return L.n_params;
}

int brl_ppo_param_offsets(const brl_ppo_config* cfg, size_t* w_offsets, size_t* b_offsets) {
    Layout L;
    if (int rc = make_layout(cfg, L)) return rc;
    BRL_REQUIRE(w_offsets && b_offsets, "ppo_param_offsets: null pointer");
    int k = 0;
    for (int hd = 0; hd < 2; ++hd)
        for (int l = 0; l < L.head[hd].n; ++l, ++k) {
            w_offsets[k] = L.head[hd].w_off[l];
            b_offsets[k] = L.head[hd].b_off[l];
        }
    return BRL_OK;
}

size_t brl_ppo_workspace_bytes(const brl_ppo_config* cfg, int batch) {
    Layout L;
    if (batch < 1 || make_layout(cfg, L) != BRL_OK) return 0;
    return ppo_ws_layout(L, batch).total;
}

int ppo_gae(const float* rewards, const float* values, const float* dones, const float* last_value, int n_envs, int T,
            float gamma, float lam, float* adv, float* returns, void* stream) {
    BRL_REQUIRE(rewards && values && dones && last_value && adv && returns, "ppo_gae: null pointer");
    BRL_REQUIRE(n_envs >= 1 && T >= 1, "ppo_gae: n_envs = %d, T = %d", n_envs, T);
    BRL_REQUIRE(gamma >= 0.f && gamma <= 1.f && lam >= 0.f && lam <= 1.f, "ppo_gae: gamma and lambda must lie in [0, 1]");
    hipStream_t s = static_cast<hipStream_t>(stream);
    LaunchTimer tm(BRL_KC_OTHER, s);
    int shift = 0;                                                   // 2^shift threads per rollout
    while ((1 << shift) < GAE_THREADS && ((long)GAE_STRETCH << shift) < T) ++shift;
    const int rollouts = GAE_THREADS >> shift, per = (T - 1) / (1 << shift) + 1;
    const dim3 grid((unsigned)((n_envs - 1) / rollouts + 1));
    auto kernel = rollouts == 1 ? gae_kernel<8> : gae_kernel<-1>;
    static_assert(GAE_THREADS == 1 << 8, "the whole workgroup");
    hipLaunchKernelGGL(kernel, grid, dim3(GAE_THREADS), 0, s, rewards, values, dones, last_value, n_envs, T, per, shift, (double)gamma,
                       (double)lam, adv, returns);
    BRL_LAUNCH_CHECK("gae_kernel");
    return BRL_OK;
}

int ppo_head_update(const brl_ppo_config* cfg, float* params, float* adam_m, float* adam_v, long long* adam_step,
                    const float* h, const int32_t* actions, const float* logp_old, const float* adv, const float* returns,
                    int T, const int32_t* perm, int epochs, int batch, float* stats, void* workspace, size_t ws_bytes,
                    void* stream) {
    Layout L;
    if (int rc = make_layout(cfg, L)) return rc;
    BRL_REQUIRE(params && adam_m && adam_v && adam_step && h && actions && logp_old && adv && returns && perm && workspace,
                "ppo_head_update: null pointer");
    BRL_REQUIRE(T >= 1 && epochs >= 0 && batch >= 1 && batch <= T, "ppo_head_update: T = %d, epochs = %d, batch = %d", T,
                epochs, batch);
    BRL_REQUIRE(*adam_step >= 0, "ppo_head_update: negative step count");
    BRL_REQUIRE(!cfg->normalize_adv || batch >= 2, "ppo_head_update: advantage normalisation needs batch >= 2");
    BRL_REQUIRE(cfg->clip_eps >= 0.f && cfg->max_grad_norm > 0.f && cfg->adam_eps > 0.f && cfg->adam_b1 >= 0.f &&
                    cfg->adam_b1 < 1.f && cfg->adam_b2 >= 0.f && cfg->adam_b2 < 1.f && cfg->adv_eps >= 0.f,
                "ppo_head_update: bad hyper-parameter");
    const PpoWs W = ppo_ws_layout(L, batch);
    if (ws_bytes < W.total) {
        set_error("ppo_head_update: workspace %zu < %zu", ws_bytes, W.total);
        return BRL_ENOSPC;
    }
    hipStream_t s = static_cast<hipStream_t>(stream);
    char* base = static_cast<char*>(workspace);
    auto at = [&](size_t off) { return reinterpret_cast<double*>(base + off); };
    double* grads = at(W.grad_off);
    double* partial = at(W.partial_off);
    double* row_terms = at(W.rows_off);
    const int A = L.head[0].dims[L.head[0].n];
    const int steps_per_epoch = T / batch;
    LaunchTimer tm(BRL_KC_OTHER, s);

    // what does not change from step to step
    GradArgs ga;
    memset(&ga, 0, sizeof(ga));
    ga.waves = W.grad_waves; ga.h = h; ga.B = batch; ga.T = T; ga.partial = partial;
    for (int hd = 0; hd < 2; ++hd) {
        const HeadShape& H = L.head[hd];
        for (int l = 0; l < H.n; ++l) {
            GradProblem& G = ga.p[ga.n++];
            G.delta = at(W.delta_off[hd][l]);
            G.in64 = l == 0 ? nullptr : at(W.act_off[hd][l - 1]);
            G.gW = grads + H.w_off[l]; G.gb = grads + H.b_off[l];
            G.in_dim = H.dims[l]; G.out_dim = H.dims[l + 1]; G.ichunks = (H.dims[l] + 63) / 64;
            G.first = W.grad_first[hd][l];
        }
    }
    AdamArgs aa;
    memset(&aa, 0, sizeof(aa));
    aa.p = params; aa.m = adam_m; aa.v = adam_v; aa.g = grads; aa.n = L.n_params; aa.n_policy = L.n_policy;
    const bool norm_launch = W.grad_waves > ADAM_OWN_NORM;
    double* total = at(W.scal_off) + 2;
    aa.partial = norm_launch ? total : partial; aa.n_partials = norm_launch ? 1 : W.grad_waves; aa.B = batch;
    aa.max_norm = (double)cfg->max_grad_norm;
    aa.b1 = (double)cfg->adam_b1; aa.b2 = (double)cfg->adam_b2; aa.eps = (double)cfg->adam_eps; aa.ent_coef = (double)cfg->ent_coef;
    aa.row_terms = row_terms;
    FirstArgs fl;
    TailArgs ta;
    memset(&fl, 0, sizeof(fl));
    memset(&ta, 0, sizeof(ta));
    if (W.tail) {
        fl.h = h; fl.B = batch; fl.T = T; fl.d = L.head[0].dims[0]; fl.splits = W.splits; fl.btiles = W.btiles;
        fl.z = at(W.z_off); fl.adv = adv; fl.adv_eps = (double)cfg->adv_eps; fl.normalize_adv = cfg->normalize_adv;
        fl.scal = at(W.scal_off);
        ta.z = fl.z; ta.splits = W.splits; ta.B = batch; ta.A = A; ta.T = T; ta.act = cfg->act;
        for (int hd = 0; hd < 2; ++hd) {
            const HeadShape& H = L.head[hd];
            fl.W[hd] = params + H.w_off[0]; fl.out_dim[hd] = H.dims[1]; fl.tiles[hd] = (H.dims[1] + 15) / 16;
            ta.n[hd] = H.n;
            for (int l = 0; l <= H.n; ++l) ta.dims[hd][l] = H.dims[l];
            for (int l = 0; l < H.n; ++l) {
                ta.W[hd][l] = params + H.w_off[l]; ta.bias[hd][l] = params + H.b_off[l];
                ta.acts[hd][l] = at(W.act_off[hd][l]); ta.delta[hd][l] = at(W.delta_off[hd][l]);
            }
        }
        ta.actions = actions; ta.logp_old = logp_old; ta.adv = adv; ta.returns = returns; ta.scal = fl.scal;
        ta.clip_eps = (double)cfg->clip_eps; ta.ent_coef = (double)cfg->ent_coef; ta.row_terms = row_terms;
    }
    // An update's Adam and the next first layer in one launch.  A workgroup then takes all samples of its tile, so past 64 of
    // them only where the tiles alone fill the chip, and up to 256: the tiles of 64 samples that two launches spread evenly are
    // then more than the launch is worth.  A step in us, two launches / one: 64 samples, hidden 256, 1024 inputs 28.5 / 26.4, 2560
    // inputs 37.6 / 34.9, hidden 64, 2560 inputs 28.8 / 26.1; 256 samples, hidden 256, 2560 inputs 68.3 / 65.5, hidden 64, 2560
    // inputs 42.8 / 48.9; hidden 256, 2560 inputs, 512 samples 106.6 / 107.4, 1024 samples 186.4 / 194.4, two hidden layers of 320
    // 321 / 351.  Rows of more than 3072 inputs spill (64 samples, hidden 256, 3200 inputs: 40.7 / 41.2).
    const int range_chunks = first_layer_range_chunks(L.head[0].dims[0]), tile_blocks = (fl.tiles[0] + fl.tiles[1]) * W.splits;
    const bool fused = W.tail && !norm_launch && fl.d % 16 == 0 && range_chunks <= FUSED_MAX_CHUNKS &&
                       W.splits == first_layer_groups(fl.d) && (W.btiles == 1 || (W.btiles <= 4 && tile_blocks >= 256));
    FusedArgs fu;
    memset(&fu, 0, sizeof(fu));
    if (fused) {
        fu.f = fl;
        fu.tile_blocks = tile_blocks;
        for (int hd = 0; hd < 2; ++hd) {
            const size_t end = hd ? L.n_params : L.n_policy, n_first = (size_t)fl.out_dim[hd] * fl.d;
            fu.w0[hd] = L.head[hd].w_off[0];
            fu.rest0[hd] = fu.w0[hd] + n_first;
            fu.rest_n[hd] = end - fu.rest0[hd];
            fu.rest_blocks[hd] = (int)((fu.rest_n[hd] + FUSED_THREADS * ADAM_PER_THREAD - 1) / (FUSED_THREADS * ADAM_PER_THREAD));
        }
    }
    bool fused_ahead = false;                                        // this mini-batch's first layer ran with the last update
    const int depth = L.head[0].n > L.head[1].n ? L.head[0].n : L.head[1].n;
    long long step = *adam_step;
    for (int e = 0; e < epochs; ++e) {
        for (int mb = 0; mb < steps_per_epoch; ++mb) {
            const int32_t* rows = perm + (size_t)e * T + (size_t)mb * batch;
            if (W.tail) {
                ta.rows = rows;
                if (!fused_ahead) {                                  // (else the last update's launch has done it)
                    fl.rows = rows;
                    const unsigned blocks = (unsigned)((fl.tiles[0] + fl.tiles[1]) * W.splits * W.btiles) + 1;   // + the advantages' scale
                    if (W.splits == 1) hipLaunchKernelGGL(ppo_first_layer_kernel<true>, dim3(blocks), dim3(256), 0, s, fl);
                    else hipLaunchKernelGGL(ppo_first_layer_kernel<false>, dim3(blocks), dim3(256), 0, s, fl);
                }
                hipLaunchKernelGGL(ppo_tail_kernel, dim3(batch), dim3(TAIL_THREADS), 0, s, ta);
            } else {
                // forward: level l of both heads in one launch
                for (int l = 0; l < depth; ++l) {
                    FwdArgs fa;
                    memset(&fa, 0, sizeof(fa));
                    fa.h = h; fa.rows = rows; fa.B = batch; fa.act = cfg->act; fa.T = T;
                    unsigned blocks = 0;
                    for (int hd = 0; hd < 2; ++hd) {
                        const HeadShape& H = L.head[hd];
                        if (l >= H.n) continue;
                        FwdProblem& P = fa.p[fa.n++];
                        P.in64 = l == 0 ? nullptr : at(W.act_off[hd][l - 1]);
                        P.W = params + H.w_off[l];
                        P.bias = params + H.b_off[l];
                        P.out = at(W.act_off[hd][l]);
                        P.in_dim = H.dims[l]; P.out_dim = H.dims[l + 1]; P.last = l == H.n - 1 ? 1 : 0;
                        P.blocks = (unsigned)(((batch + FB - 1) / FB) * ((H.dims[l + 1] + FO - 1) / FO));
                        blocks += P.blocks;
                    }
                    hipLaunchKernelGGL(ppo_forward_kernel, dim3(blocks), dim3(256), 0, s, fa);
                }
                // gradients at the outputs
                LossArgs la;
                la.logits = at(W.act_off[0][L.head[0].n - 1]);
                la.v = at(W.act_off[1][L.head[1].n - 1]);
                la.rows = rows; la.actions = actions; la.logp_old = logp_old; la.adv = adv; la.returns = returns;
                la.B = batch; la.A = A; la.T = T;
                la.clip_eps = (double)cfg->clip_eps; la.ent_coef = (double)cfg->ent_coef; la.adv_eps = (double)cfg->adv_eps;
                la.normalize_adv = cfg->normalize_adv;
                la.dlogits = at(W.delta_off[0][L.head[0].n - 1]);
                la.dv = at(W.delta_off[1][L.head[1].n - 1]);
                la.row_terms = row_terms;
                hipLaunchKernelGGL(ppo_loss_kernel, dim3(1), dim3(256), 0, s, la);
                // backward: the same distance from the output of both heads in one launch
                for (int t = 0; t < depth - 1; ++t) {
                    DeltaArgs da;
                    memset(&da, 0, sizeof(da));
                    da.B = batch; da.act = cfg->act;
                    unsigned blocks = 0;
                    for (int hd = 0; hd < 2; ++hd) {
                        const HeadShape& H = L.head[hd];
                        const int l = H.n - 1 - t;
                        if (l < 1) continue;
                        DeltaProblem& D = da.p[da.n++];
                        D.delta = at(W.delta_off[hd][l]); D.W = params + H.w_off[l]; D.a_prev = at(W.act_off[hd][l - 1]);
                        D.delta_prev = at(W.delta_off[hd][l - 1]);
                        D.in_dim = H.dims[l]; D.out_dim = H.dims[l + 1];
                        D.blocks = (unsigned)(((size_t)batch * H.dims[l] + 255) / 256);
                        blocks += D.blocks;
                    }
                    hipLaunchKernelGGL(ppo_delta_kernel, dim3(blocks), dim3(256), 0, s, da);
                }
            }
            ga.rows = rows;
            hipLaunchKernelGGL(ppo_weight_grad_kernel, dim3((unsigned)((W.grad_waves + 3) / 4)), dim3(256), 0, s, ga);
            if (norm_launch) hipLaunchKernelGGL(ppo_norm_kernel, dim3(1), dim3(NORM_THREADS), 0, s, partial, W.grad_waves, total);
            ++step;
            const double c1 = 1.0 - pow((double)cfg->adam_b1, (double)step);
            aa.step_policy = (double)cfg->lr_policy / c1;
            aa.step_value = (double)cfg->lr_value / c1;
            aa.inv_c2 = 1.0 / (1.0 - pow((double)cfg->adam_b2, (double)step));
            aa.stats = stats ? stats + ((size_t)e * steps_per_epoch + mb) * 5 : nullptr;
            const bool last = mb + 1 == steps_per_epoch && e + 1 == epochs;
            fused_ahead = fused && !last;
            if (fused_ahead) {
                fu.a = aa;
                fu.f.rows = mb + 1 < steps_per_epoch ? rows + batch : perm + (size_t)(e + 1) * T;
                const unsigned blocks = (unsigned)(fu.tile_blocks + fu.rest_blocks[0] + fu.rest_blocks[1]) + 1;   // + the advantages' scale
                auto kernel = range_chunks <= 2 ? ppo_adam_first_kernel<1> : range_chunks <= 4 ? ppo_adam_first_kernel<2> : ppo_adam_first_kernel<3>;
                hipLaunchKernelGGL(kernel, dim3(blocks), dim3(FUSED_THREADS), 0, s, fu);
                continue;
            }
            hipLaunchKernelGGL(ppo_adam_kernel, dim3((unsigned)((L.n_params + 256 * ADAM_PER_THREAD - 1) / (256 * ADAM_PER_THREAD))),
                               dim3(256), 0, s, aa);
        }
    }
    BRL_LAUNCH_CHECK("ppo_head_update");
    *adam_step = step;
    return BRL_OK;
}

}  // extern "C"
