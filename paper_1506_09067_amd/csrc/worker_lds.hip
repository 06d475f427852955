// Per-sample CHAOS training worker for any layer list whose per-sample state
// fits in LDS and that has no fused kernel of its own.
//
// Same scheme as the generic worker kernel (worker.hip): one workgroup of eight
// wavefronts is one worker and owns one sample at a time; per layer the partial
// derivatives of the layer below come from the layer's weights before the
// layer's gradient is pushed (Sections III-A.1 to III-A.3).  What bounds that
// kernel is latency: scalar loops whose every operand comes from the caches.
// Here activations, deltas and errors stay in LDS and the convolutions run on
// the fp32 matrix instructions (16x16x4), as matrix products whose operands are
// gathered by tables of offsets:
//   forward          rows = output positions, columns = maps, K = (map, kernel)
//   backward data    rows = input positions, columns = input maps, K = (map,
//                    kernel) over the deltas in a zero frame (gathered, no scatter)
//   weight gradient  rows = maps, columns = (map, kernel), K = output positions
// Every reduction has a fixed order, so one worker is sequential SGD bit for bit.
// A net of conv 16, 32, 48 and two FC layers on 32x32 inputs (68,826 weights):
// 1,495 -> 130 us a sample of one worker, an epoch of 1,044 samples by 256
// workers 7.73 -> 0.82 ms against the worker with its state in device memory.
#include "batch.h"
#include "chaos_internal.h"
#include "device_common.h"

#include <algorithm>

namespace chaos {
namespace {

constexpr int NT = 512, NW = 8;

// One 16x16x4 product step of MT row tiles against one column tile.
template <int MT>
__device__ __forceinline__ void step(const float (&a)[MT], float b, f4 (&acc)[MT]) {
#pragma unroll
    for (int i = 0; i < MT; ++i) acc[i] = mfma(a[i], b, acc[i]);
}

// Fewer jobs than half the wavefronts: each job's K is split over `parts`
// wavefronts (in multiples of four), whose partial tiles are added in order
// through red [wavefront][MT][lane][4].
struct KSplit {
    int parts, job0, stride, k0, k1;
};
__device__ __forceinline__ KSplit split_k(int jobs, int wave, int Kt) {
    KSplit s;
    s.parts = jobs <= NW / 2 ? NW / jobs : 1;
    if (s.parts == 1) return KSplit{1, wave, NW, 0, Kt};
    const int part = wave % s.parts, per = ((Kt + 3) / 4 + s.parts - 1) / s.parts * 4;
    s.job0 = wave / s.parts;
    s.stride = NW;
    s.k0 = part * per;
    s.k1 = s.k0 + per < Kt ? s.k0 + per : Kt;
    return s;
}
// sums the parts of every job: dst[col * cs + row] for row < rows, col < cols
template <int MT>
__device__ __forceinline__ void add_parts(const float *red, int jobs, int parts, int RG, int rows, int cols, int cs,
                                          float *dst) {
    for (int t = threadIdx.x; t < jobs * MT * 64; t += NT) {
        const int lane = t & 63, it = t >> 6, job = it / MT, i = it - job * MT;
        const float *src = red + ((job * parts * MT + i) * 64 + lane) * 4;
        f4 v = *(const f4 *)src;
        for (int q = 1; q < parts; ++q) v += *(const f4 *)(src + q * MT * 256);
        const int ct = job / RG, rg = job - ct * RG, col = 16 * ct + (lane & 15);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int row = 16 * (MT * rg + i) + 4 * (lane >> 4) + r;
            if (row < rows && col < cols) dst[col * cs + row] = v[r];
        }
    }
}

// z[o][p] = sum_k W[o][k] in[pos(p) + koff[k]]  (no bias, no activation)
__device__ __forceinline__ void conv_z(const LdsStage &g, const float *in, const int *koff, const float *W, float *z,
                                       float *red) {
    constexpr int MT = 4;
    const int lane = threadIdx.x & 63, lr = lane & 15, lg = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int P = g.Ho * g.Wo, Kt = g.C * g.K * g.K, RG = (P + 16 * MT - 1) / (16 * MT), CT = (g.O + 15) / 16;
    // sixteen K steps' weights are requested together, a batch ahead: a weight
    // that a push touched since it was last read comes from memory
    constexpr int D = 16;
    float wa[D], wb[D];
    int last = -1;
    const KSplit sp = split_k(RG * CT, wave, Kt);
    for (int job = sp.job0; job < RG * CT; job += sp.stride) {
        const int ct = job / RG, rg = job - ct * RG;
        f4 acc[MT];
        int base[MT];
#pragma unroll
        for (int i = 0; i < MT; ++i) {
            const int p = 16 * (MT * rg + i) + lr, pc = p < P ? p : 0, y = pc / g.Wo;
            base[i] = y * g.W + pc - y * g.Wo;
            acc[i] = f4{0.f, 0.f, 0.f, 0.f};
        }
        const int o = 16 * ct + lr;
        const float *w = W + g.w_off + (o < g.O ? o : 0) * Kt;
        auto load = [&](float (&b)[D], int k0) {
#pragma unroll
            for (int d = 0; d < D; ++d) {
                const int k = k0 + 4 * d + lg;
                b[d] = w[k < sp.k1 ? k : 0];
            }
        };
        auto run = [&](const float (&b)[D], int k0) {
#pragma unroll
            for (int d0 = 0; d0 < D; d0 += 4) {
                if (k0 + 4 * d0 >= sp.k1) continue;
                float a[4][MT];
#pragma unroll
                for (int d = 0; d < 4; ++d) {
                    const int k = k0 + 4 * (d0 + d) + lg, ko = koff[k < sp.k1 ? k : 0];
#pragma unroll
                    for (int i = 0; i < MT; ++i) a[d][i] = (k < sp.k1) ? in[base[i] + ko] : 0.0f;
                }
#pragma unroll
                for (int d = 0; d < 4; ++d)
                    if (k0 + 4 * (d0 + d) < sp.k1) step<MT>(a[d], (k0 + 4 * (d0 + d) + lg < sp.k1) ? b[d0 + d] : 0.0f, acc);
            }
        };
        // (a short kernel's weights stay in registers over the jobs of a column tile)
        if (ct != last || sp.k1 - sp.k0 > 4 * D) load(wa, sp.k0);
        last = ct;
        for (int k0 = sp.k0; k0 < sp.k1; k0 += 8 * D) {
            if (k0 + 4 * D < sp.k1) load(wb, k0 + 4 * D);
            run(wa, k0);
            if (k0 + 4 * D < sp.k1) {
                if (k0 + 8 * D < sp.k1) load(wa, k0 + 8 * D);
                run(wb, k0 + 4 * D);
            }
        }
        if (sp.parts > 1) {
#pragma unroll
            for (int i = 0; i < MT; ++i) *(f4 *)(red + ((wave * MT + i) * 64 + lane) * 4) = acc[i];
        } else if (o < g.O) {
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int p = 16 * (MT * rg + i) + 4 * lg + r;
                    if (p < P) z[o * P + p] = acc[i][r];
                }
        }
    }
    if (sp.parts > 1) {
        __syncthreads();
        add_parts<MT>(red, RG * CT, sp.parts, RG, P, g.O, P, z);
    }
}

// y = f(bias + max over each window of z); the first maximum wins (f is
// strictly increasing)
__device__ __forceinline__ void pool_act(const LdsStage &g, const float *z, const float *W, float *y, unsigned char *arg) {
    const int Pp = g.Hp * g.Wp, P = g.Ho * g.Wo;
    for (int t = threadIdx.x; t < g.O * Pp; t += NT) {
        const int o = t / Pp, q = t - o * Pp, py = q / g.Wp, px = q - py * g.Wp;
        const float *zo = z + o * P + py * g.p * g.Wo + px * g.p;
        float m = zo[0];
        int ag = 0;
        for (int u = 0; u < g.p; ++u)
            for (int v = 0; v < g.p; ++v) {
                const float c = zo[u * g.Wo + v];
                if (c > m) { m = c; ag = u * g.p + v; }
            }
        y[t] = act_y(m + W[g.b_off + o]);
        if (g.p > 1) arg[t] = (unsigned char)ag;
    }
}

// deltas of the conv outputs from the errors of the pooled outputs: d[o][PP],
// inside a frame of `fr` zeros
__device__ __forceinline__ void conv_delta(const LdsStage &g, int fr, const float *e, const float *y, const unsigned char *arg,
                           float *d) {
    const int Pp = g.Hp * g.Wp, PW = g.Wo + 2 * fr, PP = (g.Ho + 2 * fr) * PW;
    for (int t = threadIdx.x; t < g.O * PP; t += NT) d[t] = 0.0f;
    __syncthreads();
    for (int t = threadIdx.x; t < g.O * Pp; t += NT) {
        const int o = t / Pp, q = t - o * Pp, py = q / g.Wp, px = q - py * g.Wp;
        const int w = g.p > 1 ? arg[t] : 0, u = w / g.p, v = w - u * g.p;
        d[o * PP + (py * g.p + u + fr) * PW + px * g.p + v + fr] = e[t] * dact_from_y(y[t]);
    }
}

// e_in[c][q] = sum_{o,u,v} W[o][c][u][v] d[o][q - (u,v)], over the framed deltas
__device__ __forceinline__ void conv_back(const LdsStage &g, const float *d, const float *W, float *e_in,
                                          float *red) {
    constexpr int MT = 4;
    const int lane = threadIdx.x & 63, lr = lane & 15, lg = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int HW = g.H * g.W, KK = g.K * g.K, Kt = g.O * KK, RG = (HW + 16 * MT - 1) / (16 * MT), CT = (g.C + 15) / 16;
    const int PW = g.Wo + 2 * (g.K - 1), PP = (g.Ho + 2 * (g.K - 1)) * PW;
    const KSplit sp = split_k(RG * CT, wave, Kt);
    for (int job = sp.job0; job < RG * CT; job += sp.stride) {
        const int ct = job / RG, rg = job - ct * RG;
        f4 acc[MT];
        int base[MT];
#pragma unroll
        for (int i = 0; i < MT; ++i) {
            const int q = 16 * (MT * rg + i) + lr, qc = q < HW ? q : 0, y = qc / g.W;
            base[i] = y * PW + qc - y * g.W;  // d at (y + u, x + v) meets the flipped kernel
            acc[i] = f4{0.f, 0.f, 0.f, 0.f};
        }
        const int c = 16 * ct + lr;
        const float *w = W + g.w_off + (c < g.C ? c : 0) * KK;
        constexpr int D = 16;
        int k = sp.k0 + lg, o = k / KK, uv = k - o * KK;  // k = o KK + uv
        float wa[D], wb[D];
        int ka[D], kb[D];
        auto load = [&](float (&b)[D], int (&ko)[D]) {
#pragma unroll
            for (int s = 0; s < D; ++s) {
                const bool in = k < sp.k1;
                const int u = uv / g.K;
                ko[s] = in ? o * PP + u * PW + uv - u * g.K : -1;
                b[s] = w[in ? o * g.C * KK + KK - 1 - uv : 0];
                k += 4;
                uv += 4;
                while (uv >= KK) { uv -= KK; ++o; }
            }
        };
        auto run = [&](const float (&b)[D], const int (&ko)[D], int k0) {
#pragma unroll
            for (int s0 = 0; s0 < D; s0 += 4) {
                if (k0 + 4 * s0 >= sp.k1) continue;
                float a[4][MT];
#pragma unroll
                for (int s = 0; s < 4; ++s)
#pragma unroll
                    for (int i = 0; i < MT; ++i) a[s][i] = (ko[s0 + s] >= 0) ? d[base[i] + ko[s0 + s]] : 0.0f;
#pragma unroll
                for (int s = 0; s < 4; ++s)
                    if (k0 + 4 * (s0 + s) < sp.k1) step<MT>(a[s], ko[s0 + s] >= 0 ? b[s0 + s] : 0.0f, acc);
            }
        };
        load(wa, ka);
        for (int k0 = sp.k0; k0 < sp.k1; k0 += 8 * D) {
            if (k0 + 4 * D < sp.k1) load(wb, kb);
            run(wa, ka, k0);
            if (k0 + 4 * D < sp.k1) {
                if (k0 + 8 * D < sp.k1) load(wa, ka);
                run(wb, kb, k0 + 4 * D);
            }
        }
        if (sp.parts > 1) {
#pragma unroll
            for (int i = 0; i < MT; ++i) *(f4 *)(red + ((wave * MT + i) * 64 + lane) * 4) = acc[i];
        } else if (c < g.C) {
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int q = 16 * (MT * rg + i) + 4 * lg + r;
                    if (q < HW) e_in[c * HW + q] = acc[i][r];
                }
        }
    }
    if (sp.parts > 1) {
        __syncthreads();
        add_parts<MT>(red, RG * CT, sp.parts, RG, HW, g.C, HW, e_in);
    }
}

// G[o][k] = sum_p d[o][p] in[pos(p) + koff[k]], pushed.  Four column tiles a job;
// with fewer jobs than half the wavefronts each takes an eighth of the positions
// of all of them and the eighths are added in order through `red`.
__device__ __forceinline__ void conv_wgrad(const LdsStage &g, int fr, const float *in, const int *koff, const float *d, float *red,
                           const Push &push) {
    constexpr int CB = 4;
    const int lane = threadIdx.x & 63, lr = lane & 15, lg = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int P = g.Ho * g.Wo, Kt = g.C * g.K * g.K, PW = g.Wo + 2 * fr, PP = (g.Ho + 2 * fr) * PW;
    const int RT = (g.O + 15) / 16, CT = (Kt + 15) / 16, CGn = (CT + CB - 1) / CB, jobs = RT * CGn;
    const bool split = jobs < NW / 2;
    const int steps = (P + 3) / 4, per = split ? (steps + NW - 1) / NW : steps;
    const int t0 = split ? wave * per : 0, t1 = (t0 + per < steps) ? t0 + per : steps;
    for (int job = split ? 0 : wave; job < jobs; job += split ? 1 : NW) {
        const int rt = job / CGn, cg = job - rt * CGn;
        const int o = 16 * rt + lr;
        const float *dr = d + (o < g.O ? o : 0) * PP + fr * PW + fr;
        int ko[CB];
#pragma unroll
        for (int j = 0; j < CB; ++j) {
            const int k = 16 * (CB * cg + j) + lr;
            ko[j] = koff[k < Kt ? k : 0];
        }
        f4 acc[CB];
#pragma unroll
        for (int j = 0; j < CB; ++j) acc[j] = f4{0.f, 0.f, 0.f, 0.f};
        int p = 4 * t0 + lg, y = p / g.Wo, x = p - y * g.Wo;
        constexpr int U = 4;
        for (int t = t0; t < t1; t += U) {
            float a[U], b[U][CB];
#pragma unroll
            for (int s = 0; s < U; ++s) {
                const bool ok = t + s < t1 && p < P;  // past the end: a zero times the first position
                const int da = ok ? y * PW + x : 0, ia = ok ? y * g.W + x : 0;
                a[s] = ok ? dr[da] : 0.0f;
#pragma unroll
                for (int j = 0; j < CB; ++j) b[s][j] = ok ? in[ia + ko[j]] : 0.0f;
                p += 4;
                x += 4;
                while (x >= g.Wo) { x -= g.Wo; ++y; }
            }
#pragma unroll
            for (int s = 0; s < U; ++s)
                if (t + s < t1) {
#pragma unroll
                    for (int j = 0; j < CB; ++j) acc[j] = mfma(a[s], b[s][j], acc[j]);
                }
        }
        if (split) {
#pragma unroll
            for (int j = 0; j < CB; ++j) *(f4 *)(red + ((wave * CB + j) * 64 + lane) * 4) = acc[j];
            __syncthreads();
            // column tile j of the job on wavefront j
            const float *r0 = red + ((wave < CB ? wave : 0) * 64 + lane) * 4;
            f4 s = *(const f4 *)r0;
#pragma unroll
            for (int q = 1; q < NW; ++q) s += *(const f4 *)(r0 + q * CB * 256);
            const int k = 16 * (CB * cg + wave) + lr;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int oo = 16 * rt + 4 * lg + r;
                if (wave < CB && oo < g.O && k < Kt) push(g.w_off + oo * Kt + k, s[r]);
            }
            __syncthreads();
        } else {
#pragma unroll
            for (int j = 0; j < CB; ++j) {
                const int k = 16 * (CB * cg + j) + lr;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int oo = 16 * rt + 4 * lg + r;
                    if (oo < g.O && k < Kt) push(g.w_off + oo * Kt + k, acc[j][r]);
                }
            }
        }
    }
    // biases
    const int lanes = threadIdx.x & 63;
    for (int o = wave; o < g.O; o += NW) {
        float s = 0.0f;
        for (int p = lanes; p < PP; p += 64) s += d[o * PP + p];  // the frame is zeros
        s = wave_sum(s);
        if (lanes == 0) push(g.b_off + o, s);
    }
}

// y = f(b + W x): four neurons a wavefront at a time, lanes over the inputs
__device__ __forceinline__ void fc_forward(const LdsStage &g, const float *in, const float *W, float *y) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const float *w = W + g.w_off;
    for (int j0 = 4 * wave; j0 < g.O; j0 += 4 * NW) {
        float s[4] = {0.f, 0.f, 0.f, 0.f};
        int row[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) row[q] = (j0 + q < g.O ? j0 + q : g.O - 1) * g.C;
        // 256 inputs of the four rows at a time, the next 256 requested meanwhile
        float wa[4][4], wb[4][4];
        auto load = [&](float (&b)[4][4], int i0) {
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const int i = i0 + lane + 64 * c;
#pragma unroll
                for (int q = 0; q < 4; ++q) b[q][c] = w[row[q] + (i < g.C ? i : 0)];
            }
        };
        auto run = [&](const float (&b)[4][4], int i0) {
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const int i = i0 + lane + 64 * c;
                const float x = i < g.C ? in[i] : 0.0f;
#pragma unroll
                for (int q = 0; q < 4; ++q) s[q] = fmaf(i < g.C ? b[q][c] : 0.0f, x, s[q]);
            }
        };
        load(wa, 0);
        for (int i0 = 0; i0 < g.C; i0 += 512) {
            load(wb, i0 + 256);
            run(wa, i0);
            if (i0 + 256 < g.C) {
                load(wa, i0 + 512);
                run(wb, i0 + 256);
            }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float t = wave_sum(s[q]);
            if (lane == 0 && j0 + q < g.O) y[j0 + q] = act_y(t + W[g.b_off + j0 + q]);
        }
    }
}

template <int MODE>
__global__ void __launch_bounds__(NT, 2) worker_lds_kernel(LdsPlan pl, WorkArgs a) {
    extern __shared__ __align__(16) float lds[];
    __shared__ int64_t s_idx;
    const int tid = threadIdx.x;
    const float *W = a.params;
    float *x = lds, *z = lds + pl.z_off, *red = lds + pl.red_off;
    for (int l = 0; l < pl.n; ++l) {
        const LdsStage &g = pl.s[l];
        if (g.fc) continue;
        int *koff = (int *)(lds + g.tab_off);
        const int KK = g.K * g.K;
        for (int k = tid; k < g.C * KK; k += NT) {
            const int c = k / KK, uv = k - c * KK, u = uv / g.K;
            koff[k] = c * g.H * g.W + u * g.W + uv - u * g.K;
        }
    }
    for (;;) {
        // as the generic worker: every wavefront waits for its own pushes, the
        // sample then sees every push completed so far (worker.hip)
        wait_vector_memory();
        if (tid == 0) s_idx = atomicAdd(a.counter, 1);
        __syncthreads();
        const int64_t idx = s_idx;
        if (idx >= a.n) break;
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        if (a.claims && tid == 0) atomicAdd(a.claims + idx, 1);
        for (int i = tid; i < pl.in_size; i += NT) x[i] = a.x[idx * pl.in_size + i];
        const int label = a.labels[idx];
        __syncthreads();
        const float *in = x;
        for (int l = 0; l < pl.n; ++l) {
            const LdsStage &g = pl.s[l];
            float *y = lds + g.y_off;
            if (g.fc) {
                fc_forward(g, in, W, y);
            } else {
                conv_z(g, in, (const int *)(lds + g.tab_off), W, z, red);
                __syncthreads();
                pool_act(g, z, W, y, (unsigned char *)(lds + g.arg_off));
            }
            __syncthreads();
            in = y;
        }
        // output error
        float *e = lds + pl.e_off[0], *ep = lds + pl.e_off[1];
        if (tid < 64) {
            float part = 0.0f;
            for (int k = tid; k < pl.n_out; k += 64) {
                const float dk = in[k] - (k == label ? 1.0f : 0.0f);
                e[k] = dk;
                part = fmaf(dk, dk, part);
            }
            part = wave_sum(part);
            if (tid == 0 && a.loss) a.loss[idx] = 0.5f * part;
        }
        __syncthreads();
        Push push;
        push.mode = MODE;
        push.params = a.params;
        push.neg_lr = -a.lr;
        push.each = nullptr;
        push.part = nullptr;
        for (int l = pl.n - 1; l >= 0; --l) {
            const LdsStage &g = pl.s[l];
            const float *y = lds + g.y_off, *lin = l ? lds + pl.s[l - 1].y_off : x;
            if (g.fc) {
                for (int j = tid; j < g.O; j += NT) e[j] *= dact_from_y(y[j]);
                __syncthreads();
                if (l) {
                    const float *w = W + g.w_off;
                    // four inputs a thread, eight rows of each in flight
                    for (int i0 = tid; i0 < g.C; i0 += 4 * NT) {
                        float s[4] = {0.f, 0.f, 0.f, 0.f};
                        int i[4];
#pragma unroll
                        for (int q = 0; q < 4; ++q) i[q] = i0 + q * NT < g.C ? i0 + q * NT : i0;
#pragma unroll 8
                        for (int j = 0; j < g.O; ++j)
#pragma unroll
                            for (int q = 0; q < 4; ++q) s[q] = fmaf(w[j * g.C + i[q]], e[j], s[q]);
#pragma unroll
                        for (int q = 0; q < 4; ++q)
                            if (i0 + q * NT < g.C) ep[i0 + q * NT] = s[q];
                    }
                    __syncthreads();  // the layer's weights are no longer read for this sample
                }
                for (int j = tid >> 6; j < g.O; j += NW) {
                    const float dj = e[j];
                    for (int i = tid & 63; i < g.C; i += 64) push(g.w_off + j * g.C + i, dj * lin[i]);
                }
                for (int j = tid; j < g.O; j += NT) push(g.b_off + j, e[j]);
            } else {
                const int fr = l ? g.K - 1 : 0;
                conv_delta(g, fr, e, y, (const unsigned char *)(lds + g.arg_off), z);
                __syncthreads();
                if (l) {
                    conv_back(g, z, W, ep, red);
                    __syncthreads();
                }
                conv_wgrad(g, fr, lin, (const int *)(lds + g.tab_off), z, red, push);
            }
            __syncthreads();
            float *t = e;
            e = ep;
            ep = t;
        }
    }
}

} // namespace

bool worker_lds_plan(const Net &net, LdsPlan &pl) {
    pl = LdsPlan{};
    int64_t off = (net.in_size + 3) / 4 * 4, z = 0, e = net.n_out;
    for (int l = 0; l < net.n_layers; ++l) {
        const Layer &ly = net.L[l];
        if (ly.kind == kPool) return false;  // not right after a conv or FC layer
        LdsStage &g = pl.s[pl.n];
        g.fc = ly.kind == kFc;
        g.C = g.fc ? ly.nin : ly.cin;
        g.H = g.fc ? 1 : ly.hin;
        g.W = g.fc ? 1 : ly.win;
        g.O = ly.cout;
        g.K = g.fc ? 1 : ly.k;
        g.Ho = ly.hout;
        g.Wo = ly.wout;
        g.p = 1;
        g.Hp = g.Ho;
        g.Wp = g.Wo;
        g.w_off = ly.w_off;
        g.b_off = ly.b_off;
        if (l + 1 < net.n_layers && net.L[l + 1].kind == kPool) {
            ++l;
            if (g.fc || net.L[l].k > 16) return false;
            g.p = net.L[l].k;
            g.Hp = net.L[l].hout;
            g.Wp = net.L[l].wout;
        }
        const int64_t nout = (int64_t)g.O * g.Hp * g.Wp, fr = pl.n ? g.K - 1 : 0;
        if (nout > (1 << 16) || g.C > (1 << 20)) return false;
        g.y_off = (int)off;
        off += (nout + 3) / 4 * 4;
        if (!g.fc) {
            if (g.p > 1) {
                g.arg_off = (int)off;
                off += (nout + 15) / 16 * 4;
            }
            g.tab_off = (int)off;
            off += ((int64_t)g.C * g.K * g.K + 3) / 4 * 4;
            z = std::max(z, (int64_t)g.O * (g.Ho + 2 * fr) * (g.Wo + 2 * fr));
        }
        e = std::max(e, nout);
        if (pl.n) e = std::max(e, (int64_t)g.C * g.H * g.W);
        if (off > (160 << 8)) return false;
        ++pl.n;
    }
    pl.in_size = net.in_size;
    pl.n_out = net.n_out;
    pl.z_off = (int)off;
    off += (z + 3) / 4 * 4;
    pl.red_off = (int)off;
    off += NW * 4 * 256;
    for (int q = 0; q < 2; ++q) {
        pl.e_off[q] = (int)off;
        off += (e + 3) / 4 * 4;
    }
    pl.bytes = off * 4;
    return pl.bytes <= 159 * 1024;  // and the claimed index
}

int worker_lds_blocks_per_cu(const LdsPlan &pl) {
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, worker_lds_kernel<kTrainAtomic>, NT, (size_t)pl.bytes) !=
        hipSuccess)
        return 0;
    return nb;
}

hipError_t launch_worker_lds(int mode, const LdsPlan &pl, const WorkArgs &a, int grid, hipStream_t s) {
    if (mode == kTrainAtomic) worker_lds_kernel<kTrainAtomic><<<grid, NT, (size_t)pl.bytes, s>>>(pl, a);
    else if (mode == kTrainRacy) worker_lds_kernel<kTrainRacy><<<grid, NT, (size_t)pl.bytes, s>>>(pl, a);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

} // namespace chaos
