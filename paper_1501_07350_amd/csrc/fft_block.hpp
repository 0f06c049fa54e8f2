// fft_block.hpp -- two or three axis passes of a small block in one kernel.
//
// A workgroup owns a contiguous block of A x B x C elements (a plane of a
// grid: A = 1, or a whole grid), reads it once into LDS, transforms it there
// along c, b and (for whole grids) a, and writes it once.  The passes it
// replaces would each read and write the block and cost a launch; the
// arithmetic of every line is that of the stand-alone pass with the same
// radix sequence, so the results have the same bits.
//
// LDS layout: element (a, b, c) sits at (a B + b) * pitch + c with an odd
// pitch.  Lanes walk across lines in every pass (rows in the pass over c,
// columns in the others), so a wave's accesses are pitch or one apart and
// fall on different banks without padding, and one instantiation per line
// length serves every axis: a block runs each instruction a few times only,
// so that fetching its code is a good part of its time.  Every thread does at
// most one butterfly of a stage (TPL = L / the smallest radix threads per
// line).
#pragma once

#include "fft_device.hpp"

namespace offt {

struct BlockArgs {
    const void* in;
    void* out;
    const void* tw[3];   // tables W_L^m of the axes c, b, a
    int kid[3];          // kernel case of the axes c, b, a
    int A, B, C;
    int naxes;           // 2: c and b (A == 1), 3: c, b and a
    int pitch;           // row pitch in LDS, elements
    uint32_t rcp_C;      // ceil(2^32 / C): f div C for f < 2^16
    int stream_in;       // grid data loaded / stored with streaming accesses
    int stream_out;
    int conj_in;
    int conj_out;
    double scale;
};

// f div C for 0 <= f < 2^16 and 2 <= C <= 2^10: with m = ceil(2^32 / C),
// f m / 2^32 exceeds f / C by less than f / 2^32 < 1 / C.
__host__ __device__ constexpr uint32_t block_rcp(int C) { return (uint32_t)((0x100000000ull + C - 1) / C); }
__device__ __forceinline__ int block_div(int f, uint32_t rcp) { return (int)(((uint64_t)(uint32_t)f * rcp) >> 32); }

// Elements of LDS: the rows, then the twiddle tables of the axes in use.
__host__ __device__ constexpr int block_pitch(int C) { return C | 1; }
__host__ __device__ constexpr int64_t block_lds_elems(int A, int B, int C) {
    return (int64_t)A * B * block_pitch(C) + C + B + (A > 1 ? A : 0);
}

// Element j of a line in LDS.
template <typename V> struct BlockLine {
    V* p;
    int stride;
    __device__ __forceinline__ V& operator()(int j) const { return p[j * stride]; }
};

// Stage of span NS and radix R on the inputs v of butterfly t, then the next
// stages through the line's own LDS slots; the last stage's outputs go to
// sink(j, value), after a barrier if it writes those slots too.
template <typename V, int L, int NS, int R, int... Rest, typename At, typename Sink>
__device__ __forceinline__ void block_stages(V (&v)[R], const At& at, const V* __restrict__ tw, int t, bool act,
                                             bool sink_lds, Sink& sink) {
    constexpr int NBF = L / R;   // butterflies
    const bool on = act && t < NBF;
    if (on) {
        if constexpr (NS > 1) {
            constexpr int STEP = L / (NS * R);
            const int k = t % NS;
#pragma unroll
            for (int r = 1; r < R; ++r) v[r] = cmul(v[r], tw[r * k * STEP]);
        }
        dft<R>(v);
    }
    if constexpr (sizeof...(Rest) == 0) {
        static_assert(NS * R == L, "last stage must complete the transform");
        if (sink_lds) __syncthreads();
        if (on) {
#pragma unroll
            for (int r = 0; r < R; ++r) sink(t + r * NBF, v[r]);
        }
    } else {
        constexpr int R2 = FirstRadix<Rest...>::value;
        __syncthreads();   // every input of the stage has been read
        if (on) {
            const int base = (t / NS) * NS * R + (t % NS);
#pragma unroll
            for (int r = 0; r < R; ++r) at(base + r * NS) = v[r];
        }
        __syncthreads();
        V u[R2];
        if (act && t < L / R2) {
#pragma unroll
            for (int r = 0; r < R2; ++r) u[r] = at(t + r * (L / R2));
        }
        block_stages<V, L, NS * R, Rest...>(u, at, tw, t, act, sink_lds, sink);
    }
}

template <typename V, int L, int R, int... Rest, typename At, typename Sink>
__device__ __forceinline__ void block_line(const At& at, const V* __restrict__ tw, int t, bool act, bool sink_lds,
                                           Sink& sink) {
    V v[R];
    if (act && t < L / R) {
#pragma unroll
        for (int r = 0; r < R; ++r) v[r] = at(t + r * (L / R));
    }
    block_stages<V, L, 1, R, Rest...>(v, at, tw, t, act, sink_lds, sink);
}

// The pass over axis 0 (c), 1 (b) or 2 (a): blockDim / TPL lines at a time,
// lanes on consecutive lines.  The last pass writes the block to HBM.
template <typename V, int L, int TPL, int... Rs>
__device__ __forceinline__ void block_pass(const BlockArgs& a, V* __restrict__ lds, const V* __restrict__ tw,
                                           V* __restrict__ go, int axis, int tid) {
    using S = decltype(V{}.x);
    const bool last = axis == a.naxes - 1;
    const int lines = axis == 0 ? a.A * a.B : (axis == 1 ? a.A : a.B) * a.C, per = (int)blockDim.x / TPL;
    const int stride = axis == 0 ? 1 : (axis == 1 ? a.pitch : a.B * a.pitch);
    const int outer = axis == 1 ? a.B * a.pitch : a.pitch;   // from one row of lines to the next
    const int gstride = axis == 1 ? a.C : a.B * a.C;
    const int t = tid / per, w = tid - t * per;
    const S scale = (S)a.scale;
#pragma unroll 1
    for (int l0 = 0; l0 < lines; l0 += per) {
        const int l = l0 + w;
        const bool act = t < TPL && l < lines;
        int o = act ? l : 0, c = 0;      // rows: line l is row l
        if (axis > 0) {
            const int q = block_div(o, a.rcp_C);
            c = o - q * a.C;
            o = q;
        }
        const BlockLine<V> at{lds + o * outer + c, stride};
        auto sink = [&](int j, V x) {
            if (last) store_io(go + (int64_t)l + (int64_t)j * gstride, fix_out(x, a.conj_out, scale), a.stream_out != 0);
            else at(j) = x;
        };
        block_line<V, L, Rs...>(at, tw, t, act, !last, sink);
    }
}

// One block: load, then the passes over c, b and a.  Pass runs the kernel
// case of an axis.
template <typename V, typename Pass>
__device__ __forceinline__ void block_body(const BlockArgs& a, V* __restrict__ lds, int64_t block, const Pass& pass) {
    const int tid = (int)threadIdx.x, T = (int)blockDim.x;
    const int n = a.A * a.B * a.C;
    const V* g = static_cast<const V*>(a.in) + block * n;
    V* go = static_cast<V*>(a.out) + block * n;
    V* tw = lds + (int64_t)a.A * a.B * a.pitch;
    const int len[3] = {a.C, a.B, a.A};
    // the block with up to 8 loads in flight per thread
    constexpr int U = 8;
#pragma unroll 1
    for (int f0 = tid; f0 < n; f0 += U * T) {
        V x[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (f0 + u * T < n) x[u] = load_io(g + f0 + u * T, a.stream_in != 0);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int f = f0 + u * T;
            if (f < n) {
                const int r = block_div(f, a.rcp_C);
                lds[r * a.pitch + f - r * a.C] = fix_in(x[u], a.conj_in);
            }
        }
    }
    V* twk = tw;
    for (int ax = 0; ax < a.naxes; ++ax) {
        const V* src = static_cast<const V*>(a.tw[ax]);
        for (int i = tid; i < len[ax]; i += T) twk[i] = src[i];
        twk += len[ax];
    }
#pragma unroll 1
    for (int ax = 0; ax < a.naxes; ++ax) {
        __syncthreads();
        int id = tid;
        OFFT_OPAQUE_VGPR(id);   // each case's index math stays in its pass
        pass(a, lds, tw, go, ax, id);
        tw += ax == 0 ? a.C : a.B;
    }
}

}  // namespace offt
