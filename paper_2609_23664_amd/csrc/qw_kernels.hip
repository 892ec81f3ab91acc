// gfx950 kernels of libqw.
//
// Layout: a state slot is 2^n complex64 amplitudes (float2, interleaved),
// qubit q = bit q of the index.
//
// Gate pass (pass_kernel_lds, pass_kernel_flat): one workgroup (several in
// the flat form) owns one tile of 2^M amplitudes per (task, pass); the tile
// is the set of indices that differ only in the
// pass's M local bits. 2^(M-4) threads hold 16 amplitudes each in registers.
// A "phase" maps 4 local bits to the 16 register slots and the remaining
// M-4 local bits to the thread index (its 6 lowest bits to the lanes of a
// 64-wide wavefront). Ops whose target bit sits in a register slot run in
// registers; between phases the tile is exchanged through LDS (XOR-swizzled
// to spread LDS banks). The first and last phases are I/O phases: slot 0 is
// local bit 0 and the lanes are local bits 1..6, so every load/store is a
// 16-byte access and eight consecutive lanes cover one 128-byte run.
//
// All reductions are FP64 and use a fixed order (per-thread sequential,
// then a fixed shuffle tree, then the waves in order), so results do not
// depend on how many tasks share a launch.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "qw_internal.h"
#include "qw_dev.h"
#include "qw_kernels.h"

namespace qw {

// ------------------------------------------------------------- interpreter
// The interpreted pass kernels read each op record at run time and branch to
// the matching tile operation of qw_dev.h; generated kernels call the same
// operations with the record contents fixed at compile time.

// Uniform loads of the small plan records, kept in scalar registers.
struct PhaseHead {
    uint8_t reg[4];
    uint16_t op_begin, op_end;
    uint8_t io;
};

__device__ __forceinline__ PhaseHead ld_phase_head(const DevPhase *p) {
    const QW_CONST uint32_t *w = (const QW_CONST uint32_t *)(p);
    const uint32_t w0 = uni(w[0]), w1 = uni(w[1]), w2 = uni(w[2]);
    PhaseHead h;
    h.reg[0] = (uint8_t)w0;
    h.reg[1] = (uint8_t)(w0 >> 8);
    h.reg[2] = (uint8_t)(w0 >> 16);
    h.reg[3] = (uint8_t)(w0 >> 24);
    h.op_begin = (uint16_t)w1;
    h.op_end = (uint16_t)(w1 >> 16);
    h.io = (uint8_t)w2;
    return h;
}

__device__ __forceinline__ uint64_t dpdep(uint64_t v, uint64_t mask) {
    uint64_t r = 0;
    uint64_t bb = 1;
    while (mask) {
        uint64_t low = mask & (~mask + 1);
        if (v & bb) r |= low;
        bb <<= 1;
        mask &= mask - 1;
    }
    return r;
}

__device__ __forceinline__ uint32_t dpdep32(uint32_t v, uint32_t mask) {
    uint32_t r = 0;
    uint32_t bb = 1;
    while (mask) {
        uint32_t low = mask & (~mask + 1);
        if (v & bb) r |= low;
        bb <<= 1;
        mask &= mask - 1;
    }
    return r;
}

// Value of a thread or global operand bit (never a register bit).
__device__ __forceinline__ bool opbit_tg(uint8_t loc, uint8_t bit, uint32_t tl, uint64_t base) {
    return loc == LOC_THREAD ? ((tl >> bit) & 1u) : ((uint32_t)(base >> bit) & 1u);
}

// The 16 amplitudes as one value. An operation takes them out into an array,
// works on that with constant indices and puts them back: passed by reference
// through the switch over the operations, the array's addresses are merged by
// the compiler before it can split the array into registers, and every
// operation then loads and stores it in scratch memory. 4 layers on one
// 15-qubit state took 587 us that way, 128 now; 2 layers on 64 20-qubit states
// 8.05 ms, now 1.51; on 8 24-qubit states 20.7 ms, now 3.39.
typedef float Amps __attribute__((ext_vector_type(32)));

template <class F>
__device__ __forceinline__ Amps on(Amps r, F &&f) {
    float2 v[16];
    #pragma unroll
    for (int k = 0; k < 16; ++k) v[k] = make_float2(r[2 * k], r[2 * k + 1]);
    f(v);
    #pragma unroll
    for (int k = 0; k < 16; ++k) {
        r[2 * k] = v[k].x;
        r[2 * k + 1] = v[k].y;
    }
    return r;
}

#define QW_ON(CALL) r = on(r, [&](float2 (&v)[16]) __attribute__((always_inline)) { CALL; })
#define QW_SLOT4(FN, SEL, ...)                                    \
    switch (SEL) {                                                \
    case 0: QW_ON(FN<0>(v, __VA_ARGS__)); break;                  \
    case 1: QW_ON(FN<1>(v, __VA_ARGS__)); break;                  \
    case 2: QW_ON(FN<2>(v, __VA_ARGS__)); break;                  \
    default: QW_ON(FN<3>(v, __VA_ARGS__)); break;                 \
    }
#define QW_LANE6(FN, SEL, ...)                                    \
    switch (SEL) {                                                \
    case 0: QW_ON(FN<0>(v, __VA_ARGS__)); break;                  \
    case 1: QW_ON(FN<1>(v, __VA_ARGS__)); break;                  \
    case 2: QW_ON(FN<2>(v, __VA_ARGS__)); break;                  \
    case 3: QW_ON(FN<3>(v, __VA_ARGS__)); break;                  \
    case 4: QW_ON(FN<4>(v, __VA_ARGS__)); break;                  \
    default: QW_ON(FN<5>(v, __VA_ARGS__)); break;                 \
    }
// a pair of slots (a target, or one operand of a CZ, and a control)
#define QW_SLOT4C(FN, S, C)                                       \
    switch (C) {                                                  \
    case 0: QW_ON((FN<S, 0>(v))); break;                          \
    case 1: QW_ON((FN<S, 1>(v))); break;                          \
    case 2: QW_ON((FN<S, 2>(v))); break;                          \
    default: QW_ON((FN<S, 3>(v))); break;                         \
    }
#define QW_URT4(F, SEL, T)                                        \
    switch (SEL) {                                                \
    case 0: QW_ON((urt_r<0, F>(v, T))); break;                    \
    case 1: QW_ON((urt_r<1, F>(v, T))); break;                    \
    case 2: QW_ON((urt_r<2, F>(v, T))); break;                    \
    default: QW_ON((urt_r<3, F>(v, T))); break;                   \
    }
#define QW_URT6(F, SEL, T)                                        \
    switch (SEL) {                                                \
    case 0: QW_ON((urt_l<0, F>(v, T, lane))); break;              \
    case 1: QW_ON((urt_l<1, F>(v, T, lane))); break;              \
    case 2: QW_ON((urt_l<2, F>(v, T, lane))); break;              \
    case 3: QW_ON((urt_l<3, F>(v, T, lane))); break;              \
    case 4: QW_ON((urt_l<4, F>(v, T, lane))); break;              \
    default: QW_ON((urt_l<5, F>(v, T, lane))); break;             \
    }

// One op record (not OP_DSET) on the registers of a phase.
__device__ __forceinline__ Amps run_op(Amps r, const DevOp &op, const DevOp *ops, uint32_t j,
                                       uint32_t tl, uint64_t base) {
    const uint32_t lane = threadIdx.x & 63u;
    if (op.la == LOC_LANE) {
        switch (op.type) {
        case OP_U:
            QW_LANE6(u_l, op.sa, opc(ops, j, 0), opc(ops, j, 1), opc(ops, j, 2), opc(ops, j, 3), lane)
            break;
        case OP_UR:
            QW_LANE6(ur_l, op.sa, opm(ops, j, 0), opm(ops, j, 1), opm(ops, j, 2), opm(ops, j, 3), lane)
            break;
        case OP_URD: {
            const Urd e = urd_entries(ops, j);
            QW_LANE6(ur_l, op.sa, e.a, e.b, e.c, e.d, lane)
            break;
        }
        case OP_URT:
            if (op.b) {
                QW_URT6(1, op.sa, opm(ops, j, 0))
            } else {
                QW_URT6(0, op.sa, opm(ops, j, 0))
            }
            break;
        case OP_PERM:
            QW_LANE6(perm_l, op.sa, opc(ops, j, 0), opc(ops, j, 1), lane)
            break;
        case OP_CX:
            if (op.lb == LOC_REG) {
                switch (op.sa) {
                case 0: QW_SLOT4C(cx_lr, 0, op.sb) break;
                case 1: QW_SLOT4C(cx_lr, 1, op.sb) break;
                case 2: QW_SLOT4C(cx_lr, 2, op.sb) break;
                case 3: QW_SLOT4C(cx_lr, 3, op.sb) break;
                case 4: QW_SLOT4C(cx_lr, 4, op.sb) break;
                default: QW_SLOT4C(cx_lr, 5, op.sb) break;
                }
            } else {
                const bool c = opbit_tg(op.lb, op.b, tl, base);
                QW_LANE6(cx_lb, op.sa, c)
            }
            break;
        default: break;
        }
        return r;
    }
    switch (op.type) {
    case OP_URT:
        if (op.b) {
            QW_URT4(1, op.sa, opm(ops, j, 0))
        } else {
            QW_URT4(0, op.sa, opm(ops, j, 0))
        }
        break;
    case OP_UR:
        QW_SLOT4(ur_r, op.sa, opm(ops, j, 0), opm(ops, j, 1), opm(ops, j, 2), opm(ops, j, 3))
        break;
    case OP_URD: {
        const Urd e = urd_entries(ops, j);
        QW_SLOT4(ur_r, op.sa, e.a, e.b, e.c, e.d)
        break;
    }
    case OP_U:
        QW_SLOT4(u_r, op.sa, opc(ops, j, 0), opc(ops, j, 1), opc(ops, j, 2), opc(ops, j, 3))
        break;
    case OP_PERM:
        QW_SLOT4(perm_r, op.sa, opc(ops, j, 0), opc(ops, j, 1))
        break;
    case OP_CX:
        if (op.lb == LOC_REG) {
            switch (op.sa) {
            case 0: QW_SLOT4C(cx_rr, 0, op.sb) break;
            case 1: QW_SLOT4C(cx_rr, 1, op.sb) break;
            case 2: QW_SLOT4C(cx_rr, 2, op.sb) break;
            default: QW_SLOT4C(cx_rr, 3, op.sb) break;
            }
        } else {
            const bool c = opbit_tg(op.lb, op.b, tl, base);
            QW_SLOT4(cx_rb, op.sa, c)
        }
        break;
    case OP_DIAG:
        if (op.la == LOC_REG) {
            QW_SLOT4(diag_r, op.sa, opc(ops, j, 0), opc(ops, j, 1))
        } else {
            QW_ON(diag_b(v, opbit_tg(op.la, op.a, tl, base), opc(ops, j, 0), opc(ops, j, 1)));
        }
        break;
    case OP_CZ:
        if (op.la == LOC_REG && op.lb == LOC_REG) {
            switch (op.sa) {
            case 0: QW_SLOT4C(cz_rr, 0, op.sb) break;
            case 1: QW_SLOT4C(cz_rr, 1, op.sb) break;
            case 2: QW_SLOT4C(cz_rr, 2, op.sb) break;
            default: QW_SLOT4C(cz_rr, 3, op.sb) break;
            }
        } else if (op.la == LOC_REG) {
            const bool c = opbit_tg(op.lb, op.b, tl, base);
            QW_SLOT4(cz_rb, op.sa, c)
        } else if (op.lb == LOC_REG) {
            const bool c = opbit_tg(op.la, op.a, tl, base);
            QW_SLOT4(cz_rb, op.sb, c)
        } else {
            QW_ON(cz_bb(v, opbit_tg(op.la, op.a, tl, base) && opbit_tg(op.lb, op.b, tl, base)));
        }
        break;
    default: break;
    }
    return r;
}

// ------------------------------------------------------------- pass kernel
__device__ __forceinline__ uint32_t thread_local_index(uint32_t tid, const uint8_t *reg) {
    return thread_local_index(tid, reg[0], reg[1], reg[2], reg[3]);
}

// Global offsets of an I/O layout. IO_F4: register slot 0 = local bit 0,
// lanes = local bits 1..6, one 16-byte access per register pair. IO_F2:
// lanes = local bits 0..5, one 8-byte access per register. Waves are the
// remaining non-register local bits.
struct IoLayout {
    uint32_t lane_off;     // global index bits contributed by the lane
    uint32_t uni_off[16];  // tile base | wave part | register part, per register
};

// Position of the k-th set bit of mask (k counted from 0). Called with
// wave-uniform arguments, so it compiles to scalar code.
__device__ __forceinline__ uint32_t nth_set_bit(uint64_t mask, uint32_t k) {
    for (uint32_t i = 0; i < k; ++i) mask &= mask - 1;
    return (uint32_t)__builtin_ctzll(mask);
}

__device__ __forceinline__ IoLayout io_layout(uint64_t lmask, const uint8_t *reg, uint8_t kind,
                                              uint32_t lane, uint32_t wave, uint32_t m,
                                              uint32_t base) {
    IoLayout io;
    const uint32_t rmask = (1u << reg[0]) | (1u << reg[1]) | (1u << reg[2]) | (1u << reg[3]);
    uint32_t wmask;
    if (kind == IO_F4) {
        const uint32_t g4 = nth_set_bit(lmask, 4), g5 = nth_set_bit(lmask, 5),
                       g6 = nth_set_bit(lmask, 6);
        io.lane_off = ((lane & 7u) << 1) | (((lane >> 3) & 1u) << g4) |
                      (((lane >> 4) & 1u) << g5) | (((lane >> 5) & 1u) << g6);
        wmask = (((1u << m) - 1u) & ~0x7Fu) & ~rmask;
    } else {
        const uint32_t g4 = nth_set_bit(lmask, 4), g5 = nth_set_bit(lmask, 5);
        io.lane_off = (lane & 15u) | (((lane >> 4) & 1u) << g4) | (((lane >> 5) & 1u) << g5);
        wmask = (((1u << m) - 1u) & ~0x3Fu) & ~rmask;
    }
    const uint32_t wl = dpdep32(wave, wmask);
    const uint32_t woff = (uint32_t)dpdep(wl, lmask);
    const uint32_t r0 = 1u << nth_set_bit(lmask, reg[0]);
    const uint32_t r1 = 1u << nth_set_bit(lmask, reg[1]);
    const uint32_t r2 = 1u << nth_set_bit(lmask, reg[2]);
    const uint32_t r3 = 1u << nth_set_bit(lmask, reg[3]);
    #pragma unroll
    for (int k = 0; k < 16; ++k)
        io.uni_off[k] = base | woff | ((k & 1) ? r0 : 0u) | ((k & 2) ? r1 : 0u) |
                        ((k & 4) ? r2 : 0u) | ((k & 8) ? r3 : 0u);
    return io;
}

// Local index offset of register k for a phase with register bits reg[].
__device__ __forceinline__ uint32_t roff(const uint8_t *reg, int k) {
    return ((k & 1) ? (1u << reg[0]) : 0u) | ((k & 2) ? (1u << reg[1]) : 0u) |
           ((k & 4) ? (1u << reg[2]) : 0u) | ((k & 8) ? (1u << reg[3]) : 0u);
}

// LDS byte address of register k of a thread: swz is linear over GF(2), so
// swz(tl | roff(k)) = swz(tl) ^ swz(roff(k)) with the second part uniform.
__device__ __forceinline__ uint32_t lds_off(uint32_t stl8, const uint8_t *reg, int k) {
    return stl8 ^ (swz(roff(reg, k)) << 3);
}

// I/O layout from a host-computed record: a few VALU for the lane part, the
// rest is uniform (scalar loads from the record).
__device__ __forceinline__ IoLayout io_from_rec(const IoRec *rec, uint32_t lane, uint32_t wave,
                                                uint32_t base) {
    IoLayout io;
    const uint32_t w0 = uni(*(const QW_CONST uint32_t *)rec);
    const uint32_t kind = w0 & 0xFFu, g4 = (w0 >> 8) & 0xFFu, g5 = (w0 >> 16) & 0xFFu,
                   g6 = w0 >> 24;
    if (kind == IO_F4)
        io.lane_off = ((lane & 7u) << 1) | (((lane >> 3) & 1u) << g4) |
                      (((lane >> 4) & 1u) << g5) | (((lane >> 5) & 1u) << g6);
    else
        io.lane_off = (lane & 15u) | (((lane >> 4) & 1u) << g4) | (((lane >> 5) & 1u) << g5);
    const uint32_t bw = base | uni(ldu(rec->wave_off + wave));
    #pragma unroll
    for (int k = 0; k < 16; ++k) io.uni_off[k] = bw | uni(ldu(rec->reg_off + k));
    return io;
}

// Store layout of a pass: with PD_REMAP_OUT the non-local bits follow the
// pass's output relabelling (tile_base_out, and the per-wave and
// per-register xor terms of the record), otherwise those of the load.
__device__ __forceinline__ IoLayout io_out_layout(const PassDesc &d, uint32_t tile, uint32_t lane,
                                                  uint32_t wave, uint32_t base) {
    if (!(d.flags & PD_REMAP_OUT)) return io_from_rec(d.io_out, lane, wave, base);
    const uint32_t bo = uni(ldu(d.tile_base_out + tile)) ^ uni(ldu(d.io_out->wave_xor + wave));
    IoLayout io = io_from_rec(d.io_out, lane, wave, bo);
    #pragma unroll
    for (int k = 0; k < 16; ++k) io.uni_off[k] ^= uni(ldu(d.io_out->reg_xor + k));
    return io;
}

__device__ __forceinline__ Amps io_load(const void *src, const IoLayout &io, uint8_t kind) {
    const uint32_t lb = io.lane_off * 8u;
    Amps r;
    if (kind == IO_F4) {
        #pragma unroll
        for (int k2 = 0; k2 < 8; ++k2) {
            const float4 q = buf_ld4(src, io.uni_off[2 * k2], lb);
            r[4 * k2] = q.x;
            r[4 * k2 + 1] = q.y;
            r[4 * k2 + 2] = q.z;
            r[4 * k2 + 3] = q.w;
        }
    } else {
        #pragma unroll
        for (int k = 0; k < 16; ++k) {
            const float2 q = buf_ld2(src, io.uni_off[k], lb);
            r[2 * k] = q.x;
            r[2 * k + 1] = q.y;
        }
    }
    return r;
}

__device__ __forceinline__ void io_store(Amps r, void *dst, const IoLayout &io, uint8_t kind) {
    const uint32_t lb = io.lane_off * 8u;
    if (kind == IO_F4) {
        #pragma unroll
        for (int k2 = 0; k2 < 8; ++k2)
            buf_st4(dst, io.uni_off[2 * k2], lb, make_float2(r[4 * k2], r[4 * k2 + 1]),
                    make_float2(r[4 * k2 + 2], r[4 * k2 + 3]));
    } else {
        #pragma unroll
        for (int k = 0; k < 16; ++k) buf_st2(dst, io.uni_off[k], lb, make_float2(r[2 * k], r[2 * k + 1]));
    }
}

// block_sum of a workgroup of `waves` waves.
__device__ double block_sum_n(double v, double *red, uint32_t waves) {
    #pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    if (waves == 1u) return v;
    __syncthreads();
    if ((threadIdx.x & 63u) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    double s = 0.0;
    if (threadIdx.x == 0)
        for (uint32_t k = 0; k < waves; ++k) s += red[k];
    return s;
}

// Amplitudes scaled in FP64 (PD_SCALE_IN).
__device__ __forceinline__ Amps scale_in(Amps r, double s) {
    #pragma unroll
    for (int k = 0; k < 32; ++k) r[k] = (float)((double)r[k] * s);
    return r;
}

// Run the ops of one op range [o, end) on the registers. The next op record
// is requested before the current one is executed (scalar-load prefetch).
__device__ __forceinline__ Amps run_ops(Amps r, const DevOp *ops, uint32_t o, uint32_t end,
                                        uint32_t tl, uint64_t base) {
    if (o >= end) return r;
    DevOp nxt = ld_words(ops + o);
    while (o < end) {
        const DevOp op = nxt;
        const uint32_t step = (op.type == OP_DSET) ? 1u + op.sb + op.b + op.a : 1u;
        if (o + step < end) nxt = ld_words(ops + o + step);
        if (op.type == OP_DSET) {
            // thread/global members -> one factor; table; mixed members
            float2 ft = make_float2(1.0f, 0.0f);
            const uint32_t m0 = o + 1 + op.sb;
            for (uint32_t j = 0; j < op.b; ++j) {
                const DevOp mm = ld_words(ops + m0 + j);
                ft = dset_fold(ft, pdiag_tg(tl, base, mm.tmask, mm.gmask), opc(ops, m0 + j, 0),
                               opc(ops, m0 + j, 1));
            }
            // with a table or thread members, the first mixed member is
            // merged into the application
            const uint32_t merged = (op.a && (op.sb || op.b)) ? 1u : 0u;
            if (merged) {
                const DevOp mm = ld_words(ops + m0 + op.b);
                const bool pt = pdiag_tg(tl, base, mm.tmask, mm.gmask);
                const float2 d0 = opc(ops, m0 + op.b, 0), d1 = opc(ops, m0 + op.b, 1);
                if (op.sb) {
                    QW_ON(dset_apply_m(v, ops + o + 1, true, ft, pt, d0, d1, mm.rmask));
                } else {
                    QW_ON(dset_apply_m(v, ops, false, ft, pt, d0, d1, mm.rmask));
                }
            } else if (op.sb) {
                if (op.b) {
                    QW_ON(dset_apply(v, ops + o + 1, true, ft, true));
                } else {
                    QW_ON(dset_apply(v, ops + o + 1, true, ft, false));
                }
            } else if (op.b) {
                QW_ON(dset_apply(v, ops, false, ft, true));
            }
            for (uint32_t j = merged; j < op.a; ++j) {
                const DevOp mm = ld_words(ops + m0 + op.b + j);
                const bool pt = pdiag_tg(tl, base, mm.tmask, mm.gmask);
                const float2 d0 = opc(ops, m0 + op.b + j, 0), d1 = opc(ops, m0 + op.b + j, 1);
                QW_ON(pdiag_mixed(v, pt, d0, d1, mm.rmask));
            }
        } else {
            r = run_op(r, op, ops, o, tl, base);
        }
        o += step;
    }
    return r;
}

// (The tile size is a run-time argument of both forms: it only sets the
// workgroup size and the LDS bytes.) One-phase passes: workgroups of at most
// 256 threads, several per tile.
__global__ __launch_bounds__(256) void pass_kernel_flat(const PassDesc *__restrict__ descs, uint32_t n_descs,
                                                        uint32_t parts, uint32_t items, int remap) {
    const uint32_t wg_item = item_of(blockIdx.x, gridDim.x, remap);
    const uint32_t item = wg_item / parts;
    if (item >= items) return;
    const uint32_t part = wg_item % parts;
    const uint32_t p = item % n_descs;
    const uint32_t tile = item / n_descs;
    const PassDesc d = ld_words(descs + p);
    const uint32_t base = uni(ldu(d.tile_base + tile));
    const uint32_t tid = part * blockDim.x + threadIdx.x;
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t wave = uni(tid >> 6);
    const PhaseHead ph = ld_phase_head(d.phases);
    const uint32_t tl = thread_local_index(tid, ph.reg);
    Amps r = io_load(d.src, io_from_rec(d.io_in, lane, wave, base), ph.io);
    if (d.flags & PD_SCALE_IN) r = scale_in(r, *gin<double>(d.scale_in));
    r = run_ops(r, d.ops, ph.op_begin, ph.op_end, tl, base);
    io_store(r, d.dst, io_out_layout(d, tile, lane, wave, base), ph.io);
}

// Multi-phase passes: a workgroup of up to 1024 threads owns a whole tile in
// LDS for exchanges. Workgroups are persistent: each walks a list of items.
// The items of XCD x (workgroups b with b mod 8 == x) are one contiguous
// range, so the tasks that read the same snapshot tile run on one XCD at about
// the same time. Bound by the operations' issue, not by memory, so the next
// tile is not loaded ahead.
__global__ __launch_bounds__(1024) void pass_kernel_lds(const PassDesc *__restrict__ descs,
                                                        uint32_t n_descs, uint32_t items) {
    extern __shared__ float2 lds[];   // one tile: 16 amplitudes per thread
    __shared__ double red[17];
    const uint32_t w = blockIdx.x, x = w & 7u, j = w >> 3, wpx = gridDim.x >> 3;
    const uint32_t per = (items + 7u) >> 3;
    const uint32_t first = x * per;
    const uint32_t last = (first + per < items) ? first + per : items;
    uint32_t item = first + j;
    if (item >= last) return;
    const uint32_t tid = threadIdx.x;
    const uint32_t lane = tid & 63u;
    const uint32_t wave = uni(tid >> 6);
    char *lb = reinterpret_cast<char *>(lds);

    while (true) {
        const uint32_t p = item % n_descs;
        const uint32_t tile = item / n_descs;
        const PassDesc d = ld_words(descs + p);
        const uint32_t base = uni(ldu(d.tile_base + tile));
        PhaseHead ph = ld_phase_head(d.phases);
        Amps r = io_load(d.src, io_from_rec(d.io_in, lane, wave, base), ph.io);
        if (d.flags & PD_SCALE_IN) r = scale_in(r, *gin<double>(d.scale_in));
        uint32_t tl = thread_local_index(tid, ph.reg);
        const uint32_t nph = d.n_phases;
        for (uint32_t pi = 0; pi < nph; ++pi) {
            if (pi > 0) {
                const uint32_t *off_prev = d.phases[pi - 1].lds_off;
                const uint32_t *off_next = d.phases[pi].lds_off;
                const uint32_t stl8 = swz(tl) << 3;
                lds_barrier();
                #pragma unroll
                for (int k = 0; k < 16; ++k)
                    *reinterpret_cast<float2 *>(lb + (stl8 ^ uni(ldu(off_prev + k)))) =
                        make_float2(r[2 * k], r[2 * k + 1]);
                lds_barrier();
                ph = ld_phase_head(d.phases + pi);
                tl = thread_local_index(tid, ph.reg);
                const uint32_t ntl8 = swz(tl) << 3;
                #pragma unroll
                for (int k = 0; k < 16; ++k) {
                    const float2 q = *reinterpret_cast<const float2 *>(lb + (ntl8 ^ uni(ldu(off_next + k))));
                    r[2 * k] = q.x;
                    r[2 * k + 1] = q.y;
                }
            }
            r = run_ops(r, d.ops, ph.op_begin, ph.op_end, tl, base);
        }
        if (d.flags & PD_NORM_OUT) {
            double s = 0.0;
            #pragma unroll
            for (int k = 0; k < 32; ++k) {
                const double x = r[k];
                s = fma(x, x, s);
            }
            s = block_sum_n(s, red, blockDim.x >> 6);
            if (tid == 0) gout<double>(d.norm_part)[tile] = s;
        }
        io_store(r, d.dst, io_out_layout(d, tile, lane, wave, base), ph.io);
        item += wpx;
        if (item >= last) break;
        lds_barrier();  // the next tile's first exchange reuses the LDS buffer
    }
}

// ------------------------------------------------------------- small states
// n < 10: one workgroup of 64 threads holds the whole state in LDS and runs
// the ops one at a time (every bit is local).
__global__ __launch_bounds__(64) void small_pass_kernel(const PassDesc *__restrict__ descs,
                                                        uint32_t n) {
    __shared__ float2 s[512];
    __shared__ double red[2];
    const PassDesc &d = descs[blockIdx.x];
    const uint32_t dim = 1u << n;
    const uint32_t tid = threadIdx.x;
    const float2 *src = reinterpret_cast<const float2 *>(d.src);
    float2 *dst = reinterpret_cast<float2 *>(d.dst);
    const double sc = (d.flags & PD_SCALE_IN) ? *d.scale_in : 1.0;
    for (uint32_t i = tid; i < dim; i += 64) {
        float2 a = src[i];
        if (d.flags & PD_SCALE_IN) a = make_float2((float)((double)a.x * sc), (float)((double)a.y * sc));
        s[i] = a;
    }
    __syncthreads();
    for (uint32_t o = 0; o < d.n_ops; ++o) {
        const DevOp op = d.ops[o];
        if (op.type == OP_DSET) continue;  // members follow as plain parity factors
        if (op.type == OP_PDIAG) {
            const float2 d0 = make_float2(op.m[0], op.m[1]), d1 = make_float2(op.m[2], op.m[3]);
            for (uint32_t i = tid; i < dim; i += 64)
                s[i] = cmul((__popc(i & op.tmask) & 1u) ? d1 : d0, s[i]);
            __syncthreads();
            continue;
        }
        if (op.type == OP_U || op.type == OP_PERM || op.type == OP_CX || op.type == OP_UR ||
            op.type == OP_URT || op.type == OP_URD) {
            float e0 = op.m[0], e1 = op.m[1], e2 = op.m[2], e3 = op.m[3];
            if (op.type == OP_URD) {
                const Urd e = urd_entries(d.ops, o);
                e0 = e.a; e1 = e.b; e2 = e.c; e3 = e.d;
            }
            const uint32_t bit = 1u << op.a;
            for (uint32_t pr = tid; pr < dim / 2; pr += 64) {
                const uint32_t i0 = ((pr >> op.a) << (op.a + 1)) | (pr & (bit - 1));
                const uint32_t i1 = i0 | bit;
                const float2 x = s[i0], y = s[i1];
                if (op.type == OP_U) {
                    s[i0] = cmad2(make_float2(op.m[0], op.m[1]), x, make_float2(op.m[2], op.m[3]), y);
                    s[i1] = cmad2(make_float2(op.m[4], op.m[5]), x, make_float2(op.m[6], op.m[7]), y);
                } else if (op.type == OP_URT) {
                    float2 a = x, b = y;
                    if (op.b) urt_pair<1>(op.m[0], a, b);
                    else urt_pair<0>(op.m[0], a, b);
                    s[i0] = a;
                    s[i1] = b;
                } else if (op.type == OP_UR || op.type == OP_URD) {
                    s[i0] = make_float2(fmaf(e0, x.x, e1 * y.x), fmaf(e0, x.y, e1 * y.y));
                    s[i1] = make_float2(fmaf(e2, x.x, e3 * y.x), fmaf(e2, x.y, e3 * y.y));
                } else if (op.type == OP_PERM) {
                    s[i0] = cmul(make_float2(op.m[0], op.m[1]), y);
                    s[i1] = cmul(make_float2(op.m[2], op.m[3]), x);
                } else if ((i0 >> op.b) & 1u) {
                    s[i0] = y;
                    s[i1] = x;
                }
            }
        } else if (op.type == OP_DIAG) {
            const float2 d0 = make_float2(op.m[0], op.m[1]), d1 = make_float2(op.m[2], op.m[3]);
            for (uint32_t i = tid; i < dim; i += 64) s[i] = cmul(((i >> op.a) & 1u) ? d1 : d0, s[i]);
        } else if (op.type == OP_CZ) {
            for (uint32_t i = tid; i < dim; i += 64)
                if (((i >> op.a) & 1u) && ((i >> op.b) & 1u)) s[i] = make_float2(-s[i].x, -s[i].y);
        }
        __syncthreads();
    }
    if (d.flags & PD_NORM_OUT) {
        double acc = 0.0;
        for (uint32_t i = tid; i < dim; i += 64) {
            const double x = s[i].x, y = s[i].y;
            acc = fma(x, x, acc);
            acc = fma(y, y, acc);
        }
        acc = block_sum<64>(acc, red);
        if (tid == 0) d.norm_part[0] = acc;
    }
    for (uint32_t i = tid; i < dim; i += 64) dst[i] = s[i];
}

// ------------------------------------------------------------- renorm
// For every descriptor with PD_NORM_OUT: scale_out = 1/sqrt(sum of tiles).
__global__ __launch_bounds__(256) void norm_finalize_kernel(const PassDesc *__restrict__ descs,
                                                            uint32_t tiles) {
    __shared__ double red[5];
    const PassDesc &d = descs[blockIdx.x];
    if (!(d.flags & PD_NORM_OUT)) return;
    double s = 0.0;
    for (uint32_t t = threadIdx.x; t < tiles; t += 256) s += d.norm_part[t];
    s = block_sum<256>(s, red);
    if (threadIdx.x == 0) *d.scale_out = 1.0 / sqrt(s);
}

// ------------------------------------------------------------- uploads
// Plan data from pinned host memory: at most 16 KiB per workgroup (a 16-byte
// read over the bus per thread, all in flight) up to 64 workgroups, then more
// rounds. Bound by the bus's latency, then its rate: 17 to 64 KiB in 4.7 us,
// 240 KiB in 7.9 (8.4 with up to 32 KiB a workgroup), 1 MiB in 23. Smaller
// blobs go another way (stage_blob). `done` tells the host that
// the source has been read; the data itself is ordered by the kernel's end.
__global__ __launch_bounds__(1024) void upload_kernel(uint4 *__restrict__ dst, const uint4 *__restrict__ src,
                                                      uint32_t count, uint32_t *done, uint32_t seq) {
    const uint32_t per = (count + gridDim.x - 1) / gridDim.x, b = blockIdx.x * per;
    const uint32_t e = b + per < count ? b + per : count;
    for (uint32_t i = b + threadIdx.x; i < e; i += 1024) dst[i] = src[i];
    __syncthreads();   // every wave's reads have returned
    if (threadIdx.x == 0) __hip_atomic_store(done + blockIdx.x, seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// ------------------------------------------------------------- init / copy
// |0> into consecutive slots of slot_f4 (a power of two) float4, PER of them a
// thread at a time. Bound by the write rate: one float4 a thread and a 64-bit
// remainder for each took 5.4 us for 8 MiB, 18.5 for 128 MiB, 62 for 384 MiB and
// 375 for 2 GiB, this 4.6, 16.2, 61 and 363. THROUGH: written through the L2
// (states that the next launch finds in the last-level cache; no write-back at
// the end of the launch).
template <uint32_t PER, bool THROUGH>
__global__ __launch_bounds__(256) void init_kernel(float4 *base, uint64_t slot_f4, uint64_t total_f4) {
    const uint64_t step = (uint64_t)gridDim.x * (256 * PER);
    for (uint64_t c = (uint64_t)blockIdx.x * (256 * PER); c < total_f4; c += step) {
        #pragma unroll
        for (uint32_t k = 0; k < PER; ++k) {
            const uint64_t i = c + k * 256 + threadIdx.x;
            const qw_v4u q = {(i & (slot_f4 - 1)) == 0 ? __float_as_uint(1.0f) : 0u, 0u, 0u, 0u};
            if (i < total_f4)
                __builtin_amdgcn_raw_buffer_store_b128(q, rsrc_at(base, 2 * (c + k * 256)), threadIdx.x * 16u, 0,
                                                       THROUGH ? 16 : 0);
        }
    }
}

__global__ __launch_bounds__(256) void copy_kernel(float4 *__restrict__ dst,
                                                   const float4 *__restrict__ src,
                                                   uint64_t count) {
    for (uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x; i < count;
         i += (uint64_t)gridDim.x * 256)
        dst[i] = src[i];
}

// ------------------------------------------------------------- expectation
// Small states (n < 10): one workgroup per slot, the state staged in LDS;
// every term is summed over all amplitudes in FP64 by one wave (per lane in
// index order, then a fixed butterfly), the terms dealt to 8 waves. Bound by
// latency: one wave for all terms waited for each term's butterfly in turn
// (50 terms at 9 qubits: 74 us, now 13 us).
constexpr int kSmallWaves = 8;

__global__ __launch_bounds__(64 * kSmallWaves) void reduce_small_kernel(
    const ReduceDescSmall *__restrict__ descs, uint32_t n) {
    __shared__ float2 s[512];
    const ReduceDescSmall &d = descs[blockIdx.x];
    const uint32_t dim = 1u << n;
    const float2 *psi = reinterpret_cast<const float2 *>(d.psi);
    for (uint32_t i = threadIdx.x; i < dim; i += 64 * kSmallWaves) s[i] = psi[i];
    __syncthreads();
    const uint32_t lane = threadIdx.x & 63u;
    for (uint32_t j = threadIdx.x >> 6; j < d.n_terms; j += kSmallWaves) {
        const TermSmall t = d.terms[j];
        double acc = 0.0;
        for (uint32_t l = lane; l < dim; l += 64) {
            const float2 a = s[l], b = s[l ^ t.x];
            const double re = fma((double)b.x, (double)a.x, (double)b.y * (double)a.y);
            const double im = fma((double)b.x, (double)a.y, -((double)b.y * (double)a.x));
            double val;
            switch (t.ny_mod4) {
            case 0: val = re; break;
            case 1: val = -im; break;
            case 2: val = -re; break;
            default: val = im; break;
            }
            acc += (__popc(l & t.z) & 1u) ? -val : val;
        }
        #pragma unroll
        for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o, 64);
        if (lane == 0) d.part[t.out_index] = acc;
    }
}

template <bool ODD>
__device__ __forceinline__ float pair_sum_x(uint32_t xr, const float2 (&v)[16], uint32_t smask) {
    switch (xr) {
    case 1: return pair_sum<1, ODD>(v, smask);
    case 2: return pair_sum<2, ODD>(v, smask);
    case 3: return pair_sum<3, ODD>(v, smask);
    case 4: return pair_sum<4, ODD>(v, smask);
    case 5: return pair_sum<5, ODD>(v, smask);
    case 6: return pair_sum<6, ODD>(v, smask);
    case 7: return pair_sum<7, ODD>(v, smask);
    case 8: return pair_sum<8, ODD>(v, smask);
    case 9: return pair_sum<9, ODD>(v, smask);
    case 10: return pair_sum<10, ODD>(v, smask);
    case 11: return pair_sum<11, ODD>(v, smask);
    case 12: return pair_sum<12, ODD>(v, smask);
    case 13: return pair_sum<13, ODD>(v, smask);
    case 14: return pair_sum<14, ODD>(v, smask);
    default: return pair_sum<15, ODD>(v, smask);
    }
}


// Register-phase reducer. One workgroup per (slot, group, row of tiles):
// each tile is loaded with the I/O layout, staged in LDS, and re-read with
// each phase's layout. Terms are taken 8 at a time (in phase order): every
// thread adds each term's FP32 value over the row's tiles in tile order,
// then the 8 sums are converted to FP64 and summed across the wave by a
// butterfly that halves the number of values per lane at each of the first
// three steps (fixed order); wave sums are added in wave order. A term's
// result does not depend on the other terms of its chunk, so the generated
// reducers (all terms of a tile at once) round identically. The row's tiles
// are re-read for each chunk of 8 terms.
template <int M>
__global__ __launch_bounds__(1 << (M - 4)) void reduce_kernel(const ReduceDesc *__restrict__ descs,
                                                              uint32_t n_descs, uint32_t n,
                                                              uint32_t items) {
    constexpr int T = 1 << (M - 4);
    constexpr int W = T / 64;
    __shared__ float2 lds[1 << M];
    __shared__ double red[W * kMaxGroupTerms];
    const uint32_t item = blockIdx.x;
    if (item >= items) return;
    const uint32_t p = item % n_descs;
    const uint32_t tiles = 1u << (n - M), rt = red_row_tiles(tiles);
    const uint64_t row = item / n_descs;
    const ReduceDesc d = ld_words(descs + p);
    const uint64_t lmask = d.local_mask;
    const uint64_t full = (n >= 64) ? ~0ull : ((1ull << n) - 1ull);
    const uint32_t tid = threadIdx.x;
    const uint32_t lane = tid & 63u, wave = tid >> 6;
    const uint8_t io[4] = {0, 7, 8, 9};   // I/O layout: register slots = local bits 0, 7, 8, 9

    for (uint32_t j0 = 0; j0 < d.n_terms; j0 += 8u) {
        const uint32_t j1 = j0 + 8u < d.n_terms ? j0 + 8u : d.n_terms;
        float q[8];
        #pragma unroll
        for (int i = 0; i < 8; ++i) q[i] = 0.0f;
        for (uint32_t k = 0; k < rt; ++k) {
            const uint64_t tile = row * rt + k;
            const uint64_t base = dpdep(tile, full & ~lmask);
            float2 v[16];
            {
                const uint32_t tl = thread_local_index(tid, io);
                const IoLayout lay = io_layout(lmask, io, IO_F4, lane, uni(tid >> 6), M, (uint32_t)base);
                const Amps r = io_load(d.psi, lay, IO_F4);
                #pragma unroll
                for (int k2 = 0; k2 < 16; ++k2) v[k2] = make_float2(r[2 * k2], r[2 * k2 + 1]);
                __syncthreads();   // the previous tile's LDS reads are done
                const uint32_t stl8 = swz(tl) << 3;
                char *lb = reinterpret_cast<char *>(lds);
                #pragma unroll
                for (int r = 0; r < 16; ++r)
                    *reinterpret_cast<float2 *>(lb + lds_off(stl8, io, r)) = v[r];
            }
            __syncthreads();
            for (uint32_t pi = 0; pi < d.n_phases; ++pi) {
                const RedPhase ph = ld_words(d.phases + pi);
                if (ph.t_end <= j0 || ph.t_begin >= j1) continue;
                const uint32_t tl = thread_local_index(tid, ph.reg);
                if (!ph.diag) {
                    const uint32_t stl8 = swz(tl) << 3;
                    const char *lb = reinterpret_cast<const char *>(lds);
                    #pragma unroll
                    for (int r = 0; r < 16; ++r)
                        v[r] = *reinterpret_cast<const float2 *>(lb + lds_off(stl8, ph.reg, r));
                }
                float pr[16];
                if (ph.diag) {
                    #pragma unroll
                    for (int r = 0; r < 16; ++r) pr[r] = fmaf(v[r].x, v[r].x, v[r].y * v[r].y);
                }
                const uint32_t jb = ph.t_begin > j0 ? ph.t_begin : j0;
                const uint32_t je = ph.t_end < j1 ? ph.t_end : j1;
                for (uint32_t j = jb; j < je; ++j) {
                    const TermDev t = ld_words(d.terms + j);
                    float a;
                    if (ph.diag) {
                        a = diag_sum(pr, t.smask);
                    } else {
                        a = t.odd ? pair_sum_x<true>(t.xr, v, t.smask)
                                  : pair_sum_x<false>(t.xr, v, t.smask);
                        a *= 2.0f;
                    }
                    const uint32_t par = (t.neg ^ __popc(tl & t.zt) ^ (uint32_t)__popcll(base & t.zg)) & 1u;
                    if (par) a = -a;
                    // q[j - j0] += a, with constant register indices
                    #pragma unroll
                    for (int i = 0; i < 8; ++i)
                        if ((uint32_t)i == j - j0) q[i] += a;
                }
            }
        }
        const double h = wave_reduce8(q, lane);
        if (lane < 8u) {
            const uint32_t pos = 4u * (lane & 1u) + 2u * ((lane >> 1) & 1u) + ((lane >> 2) & 1u);
            if (j0 + pos < j1) {
                // a per-lane load (ld_words reads wave-uniform records)
                const uint32_t col = d.terms[j0 + pos].col;
                red[wave * kMaxGroupTerms + col] = h;
            }
        }
    }
    __syncthreads();
    for (uint32_t c = tid; c < d.n_terms; c += T) {
        double s = 0.0;
        for (int w = 0; w < W; ++w) s += red[w * kMaxGroupTerms + c];
        gout<double>(d.part)[row * d.n_terms_total + gin<uint32_t>(d.cols)[c]] = s;
    }
}

// The rows' partials from each thread's values per tile (RowSum): one
// workgroup per 8 columns of a row adds the row's tiles in FP32 in tile order,
// then lanes and waves in FP64, as the reducers that sweep whole rows do.
// Bound by latency: 32 loads a thread, all in flight, and two barriers.
__global__ __launch_bounds__(1024) void row_sum_kernel(const RowSum *__restrict__ src, uint32_t n_src,
                                                       double *__restrict__ part, uint32_t n_terms,
                                                       uint32_t tiles) {
    __shared__ double red[16 * 8];
    const uint32_t chunk = blockIdx.x, row = blockIdx.y, slot = blockIdx.z, rows = gridDim.y;
    const uint32_t T = blockDim.x, tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    uint32_t s = 0;
    while (s + 1u < n_src && src[s + 1u].chunk0 <= chunk) ++s;
    const RowSum d = src[s];
    const uint32_t j0 = 8u * (chunk - d.chunk0), rt = red_row_tiles(tiles);
    const float *a = d.acc + ((uint64_t)slot * tiles + row * rt) * d.nt * T + tid;
    float v[kRedRowTiles][8];
    #pragma unroll
    for (uint32_t k = 0; k < kRedRowTiles; ++k) {
        #pragma unroll
        for (uint32_t i = 0; i < 8; ++i)
            v[k][i] = (k < rt && j0 + i < d.nt) ? a[((uint64_t)k * d.nt + j0 + i) * T] : 0.0f;
    }
    float q[8];
    #pragma unroll
    for (uint32_t i = 0; i < 8; ++i) {
        q[i] = v[0][i];
        #pragma unroll
        for (uint32_t k = 1; k < kRedRowTiles; ++k) q[i] = k < rt ? q[i] + v[k][i] : q[i];
    }
    const double h = wave_reduce8(q, lane);
    const uint32_t pos = 4u * (lane & 1u) + 2u * ((lane >> 1) & 1u) + ((lane >> 2) & 1u);
    if (lane < 8u) red[wave * 8u + pos] = h;
    __syncthreads();
    if (tid < 8u && j0 + tid < d.nt) {
        double sum = 0.0;
        for (uint32_t w = 0; w < T / 64u; ++w) sum += red[w * 8u + tid];
        part[((uint64_t)slot * rows + row) * n_terms + d.cols[j0 + tid]] = sum;
    }
}

// out[s] = sum_j coeff[j] * (sum over rows of part[s][row][j]); one
// workgroup per slot. A term's rows are added by one wave in the order of 256
// threads taking rows t, t + 256, ... (four groups of 64 lanes, a butterfly
// each, the groups in order); the terms are dealt to 16 waves and then added
// in term order. Bound by latency: one workgroup that took the terms one after
// the other, two barriers each, spent 39 us on 50 terms of 24-qubit states
// (256 rows) and 7.1 us on 10 terms of one row; this takes 13 us and 4.0 us.
constexpr int kFinalizeWaves = 16;
constexpr uint32_t kFinalizeTerms = 1024;   // terms held at a time

__global__ __launch_bounds__(64 * kFinalizeWaves) void expect_finalize_kernel(
    const double *__restrict__ part, const double *__restrict__ coeff, uint32_t n_terms, uint32_t rows,
    double *__restrict__ out) {
    __shared__ double sum[kFinalizeTerms], co[kFinalizeTerms];
    const uint32_t s = blockIdx.x, lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
    const double *ps = part + (uint64_t)s * rows * n_terms;
    double e = 0.0;
    for (uint32_t j0 = 0; j0 < n_terms; j0 += kFinalizeTerms) {
        const uint32_t cnt = n_terms - j0 < kFinalizeTerms ? n_terms - j0 : kFinalizeTerms;
        for (uint32_t j = threadIdx.x; j < cnt; j += 64 * kFinalizeWaves) co[j] = coeff[j0 + j];
        #pragma unroll 2
        for (uint32_t j = wave; j < cnt; j += kFinalizeWaves) {
            double a[4] = {0.0, 0.0, 0.0, 0.0};
            #pragma unroll
            for (uint32_t v = 0; v < 4; ++v)
                for (uint32_t t = 64u * v + lane; t < rows; t += 256) a[v] += ps[(uint64_t)t * n_terms + j0 + j];
            double tot = 0.0;
            #pragma unroll
            for (uint32_t v = 0; v < 4; ++v) {
                if (64u * v >= rows) break;   // (a group without rows adds zero)
                #pragma unroll
                for (int o = 32; o > 0; o >>= 1) a[v] += __shfl_xor(a[v], o, 64);
                tot += a[v];
            }
            if (lane == 0) sum[j] = tot;
        }
        __syncthreads();
        if (threadIdx.x == 0)
            for (uint32_t j = 0; j < cnt; ++j) e = fma(co[j], sum[j], e);
        __syncthreads();
    }
    if (threadIdx.x == 0) out[s] = e;
}

// ------------------------------------------------------------- sampling
// SplitMix64 output function (Steele, Lea and Flood 2014) used as a hash of
// the counter (seed, task, shot).
__device__ __forceinline__ uint64_t splitmix(uint64_t x) {
    x += 0x9E3779B97F4A7C15ull;
    x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ull;
    x = (x ^ (x >> 27)) * 0x94D049BB133111EBull;
    return x ^ (x >> 31);
}

// Chunk sums of |psi|^2 (FP64) for the joint measurement masses: one wave
// per chunk of 128 * NL amplitudes (NL 16-byte loads a lane, all in flight,
// then a fixed butterfly), four chunks a workgroup; grid (chunks / 4, slots).
// Bound by the one read of the state. No LDS and no barrier: a workgroup per
// chunk of 256 amplitudes (one 8-byte load a lane and a two-barrier block
// sum each) read 4 states of 22 qubits at 3.0 TB/s (45 us), this form
// takes 22 us (6.0 TB/s).
template <int NL>
__global__ __launch_bounds__(256) void mass_sum_kernel(const float2 *const *__restrict__ slots,
                                                       uint32_t chunks, double *__restrict__ csum) {
    const uint32_t c = blockIdx.x * 4u + (threadIdx.x >> 6), s = blockIdx.y, lane = threadIdx.x & 63u;
    if (c >= chunks) return;
    const float4 *psi = reinterpret_cast<const float4 *>(slots[s] + (uint64_t)c * (128u * NL));
    float4 v[NL];
    #pragma unroll
    for (int i = 0; i < NL; ++i) v[i] = psi[i * 64 + lane];
    double acc = 0.0;
    #pragma unroll
    for (int i = 0; i < NL; ++i) {
        const double x0 = v[i].x, y0 = v[i].y, x1 = v[i].z, y1 = v[i].w;
        acc += fma(x0, x0, y0 * y0) + fma(x1, x1, y1 * y1);
    }
    #pragma unroll
    for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o, 64);
    if (lane == 0) csum[(uint64_t)s * chunks + c] = acc;
}

// Measurement sums of slot s over chunk c of 2^C amplitudes: the FP64 sum
// of |psi_i|^2 and the same sum over the indices with bit qubit[s] set
// (fixed order: per thread in index order, two amplitudes a 16-byte load,
// then the block sum).
__global__ __launch_bounds__(256) void measure_sum_kernel(const float2 *const *__restrict__ slots,
                                                          const uint32_t *__restrict__ qubit,
                                                          uint32_t C, uint32_t chunks,
                                                          double *__restrict__ part) {
    __shared__ double red[5];
    const uint32_t c = blockIdx.x, s = blockIdx.y;
    const uint64_t first = (uint64_t)c << C;
    const float4 *psi = reinterpret_cast<const float4 *>(slots[s] + first);
    const uint32_t q = qubit[s];
    const uint32_t pairs = 1u << (C - 1);
    double acc = 0.0, acc1 = 0.0;
    #pragma unroll 8
    for (uint32_t i = threadIdx.x; i < pairs; i += 256) {
        const float4 v = psi[i];
        const double x0 = v.x, y0 = v.y, x1 = v.z, y1 = v.w;
        const double w0 = fma(x0, x0, y0 * y0), w1 = fma(x1, x1, y1 * y1);
        acc += w0 + w1;
        if (q == 0) acc1 += w1;
        else if (((first + 2u * i) >> q) & 1ull) acc1 += w0 + w1;
    }
    acc = block_sum<256>(acc, red);
    acc1 = block_sum<256>(acc1, red);
    if (threadIdx.x == 0) {
        part[2 * ((uint64_t)s * chunks + c)] = acc;
        part[2 * ((uint64_t)s * chunks + c) + 1] = acc1;
    }
}

// Chunk sums of slot s added in a fixed order (per thread strided, then the
// block sum): out[2 s] = S, out[2 s + 1] = S1.
__global__ __launch_bounds__(256) void measure_finalize_kernel(const double *__restrict__ part,
                                                               uint32_t chunks,
                                                               double *__restrict__ out) {
    __shared__ double red[5];
    const uint32_t s = blockIdx.x;
    const double *in = part + 2 * (uint64_t)s * chunks;
    double a = 0.0, a1 = 0.0;
    #pragma unroll 4
    for (uint32_t c = threadIdx.x; c < chunks; c += 256) {
        a += in[2 * c];
        a1 += in[2 * c + 1];
    }
    a = block_sum<256>(a, red);
    a1 = block_sum<256>(a1, red);
    if (threadIdx.x == 0) {
        out[2 * s] = a;
        out[2 * s + 1] = a1;
    }
}

// Joint measurement masses: chunk c of slot s (FP64 sum csum[(s <<
// chunks_log2) + c]) lies in one outcome bin, since every measured qubit is
// at or above the chunk bits; bin b of slot s (its measured bits in
// ascending qubit order) is the sum of the chunks whose index has b on the
// measured bits M = mq[s] << shift and any f on the others. A workgroup of
// 256 threads sums one bin with strided f, or, when a bin has fewer than 256
// chunks, 256 / nfree bins at once (nfree threads each), then a fixed tree.
// Bound by latency (each chunk sum is read once, a few MB at most): with one
// thread per bin, 8 bins of a 22-qubit state were 8 serial chains of 2,048
// loads, 1,132 us for 4 states; now 5.7 us.
__global__ __launch_bounds__(256) void bin_mass_kernel(const double *__restrict__ csum,
                                                       uint32_t chunks_log2, uint32_t shift,
                                                       const uint64_t *__restrict__ mq,
                                                       uint32_t bin_stride,
                                                       double *__restrict__ out) {
    __shared__ double red[256];
    const uint32_t s = blockIdx.y, t = threadIdx.x;
    const uint32_t all = (uint32_t)((1ull << chunks_log2) - 1ull);
    const uint32_t M = (uint32_t)(mq[s] << shift), F = all & ~M;
    const uint32_t k = (uint32_t)__popc(M), fl = chunks_log2 - k;
    if (blockIdx.x >= joint_blocks(chunks_log2, k)) return;
    const uint32_t seg = fl < 8u ? fl : 8u;                  // log2 of the threads of one bin
    const uint32_t b = (blockIdx.x << (8u - seg)) + (t >> seg), f0 = t & ((1u << seg) - 1u);
    double a = 0.0;
    if (b < (1u << k)) {
        const double *in = csum + ((uint64_t)s << chunks_log2) + dpdep32(b, M);
        // f0, f0 + 256, ... deposited into F: adding 256 carries through the
        // other bits set to one (no second step when a bin has <= 256 chunks)
        const uint32_t step = fl > 8u ? dpdep32(256u, F) : 0u;
        uint32_t c = dpdep32(f0, F);
        #pragma unroll 8
        for (uint32_t i = 0; i < (1u << (fl - seg)); ++i) {
            a += in[c];
            c = ((c | ~F) + step) & F;
        }
    }
    red[t] = a;
    __syncthreads();
    for (uint32_t h = (1u << seg) >> 1; h > 0; h >>= 1) {
        if (f0 < h) red[t] += red[t + h];
        __syncthreads();
    }
    if (f0 == 0 && b < (1u << k)) out[(uint64_t)s * bin_stride + b] = red[t];
}

// Dense export of a stabilizer state (STAB -> SV): amplitude k is
// 2^{-r/2} i^e when k = x0 ^ (sum of the X parts x_i of the generators whose
// pivot bit p_i is set in d = k ^ x0), e collecting each such generator's
// phase (ph_i, then (-1)^{z_i . cur} as it acts on the current basis state
// cur in increasing i), else 0.
// With a_i = ph_i + 2 z_i . x0, e is the quadratic form sum a_i + 2 sum_{j <
// i} z_i . x_j over the generators i, j present (mod 4). So for any split of
// the pivots into lower and upper ones, e is the lower generators' part plus
// the upper ones' plus cross terms that are linear in the lower ones once the
// upper ones are fixed: twice the parity of a mask lam over d's lower bits
// (export_part). A tile of 2^12 indices takes the generators with pivots
// inside it from one table in LDS (X sum, and the part's two bits on top),
// built once per workgroup from 64 lower and 64 upper entries, and one loop
// over the generators per tile for the rest. An amplitude then costs a table
// read and about ten integer operations; bound by the store. Evaluating r
// generators with 64-bit popcounts per amplitude took 130 us at 24 qubits
// (1.0 TB/s), this takes 32 us (4.2 TB/s).
constexpr int kExportTileBits = 12, kExportSplit = 6;

struct ExportGen {
    uint32_t x, z, a, p, g;   // X and Z parts, a_i, pivot, and the cross mask
};
struct ExportPart {
    uint32_t cur, e, lam;     // X sum, phase, cross mask of the generators below lo
};

// The generators with pivots in [lo, hi) that are present in d.
__device__ __forceinline__ ExportPart export_part(const ExportGen *gen, uint32_t r4, uint32_t d,
                                                  uint32_t lo, uint32_t hi) {
    ExportPart q = {0u, 0u, 0u};
    #pragma unroll 4
    for (uint32_t i = 0; i < r4; ++i) {
        const ExportGen g = gen[i];
        const uint32_t par = (uint32_t)__popc(g.z & q.cur);
        const uint32_t in = g.p >= lo && g.p < hi ? 0u - ((d >> g.p) & 1u) : 0u;
        q.lam ^= g.p < lo ? (par & 1u) << g.p : (g.g & in);
        q.e += (g.a + 2u * par) & in;
        q.cur ^= g.x & in;
    }
    return q;
}

__global__ __launch_bounds__(256) void stab_export_kernel(float2 *__restrict__ psi, uint32_t n,
                                                          uint64_t x0_, uint32_t r,
                                                          const uint64_t *__restrict__ xs,
                                                          const uint64_t *__restrict__ zs,
                                                          const uint32_t *__restrict__ ph,
                                                          const uint32_t *__restrict__ piv,
                                                          float norm) {
    __shared__ ExportGen gen[32];   // r <= n <= 30, padded with absent ones (pivot 31)
    __shared__ ExportPart low[1 << kExportSplit], mid[1 << (kExportTileBits - kExportSplit)];
    __shared__ uint2 tab2[(1 << kExportTileBits) / 2];
    uint32_t *tab = reinterpret_cast<uint32_t *>(tab2);
    const uint32_t T = n < (uint32_t)kExportTileBits ? n : (uint32_t)kExportTileBits;
    const uint32_t L = T < (uint32_t)kExportSplit ? T : (uint32_t)kExportSplit;
    const uint32_t x0 = (uint32_t)x0_, t = threadIdx.x, r4 = (r + 3u) & ~3u;
    if (t < 32u) {
        ExportGen g = {0u, 0u, 0u, 31u, 0u};
        if (t < r) {
            g.x = (uint32_t)xs[t];
            g.z = (uint32_t)zs[t];
            g.p = piv[t];
            g.a = ph[t] + 2u * (uint32_t)__popc(g.z & x0);
        }
        gen[t] = g;
    }
    __syncthreads();
    if (t < r) {
        // cross terms of a generator with the ones before it
        uint32_t g = 0;
        for (uint32_t i = 0; i < t; ++i) g |= ((uint32_t)__popc(gen[t].z & gen[i].x) & 1u) << gen[i].p;
        gen[t].g = g;
    }
    __syncthreads();
    if (t < 64u) {
        if (t < (1u << L)) low[t] = export_part(gen, r4, t ^ x0, 0u, L);
    } else if (t < 128u) {
        const uint32_t m = t - 64u;
        if (m < (1u << (T - L))) mid[m] = export_part(gen, r4, (m << L) ^ x0, L, T);
    }
    __syncthreads();
    const uint32_t lmask = (1u << L) - 1u, tmask = (1u << T) - 1u;
    for (uint32_t l = t; l <= tmask; l += 256) {
        const ExportPart a = low[l & lmask], b = mid[l >> L];
        const uint32_t e = a.e + b.e + 2u * (uint32_t)__popc(b.lam & lmask & (l ^ x0));
        tab[l] = (a.cur ^ b.cur) | (e << 30);
    }
    __syncthreads();
    const uint32_t tiles = 1u << (n - T), pairs = 1u << (T - 1);
    for (uint32_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        const uint32_t base = tile << T;
        const ExportPart hi = export_part(gen, r4, base ^ x0, T, 31u);
        const uint32_t e0 = hi.e, lam = hi.lam & tmask;
        const uint32_t cur = hi.cur ^ x0 ^ base;
        // an amplitude is in the support when cur ^ (its table's X sum) is its tile index
        float4 *out = reinterpret_cast<float4 *>(psi + base);
        auto amp = [&](uint32_t l, uint32_t w, float &re, float &im) {
            const uint32_t e = e0 + (w >> 30) + 2u * (uint32_t)__popc(lam & (l ^ x0));
            const bool in = ((cur ^ w) & 0x3FFFFFFFu) == l;
            const float v = in ? ((e & 2u) ? -norm : norm) : 0.0f;
            re = (e & 1u) ? 0.0f : v;
            im = (e & 1u) ? v : 0.0f;
        };
        #pragma unroll 4
        for (uint32_t q = t; q < pairs; q += 256) {
            const uint2 w = tab2[q];
            float4 o;
            amp(2u * q, w.x, o.x, o.y);
            amp(2u * q + 1u, w.y, o.z, o.w);
            out[q] = o;
        }
    }
}

// Exclusive prefix of a slot's chunk sums and its total, in FP64 with a
// fixed order: blocks of 1,024 threads * PER consecutive chunks, per thread in
// order, thread sums by a wave scan, wave sums in order, blocks in order. One
// workgroup per slot; PER = 16 takes its chunks through LDS (rows of 16 padded
// to 17) so that global accesses stay coalesced, PER = 1 serves states of at
// most 1,024 chunks (20 qubits). Bound by latency and one CU's access rate:
// 256 threads that walked 64 chunks each twice, with a serial scan of the 256
// sums between, took 32 us for one 24-qubit state (16,384 chunks); 16
// consecutive loads a thread straight from memory 18 us; this 8.0 us.
template <int PER>
__global__ __launch_bounds__(1024) void chunk_scan_kernel(const double *__restrict__ csum,
                                                          uint32_t chunks,
                                                          double *__restrict__ cpre,
                                                          double *__restrict__ total) {
    __shared__ double wsum[16];
    __shared__ double stage[PER > 1 ? 1024 * (PER + 1) : 1];
    const uint32_t s = blockIdx.x, t = threadIdx.x, lane = t & 63u, wave = t >> 6;
    const double *in = csum + (uint64_t)s * chunks;
    double *outp = cpre + (uint64_t)s * chunks;
    auto at = [](uint32_t c) { return c + c / PER; };
    double carry = 0.0;
    for (uint32_t b0 = 0; b0 < chunks; b0 += 1024u * PER) {
        double v[PER], acc = 0.0;
        #pragma unroll
        for (uint32_t i = 0; i < PER; ++i) {
            const uint32_t c = i * 1024u + t;
            v[i] = b0 + c < chunks ? in[b0 + c] : 0.0;
        }
        if constexpr (PER > 1) {
            #pragma unroll
            for (uint32_t i = 0; i < PER; ++i) stage[at(i * 1024u + t)] = v[i];
            __syncthreads();
            #pragma unroll
            for (uint32_t i = 0; i < PER; ++i) v[i] = stage[at(t * PER + i)];
        }
        #pragma unroll
        for (uint32_t i = 0; i < PER; ++i) acc += v[i];
        double x = acc;   // inclusive wave scan of the thread sums
        #pragma unroll
        for (uint32_t o = 1; o < 64u; o <<= 1) {
            const double y = __shfl_up(x, o, 64);
            if (lane >= o) x += y;
        }
        if (lane == 63u) wsum[wave] = x;
        __syncthreads();
        double off = carry, all = carry;
        #pragma unroll
        for (uint32_t w = 0; w < 16u; ++w) {
            if (w < wave) off += wsum[w];
            all += wsum[w];
        }
        const double before = __shfl_up(x, 1, 64);
        double run = lane ? off + before : off;
        #pragma unroll
        for (uint32_t i = 0; i < PER; ++i) {
            const double r = run;
            run += v[i];
            v[i] = r;
        }
        if constexpr (PER > 1) {
            #pragma unroll
            for (uint32_t i = 0; i < PER; ++i) stage[at(t * PER + i)] = v[i];   // the thread's own entries
            __syncthreads();
            #pragma unroll
            for (uint32_t i = 0; i < PER; ++i) v[i] = stage[at(i * 1024u + t)];
        }
        #pragma unroll
        for (uint32_t i = 0; i < PER; ++i) {
            const uint32_t c = b0 + i * 1024u + t;
            if (c < chunks) outp[c] = v[i];
        }
        carry = all;
        __syncthreads();
    }
    if (t == 0) total[s] = carry;
}

// Sub-chunk (64 amplitudes) and chunk (1,024) sums of |psi|^2 (FP64) for the
// sampler, one wave per chunk; grid (chunks / 4, slots). A lane takes two
// amplitudes of each of 8 sub-chunks (8 loads of 16 bytes, all in flight); a
// sub-chunk's 32 lane values are added by the butterfly 16, 8, 4, 2, 1, the
// number of sub-chunks per lane halving in its first three steps; the chunk
// sum is the sequential sum of its sub-chunk sums. Bound by the one read of
// the state: a workgroup per chunk with one load a lane at a time read a
// 24-qubit state at 4.7 TB/s (28.5 us), this takes 20.5 us (6.5 TB/s).
__global__ __launch_bounds__(256) void sub_sum_kernel(const float2 *const *__restrict__ slots,
                                                      uint32_t chunks, double *__restrict__ csum,
                                                      double *__restrict__ ssum) {
    __shared__ double subs[4][16];
    const uint32_t wave = threadIdx.x >> 6, lane = threadIdx.x & 63u;
    const uint32_t c = blockIdx.x * 4u + wave, s = blockIdx.y;
    const bool ok = c < chunks;
    if (ok) {
        const float4 *psi = reinterpret_cast<const float4 *>(slots[s] + ((uint64_t)c << 10));
        float4 a[8];
        #pragma unroll
        for (int i = 0; i < 8; ++i) a[i] = psi[i * 64 + lane];
        double v[8];   // sub-chunk 2 i + (lane >> 5)
        #pragma unroll
        for (int i = 0; i < 8; ++i) {
            const double x0 = a[i].x, y0 = a[i].y, x1 = a[i].z, y1 = a[i].w;
            v[i] = fma(x0, x0, y0 * y0) + fma(x1, x1, y1 * y1);
        }
        const bool b4 = lane & 16u, b3 = lane & 8u, b2 = lane & 4u;
        double f[4], g[2], h;
        #pragma unroll
        for (int i = 0; i < 4; ++i) f[i] = (b4 ? v[4 + i] : v[i]) + __shfl_xor(b4 ? v[i] : v[4 + i], 16, 64);
        #pragma unroll
        for (int i = 0; i < 2; ++i) g[i] = (b3 ? f[2 + i] : f[i]) + __shfl_xor(b3 ? f[i] : f[2 + i], 8, 64);
        h = (b2 ? g[1] : g[0]) + __shfl_xor(b2 ? g[0] : g[1], 4, 64);
        h += __shfl_xor(h, 2, 64);
        h += __shfl_xor(h, 1, 64);
        // lane bits 4, 3, 2 hold the load index, bit 5 the half
        if ((lane & 3u) == 0u) {
            const uint32_t i = 4u * ((lane >> 4) & 1u) + 2u * ((lane >> 3) & 1u) + ((lane >> 2) & 1u);
            const uint32_t j = 2u * i + (lane >> 5);
            subs[wave][j] = h;
            ssum[((uint64_t)s * chunks + c) * 16u + j] = h;
        }
    }
    __syncthreads();
    if (ok && lane == 0) {
        double acc = 0.0;
        #pragma unroll
        for (int j = 0; j < 16; ++j) acc += subs[wave][j];
        csum[(uint64_t)s * chunks + c] = acc;
    }
}

// The same for states below 10 qubits: one chunk of 2^n amplitudes, its
// sub-chunks of 2^S (S <= 6) summed by one amplitude per lane.
__global__ __launch_bounds__(256) void sub_sum_small_kernel(const float2 *const *__restrict__ slots,
                                                            uint32_t n, uint32_t S,
                                                            double *__restrict__ csum,
                                                            double *__restrict__ ssum) {
    __shared__ double subs[8];
    const uint32_t s = blockIdx.x, spc = 1u << (n - S), L = 1u << S;
    const float2 *psi = slots[s];
    const uint32_t wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    for (uint32_t j = wave; j < spc; j += 4) {
        double v = 0.0;
        if (lane < L) {
            const float2 a = psi[(j << S) + lane];
            const double x = a.x, y = a.y;
            v = fma(x, x, y * y);
        }
        for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
        if (lane == 0) {
            subs[j] = v;
            ssum[(uint64_t)s * spc + j] = v;
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double acc = 0.0;
        for (uint32_t j = 0; j < spc; ++j) acc += subs[j];
        csum[s] = acc;
    }
}

// Draws. The target u * total of a shot is located by a search over the chunk
// prefixes, a scan of the chunk's (at most 16) sub-chunk sums and a scan of one
// sub-chunk's (at most 64) amplitudes, the running sum continuing in FP64 from
// the chunk prefix, one element after the other. Where rounding leaves the
// target past a level's last element, that level's last element of non-zero
// mass is taken, so every outcome has non-zero probability.
//
// Few shots: 8 lanes per shot, 32 shots per workgroup. They are bound by the
// chain of dependent loads, which 8 lanes shorten (one thread per shot waited
// for log2(chunks) + up to 80 of them); the amplitudes of the 32 shots go
// through LDS and one lane per shot adds them. 1,024 shots of a 24-qubit state:
// 21 us with one thread per shot, 8.4 us like this.
constexpr uint32_t kDrawLanes = 8, kDrawShots = 256 / kDrawLanes;

__global__ __launch_bounds__(256) void draw_kernel(const float2 *const *__restrict__ slots,
                                                   uint32_t n_slots, uint32_t C, uint32_t S,
                                                   uint32_t chunks, const double *__restrict__ csum,
                                                   const double *__restrict__ cpre,
                                                   const double *__restrict__ ssum,
                                                   const double *__restrict__ total,
                                                   uint64_t seed, uint64_t task_base,
                                                   uint32_t shots, uint32_t *__restrict__ out) {
    __shared__ double sub[kDrawShots][17];
    __shared__ double prob[kDrawShots][65];   // (odd row lengths: the shots' columns lie in other banks)
    __shared__ double s_at[kDrawShots], s_target[kDrawShots];
    __shared__ uint32_t s_base[kDrawShots];
    const uint32_t lane = threadIdx.x & (kDrawLanes - 1), shot = threadIdx.x / kDrawLanes;
    const uint32_t group = (threadIdx.x & 63u) & ~(kDrawLanes - 1);
    const uint32_t spc = 1u << (C - S), L = 1u << S;
    const uint32_t all = n_slots * shots, first = blockIdx.x * kDrawShots;   // at most kDrawMany
    const uint32_t gid = first + shot < all ? first + shot : all - 1;   // idle groups repeat the last shot
    const uint32_t s = gid / shots, sh = gid - s * shots;
    const uint64_t h = splitmix(seed ^ (((task_base + s) << 32) + sh));
    const double u = (double)(h >> 11) * (1.0 / 9007199254740992.0);
    const double target = u * total[s];
    const double *pre = cpre + (uint64_t)s * chunks;
    const double *cs = csum + (uint64_t)s * chunks;
    // last chunk with pre[c] <= target, then back over chunks without mass
    uint32_t lo = 0, len = chunks;
    while (len > 1u) {
        const uint32_t stride = len >= kDrawLanes ? len / kDrawLanes : 1u;
        const bool in = lane * stride < len && pre[lo + lane * stride] <= target;
        const uint32_t hit = (uint32_t)(__ballot(in) >> group) & ((1u << kDrawLanes) - 1u);
        lo += hit ? (31u - (uint32_t)__clz(hit)) * stride : 0u;
        len = stride;
    }
    while (lo > 0 && cs[lo] == 0.0) --lo;
    const double *sb = ssum + ((uint64_t)s * chunks + lo) * spc;
    double run = pre[lo], run_last = run;
    #pragma unroll
    for (uint32_t i = 0; i < 16 / kDrawLanes; ++i)
        if (i * kDrawLanes + lane < spc) sub[shot][i * kDrawLanes + lane] = sb[i * kDrawLanes + lane];
    lds_wave_sync();
    // j: the first element that takes the running sum past the target
    // (counted without branches), else the last one of non-zero mass
    uint32_t j = 0, last_j = 0;
    double at = run;   // running sum before element j
    bool past = false;
    #pragma unroll 4
    for (uint32_t k = 0; k < spc; ++k) {
        const double v = sub[shot][k];
        at = past ? at : run;
        last_j = v > 0.0 ? k : last_j;
        run_last = v > 0.0 ? run : run_last;
        run += v;
        past = past || run > target;
        j += past ? 0u : 1u;
    }
    if (!past) {
        j = last_j;
        at = run_last;
    }
    const uint64_t base = ((uint64_t)lo << C) + ((uint64_t)j << S);
    const float2 *psi = slots[s] + base;
    #pragma unroll
    for (uint32_t i = 0; i < 64 / kDrawLanes; ++i) {
        const uint32_t l = i * kDrawLanes + lane;
        if (l < L) {
            const float2 a = psi[l];
            const double x = a.x, y = a.y;
            prob[shot][l] = fma(x, x, y * y);
        }
    }
    if (lane == 0) {
        s_at[shot] = at;
        s_target[shot] = target;
        s_base[shot] = (uint32_t)base;
    }
    __syncthreads();
    const uint32_t q = threadIdx.x;
    if (q < kDrawShots && first + q < all) {
        const double tq = s_target[q];
        double rq = s_at[q];
        uint32_t res = 0, last_i = 0;
        bool over = false;
        auto step = [&](uint32_t i) {
            const double pr = prob[q][i];
            rq += pr;
            last_i = pr > 0.0 ? i : last_i;
            over = over || rq > tq;
            res += over ? 0u : 1u;
        };
        if (L == 64u) {
            #pragma unroll
            for (uint32_t i = 0; i < 64u; ++i) step(i);
        } else {
            for (uint32_t i = 0; i < L; ++i) step(i);
        }
        if (!over) res = last_i;
        out[first + q] = s_base[q] + res;
    }
}

// Many shots (more than kDrawMany): one thread per shot. They are bound by the
// scans' additions; with 8 lanes a shot one of a workgroup's four waves adds,
// and all 64 amplitudes of its 32 shots whatever the state. Here every thread
// adds, and stops after the 4 sums and the 8 amplitudes (64 bytes, all loads in
// flight) in which its target lies. Whole calls with 8 lanes a shot / like this
// (with one thread a shot and a load for every element): 65,536 shots of 64
// 18-qubit states, spread 721 / 331 us (688), GHZ 522 / 159 (222), |0...0>
// 499 / 67 (67); 2^20 shots of a 26-qubit state 410 / 283 (633). The line:
// 32,768 shots of an 18-qubit state 17.3 / 18.5, 65,536 22.3 / 18.9. Loads of 16
// amplitudes gain 4 % on 18 to 26 spread qubits and lose 6 % on 14 (223 / 237).
constexpr uint64_t kDrawMany = 49152;

template <bool WIDE>
__global__ __launch_bounds__(256) void draw_many_kernel(
    const float2 *const *__restrict__ slots, uint32_t n_slots, uint32_t C, uint32_t S, uint32_t chunks,
    const double *__restrict__ csum, const double *__restrict__ cpre, const double *__restrict__ ssum,
    const double *__restrict__ total, uint64_t seed, uint64_t task_base, uint32_t shots,
    uint32_t *__restrict__ out) {
    const uint64_t gid = (uint64_t)blockIdx.x * 256 + threadIdx.x, all = (uint64_t)n_slots * shots;
    if (gid >= all) return;
    uint32_t s, sh;
    if (all <= 0xFFFFFFFFull) {   // a 32-bit division where it suffices
        s = (uint32_t)gid / shots;
        sh = (uint32_t)gid - s * shots;
    } else {
        s = (uint32_t)(gid / shots);
        sh = (uint32_t)(gid % shots);
    }
    const uint64_t h = splitmix(seed ^ (((task_base + s) << 32) + sh));
    const double u = (double)(h >> 11) * (1.0 / 9007199254740992.0);
    const double target = u * total[s];
    const double *pre = cpre + (uint64_t)s * chunks;
    const double *cs = csum + (uint64_t)s * chunks;
    // last chunk with pre[c] <= target, then back over chunks without mass
    uint32_t lo = 0;
    for (uint32_t half = chunks >> 1; half > 0; half >>= 1)
        if (pre[lo + half] <= target) lo += half;
    while (lo > 0 && cs[lo] == 0.0) --lo;
    const uint32_t spc = 1u << (C - S), L = 1u << S;
    const double *sb = ssum + ((uint64_t)s * chunks + lo) * spc;
    // j: the first element that takes the running sum past the target, else
    // the last one of non-zero mass (the zeros after spc change neither)
    double run = pre[lo], at = run, run_last = run;
    uint32_t j = 0, last_j = 0;
    bool past = false;
    #pragma unroll
    for (uint32_t k0 = 0; k0 < 16; k0 += 4) {
        if (past) continue;
        double v[4];
        #pragma unroll
        for (uint32_t i = 0; i < 4; ++i) v[i] = k0 + i < spc ? sb[k0 + i] : 0.0;
        #pragma unroll
        for (uint32_t i = 0; i < 4; ++i) {
            at = past ? at : run;
            last_j = v[i] > 0.0 ? k0 + i : last_j;
            run_last = v[i] > 0.0 ? run : run_last;
            run += v[i];
            past = past || run > target;
            j += past ? 0u : 1u;
        }
    }
    if (!past) {
        j = last_j;
        at = run_last;
    }
    const uint64_t base = ((uint64_t)lo << C) + ((uint64_t)j << S);
    const float2 *psi = slots[s] + base;
    uint32_t res = 0, last_i = 0;
    bool over = false;
    auto step = [&](uint32_t i, float re, float im) {
        const double x = re, y = im, pr = fma(x, x, y * y);
        at += pr;
        last_i = pr > 0.0 ? i : last_i;
        over = over || at > target;
        res += over ? 0u : 1u;
    };
    if constexpr (WIDE) {
        const float4 *p4 = reinterpret_cast<const float4 *>(psi);
        #pragma unroll 1
        for (uint32_t b = 0; b < 64u && !over; b += 8u) {
            float4 q[4];
            #pragma unroll
            for (uint32_t i = 0; i < 4; ++i) q[i] = p4[(b >> 1) + i];
            #pragma unroll
            for (uint32_t i = 0; i < 4; i += 2) {
                if (over) continue;
                step(b + 2 * i, q[i].x, q[i].y);
                step(b + 2 * i + 1, q[i].z, q[i].w);
                step(b + 2 * i + 2, q[i + 1].x, q[i + 1].y);
                step(b + 2 * i + 3, q[i + 1].z, q[i + 1].w);
            }
        }
    } else {
        for (uint32_t i = 0; i < L && !over; ++i) step(i, psi[i].x, psi[i].y);
    }
    out[gid] = (uint32_t)base + (over ? res : last_i);
}

// ------------------------------------------------------------- launchers
static_assert(sizeof(float2) == 8, "float2");

static uint32_t cu_count() {
    static uint32_t cached = 0;
    if (cached) return cached;
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) == hipSuccess &&
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess &&
        cus > 0)
        cached = (uint32_t)cus;
    else
        cached = 256;
    return cached;
}

hipError_t launch_pass(hipStream_t st, const PassDesc *d, uint32_t n_descs, uint32_t n,
                       uint32_t m, int remap, bool use_lds) {
    if (n_descs == 0) return hipSuccess;
    if (m < (uint32_t)kMinTileBits) {
        hipLaunchKernelGGL(small_pass_kernel, dim3(n_descs), dim3(64), 0, st, d, n);
        return hipGetLastError();
    }
    if (m > (uint32_t)kMaxTileBits) return hipErrorInvalidValue;
    const uint64_t items64 = (uint64_t)n_descs << (n - m);
    const uint32_t T = 1u << (m - 4), wg = T < 256 ? T : 256, parts = T / wg;
    if (items64 * parts > 0x7FFFFFF8ull) return hipErrorInvalidValue;
    const uint32_t items = (uint32_t)items64;
    if (use_lds) {
        // one persistent workgroup per CU, more of smaller tiles (a multiple
        // of 8 for the XCD split)
        const uint32_t full = cu_count() * (1024u / T < 8u ? 1024u / T : 8u);
        const uint32_t need = ((items + 7u) / 8u) * 8u;
        const uint32_t grid = ((std::min(full, need) + 7u) / 8u) * 8u;
        hipLaunchKernelGGL(pass_kernel_lds, dim3(grid), dim3(T), sizeof(float2) << m, st, d, n_descs, items);
    } else {
        uint32_t grid = items * parts;
        if (remap) grid = ((grid + 7u) / 8u) * 8u;
        hipLaunchKernelGGL(pass_kernel_flat, dim3(grid), dim3(wg), 0, st, d, n_descs, parts, items, remap);
    }
    return hipGetLastError();
}

hipError_t launch_norm_finalize(hipStream_t st, const PassDesc *d, uint32_t n_descs,
                                uint32_t tiles) {
    if (n_descs == 0) return hipSuccess;
    hipLaunchKernelGGL(norm_finalize_kernel, dim3(n_descs), dim3(256), 0, st, d, tiles);
    return hipGetLastError();
}

hipError_t launch_upload(hipStream_t st, void *dst, const void *src, uint64_t bytes, uint32_t *done,
                         uint32_t seq, uint32_t *blocks) {
    const uint64_t count = (bytes + 15) / 16;
    if (count > 0xFFFFFFFFull - 1024ull * kUploadBlocks) return hipErrorInvalidValue;
    *blocks = upload_blocks(bytes);
    hipLaunchKernelGGL(upload_kernel, dim3(*blocks), dim3(1024), 0, st, static_cast<uint4 *>(dst),
                       static_cast<const uint4 *>(src), (uint32_t)count, done, seq);
    return hipGetLastError();
}

hipError_t launch_init(hipStream_t st, void *base, uint32_t n, uint32_t n_slots) {
    const uint64_t slot_f4 = (1ull << n) / 2;
    if (slot_f4 == 0) {
        // n == 0 is rejected by the host; keep the kernel safe anyway
        return hipErrorInvalidValue;
    }
    const uint64_t total = slot_f4 * n_slots, bytes = total * sizeof(float4);
    if (total == 0) return hipSuccess;
    // Up to the last-level cache's size four at a time (128 MiB 16.2 us, one at
    // a time 16.6). Above it the write order decides: one at a time below 1 GiB
    // (384 MiB 61, four 70; 768 MiB 128, 132) and from 4 GiB (722, 733), four in
    // between (1 GiB 183, four 177; 1.5 GiB 270, 273; 2 GiB 375, 363).
    const bool fits = bytes <= kIoCacheBytes, mid = bytes >= (1ull << 30) && bytes < (4ull << 30);
    const uint64_t per = 256 * (fits || mid ? 4 : 1);
    const uint64_t blocks = std::min<uint64_t>((total + per - 1) / per, 65536);
    auto *kernel = fits ? init_kernel<4, true> : mid ? init_kernel<4, false> : init_kernel<1, true>;
    hipLaunchKernelGGL(kernel, dim3((uint32_t)blocks), dim3(256), 0, st, reinterpret_cast<float4 *>(base),
                       slot_f4, total);
    return hipGetLastError();
}

hipError_t launch_copy(hipStream_t st, void *dst, const void *src, uint64_t bytes) {
    const uint64_t count = bytes / 16;
    uint64_t blocks = (count + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    if (blocks == 0) return hipSuccess;
    hipLaunchKernelGGL(copy_kernel, dim3((uint32_t)blocks), dim3(256), 0, st,
                       reinterpret_cast<float4 *>(dst), reinterpret_cast<const float4 *>(src),
                       count);
    return hipGetLastError();
}

hipError_t launch_reduce(hipStream_t st, const ReduceDesc *d, uint32_t n_descs, uint32_t n,
                         uint32_t M) {
    const uint64_t tiles = 1ull << (n - M);
    const uint64_t items = (uint64_t)n_descs * (tiles / red_row_tiles((uint32_t)tiles));
    if (items == 0) return hipSuccess;
    if (items > 0x7FFFFFFFull) return hipErrorInvalidValue;
    switch (M) {
#define QW_RED(MM)                                                                       \
    case MM:                                                                             \
        hipLaunchKernelGGL(reduce_kernel<MM>, dim3((uint32_t)items), dim3(1 << (MM - 4)), 0, st, \
                           d, n_descs, n, (uint32_t)items);                              \
        break;
        QW_RED(10) QW_RED(11) QW_RED(12) QW_RED(13) QW_RED(14)
#undef QW_RED
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_reduce_small(hipStream_t st, const ReduceDescSmall *d, uint32_t n_descs,
                               uint32_t n) {
    if (n_descs == 0) return hipSuccess;
    hipLaunchKernelGGL(reduce_small_kernel, dim3(n_descs), dim3(64 * kSmallWaves), 0, st, d, n);
    return hipGetLastError();
}

hipError_t launch_row_sum(hipStream_t st, const RowSum *src, uint32_t n_src, uint32_t n_chunks, double *part,
                          uint32_t n_terms, uint32_t tiles, uint32_t n_slots, uint32_t T) {
    const uint32_t rows = tiles / red_row_tiles(tiles);
    if (n_chunks == 0 || n_slots == 0) return hipSuccess;
    if (T < 64 || T > 1024 || n_slots > 65535 || rows > 65535) return hipErrorInvalidValue;
    hipLaunchKernelGGL(row_sum_kernel, dim3(n_chunks, rows, n_slots), dim3(T), 0, st, src, n_src, part,
                       n_terms, tiles);
    return hipGetLastError();
}

hipError_t launch_expect_finalize(hipStream_t st, const double *part, const double *coeff,
                                  uint32_t n_terms, uint32_t rows, uint32_t n_slots,
                                  double *out) {
    if (n_slots == 0) return hipSuccess;
    hipLaunchKernelGGL(expect_finalize_kernel, dim3(n_slots), dim3(64 * kFinalizeWaves), 0, st, part, coeff,
                       n_terms, rows, out);
    return hipGetLastError();
}

hipError_t launch_sample(hipStream_t st, const float2 *const *slots, uint32_t n_slots,
                         uint32_t n, double *csum, double *cpre, double *ssum, double *total,
                         uint64_t seed, uint64_t task_base, uint32_t shots, uint32_t *out) {
    const uint32_t C = sample_chunk_bits(n), S = sample_sub_bits(n);
    const uint32_t chunks = 1u << (n - C);
    if (C == 10)
        hipLaunchKernelGGL(sub_sum_kernel, dim3((chunks + 3) / 4, n_slots), dim3(256), 0, st, slots, chunks,
                           csum, ssum);
    else
        hipLaunchKernelGGL(sub_sum_small_kernel, dim3(n_slots), dim3(256), 0, st, slots, C, S, csum, ssum);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (chunks > 1024)
        hipLaunchKernelGGL(chunk_scan_kernel<16>, dim3(n_slots), dim3(1024), 0, st, csum, chunks, cpre, total);
    else
        hipLaunchKernelGGL(chunk_scan_kernel<1>, dim3(n_slots), dim3(1024), 0, st, csum, chunks, cpre, total);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    const uint64_t draws = (uint64_t)n_slots * shots;
    if (draws == 0) return hipSuccess;
    if (draws > kDrawMany) {
        const uint64_t groups = (draws + 255) / 256;
        if (groups > 0x7FFFFFFFull) return hipErrorInvalidValue;
        auto *kernel = S == 6 ? draw_many_kernel<true> : draw_many_kernel<false>;
        hipLaunchKernelGGL(kernel, dim3((uint32_t)groups), dim3(256), 0, st, slots, n_slots, C, S, chunks, csum,
                           cpre, ssum, total, seed, task_base, shots, out);
        return hipGetLastError();
    }
    const uint32_t blocks = (uint32_t)((draws + kDrawShots - 1) / kDrawShots);
    hipLaunchKernelGGL(draw_kernel, dim3(blocks), dim3(256), 0, st, slots, n_slots, C, S, chunks, csum, cpre,
                       ssum, total, seed, task_base, shots, out);
    return hipGetLastError();
}

hipError_t launch_measure_sums(hipStream_t st, const float2 *const *slots, const uint32_t *qubit,
                               uint32_t n_slots, uint32_t n, double *part, double *out) {
    if (n_slots == 0) return hipSuccess;
    const uint32_t C = n < 12 ? n : 12;
    const uint32_t chunks = 1u << (n - C);
    hipLaunchKernelGGL(measure_sum_kernel, dim3(chunks, n_slots), dim3(256), 0, st, slots, qubit, C,
                       chunks, part);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(measure_finalize_kernel, dim3(n_slots), dim3(256), 0, st, part, chunks, out);
    return hipGetLastError();
}

hipError_t launch_joint_masses(hipStream_t st, const float2 *const *slots, const uint64_t *mq,
                               uint32_t n_slots, uint32_t n, uint32_t C, uint32_t max_blocks,
                               double *csum, uint32_t bin_stride, double *out) {
    if (n_slots == 0) return hipSuccess;
    const uint32_t cb = joint_chunk_bits(C), chunks = 1u << (n - cb);
    const dim3 grid((chunks + 3) / 4, n_slots), wg(256);
    if (cb == 8) hipLaunchKernelGGL(mass_sum_kernel<2>, grid, wg, 0, st, slots, chunks, csum);
    else if (cb == 9) hipLaunchKernelGGL(mass_sum_kernel<4>, grid, wg, 0, st, slots, chunks, csum);
    else if (cb == 10) hipLaunchKernelGGL(mass_sum_kernel<8>, grid, wg, 0, st, slots, chunks, csum);
    else return hipErrorInvalidValue;
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(bin_mass_kernel, dim3(max_blocks, n_slots), dim3(256), 0, st, csum, n - cb, C - cb, mq,
                       bin_stride, out);
    return hipGetLastError();
}

namespace {

// One workgroup per task. A joint cluster's bin masses are staged in LDS;
// each step sums those with the step's bit clear and set with a fixed order
// (per-thread strided sums, a wave butterfly, then the waves in order),
// decides, and keeps the bins that agree with the outcome: bin b moves to b
// with bit p removed, which keeps their order. Bound by latency: two barriers
// a step instead of a tree of nine through LDS (11 measurements: 20 us, now
// 14 us).
constexpr int kDecideThreads = 256;

__device__ __forceinline__ void decide_sums(const double *mass, uint32_t len, uint32_t p, double *red,
                                            double *zero, double *one) {
    const uint32_t t = threadIdx.x;
    double a0 = 0.0, a1 = 0.0;
    for (uint32_t b = t; b < len; b += kDecideThreads) {
        const double v = mass[b];
        if ((b >> p) & 1u) a1 += v;
        else a0 += v;
    }
    #pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        a0 += __shfl_xor(a0, o, 64);
        a1 += __shfl_xor(a1, o, 64);
    }
    if ((t & 63u) == 0) {
        red[2 * (t >> 6)] = a0;
        red[2 * (t >> 6) + 1] = a1;
    }
    __syncthreads();
    a0 = red[0];
    a1 = red[1];
    #pragma unroll
    for (int w = 1; w < kDecideThreads / 64; ++w) {
        a0 += red[2 * w];
        a1 += red[2 * w + 1];
    }
    *zero = a0;
    *one = a1;
}

__global__ __launch_bounds__(kDecideThreads) void meas_decide_kernel(
    const uint32_t *__restrict__ task_first, const uint32_t *__restrict__ task_count,
    const MeasDec *__restrict__ dec, uint32_t n_tasks, int joint, double *__restrict__ sums,
    uint32_t bin_stride, float *__restrict__ dyn, uint8_t *__restrict__ outc, uint32_t *__restrict__ err) {
    __shared__ double buf[2][1u << 12];
    __shared__ double red[2 * (kDecideThreads / 64)];
    __shared__ MeasDec sd[12];   // the task's measurements (k <= 12, the caller's cluster bound)
    const uint32_t i = blockIdx.x, t = threadIdx.x;
    if (i >= n_tasks) return;
    const uint32_t k = task_count[i];
    if (t < k) sd[t] = dec[task_first[i] + t];
    __syncthreads();
    uint32_t bits = 0;     // outcome of measurement j in bit j
    double chosen = 1.0;   // mass of the chosen outcome
    bool zero = false;
    if (!joint) {
        const double S = sums[2 * i], S1 = sums[2 * i + 1];
        if (!(S > 0.0)) {
            zero = true;
        } else {
            const uint32_t b = sd[0].u < S1 / S ? 1u : 0u;
            bits = b;
            chosen = b ? S1 : S - S1;
        }
    } else {
        uint32_t len = 1u << k;  // k <= 12 (the caller's cluster bound)
        const double *src = sums + (size_t)i * bin_stride;
        for (uint32_t b = t; b < len; b += kDecideThreads) buf[0][b] = src[b];
        __syncthreads();
        int cur = 0;
        for (uint32_t j = 0; j < k && !zero; ++j) {
            const uint32_t p = sd[j].pos;
            double none, one;
            decide_sums(buf[cur], len, p, red, &none, &one);
            const double tot = none + one;
            if (j == 0 && !(tot > 0.0)) {
                zero = true;   // the same in every thread
                break;
            }
            const uint32_t bit = sd[j].u < one / tot ? 1u : 0u;
            bits |= bit << j;
            const uint32_t lo = (1u << p) - 1u;
            for (uint32_t b = t; b < len; b += kDecideThreads)
                if (((b >> p) & 1u) == bit) buf[cur ^ 1][((b >> (p + 1)) << p) | (b & lo)] = buf[cur][b];
            __syncthreads();   // also: every thread has read red
            cur ^= 1;
            len >>= 1;
        }
        chosen = buf[cur][0];
    }
    if (zero) {
        if (t == 0) *err = 1u;
        chosen = 1.0;
    }
    if (t >= k) return;
    const float fac = (float)(1.0 / sqrt(chosen));
    const MeasDec &m = sd[t];   // one thread per measurement
    const uint32_t b = (bits >> t) & 1u;
    const float f = t == 0 ? fac : 1.0f;
    float *e = dyn + 4ull * m.dyn;
    // [[e0, e1], [e2, e3]]: P0 = diag(f, 0), P1 = diag(0, f), X P1 = [[0, f], [0, 0]]
    e[0] = b ? 0.0f : f;
    e[1] = (b && m.reset) ? f : 0.0f;
    e[2] = 0.0f;
    e[3] = (b && !m.reset) ? f : 0.0f;
    outc[m.outc] = (uint8_t)b;
}

__global__ void meas_clear_kernel(uint32_t *err) {
    if (threadIdx.x == 0) *err = 0u;
}

__global__ void zero_words_kernel(uint32_t *p, uint64_t count) {
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count;
         i += (uint64_t)gridDim.x * blockDim.x)
        p[i] = 0u;
}

}  // namespace

hipError_t launch_meas_decide(hipStream_t st, const uint32_t *task_first, const uint32_t *task_count,
                              const MeasDec *dec, uint32_t n_tasks, int joint, double *sums,
                              uint32_t bin_stride, float *dyn, uint8_t *outc, uint32_t *err) {
    if (n_tasks == 0) return hipSuccess;
    hipLaunchKernelGGL(meas_decide_kernel, dim3(n_tasks), dim3(kDecideThreads), 0, st, task_first, task_count,
                       dec, n_tasks, joint, sums, bin_stride, dyn, outc, err);
    return hipGetLastError();
}

hipError_t launch_meas_clear(hipStream_t st, uint32_t *err) {
    hipLaunchKernelGGL(meas_clear_kernel, dim3(1), dim3(64), 0, st, err);
    return hipGetLastError();
}

hipError_t launch_zero_words(hipStream_t st, uint32_t *p, uint64_t count) {
    if (count == 0) return hipSuccess;
    const uint64_t blocks = std::min<uint64_t>((count + 255) / 256, 1024);
    hipLaunchKernelGGL(zero_words_kernel, dim3((uint32_t)blocks), dim3(256), 0, st, p, count);
    return hipGetLastError();
}

hipError_t launch_stab_export(hipStream_t st, float2 *psi, uint32_t n, uint64_t x0, uint32_t r,
                              const uint64_t *xs, const uint64_t *zs, const uint32_t *ph,
                              const uint32_t *piv, float norm) {
    if (n > 30 || r > n) return hipErrorInvalidValue;   // the kernel holds 32 generators in 32-bit words
    const uint32_t tiles = n > (uint32_t)kExportTileBits ? 1u << (n - kExportTileBits) : 1u;
    const uint32_t blocks = std::min(tiles, 2048u);
    hipLaunchKernelGGL(stab_export_kernel, dim3((uint32_t)blocks), dim3(256), 0, st, psi, n, x0, r, xs, zs,
                       ph, piv, norm);
    return hipGetLastError();
}

hipError_t kernels_init() { return hipSuccess; }

}  // namespace qw
