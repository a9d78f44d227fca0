// Value enhancement (paper Section 3.2, Eq. 3): the values that enter attention are V + log(s), where s is
// the number of tokens merged into each token; the logarithm is added to every channel of the token's row.
//
// A wavefront owns two consecutive rows and goes through their 16-byte pieces as one list, four per lane in flight; the
// first four are requested before the fp64 logarithms of the two sizes are taken.  The sum is formed in fp64 and rounded
// once.  Bound: HBM, 2 * rows * D * e bytes; short inputs are bound by the latency of one wavefront, so a wavefront has
// little to do one after the other (8 x 32 x 32 x 1280 bf16: 15.5 us with eight rows per
// wavefront, 9.6 with two).
#include <type_traits>

#include "common.hpp"
#include "oim.hpp"

namespace luvc {

constexpr int kVeRows = 2, kVePieces = 4;

template <typename T, bool VECTOR>
__global__ void __launch_bounds__(256)
value_enhance(const T* __restrict__ v, const int32_t* __restrict__ sizes, int64_t rows, int D, int64_t v_stride, int64_t out_stride,
              T* __restrict__ out)
{
    using tr = io_traits<T>;
    constexpr int V = tr::kVec;
    const int lane = threadIdx.x & 63;
    const int64_t row0 = (((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6) * kVeRows;
    if (row0 >= rows) return;
    const int64_t row1 = row0 + 1 < rows ? row0 + 1 : row0;
    const int s0 = sizes[row0], s1 = sizes[row1];
    const int per_row = VECTOR ? D / V : D, total = row1 > row0 ? 2 * per_row : per_row;
    using piece_t = typename std::conditional<VECTOR, typename tr::vec_t, T>::type;
    const int width = VECTOR ? V : 1;
    auto in_at = [&](int i) { return reinterpret_cast<const piece_t*>(i < per_row ? v + row0 * v_stride + (int64_t)i * width : v + row1 * v_stride + (int64_t)(i - per_row) * width); };
    auto out_at = [&](int i) { return reinterpret_cast<piece_t*>(i < per_row ? out + row0 * out_stride + (int64_t)i * width : out + row1 * out_stride + (int64_t)(i - per_row) * width); };
    piece_t p[kVePieces];
    auto fetch = [&](int base) {
#pragma unroll
        for (int u = 0; u < kVePieces; ++u) {
            const int i = base + u * 64 + lane;
            p[u] = *in_at(i < total ? i : total - 1);
        }
    };
    fetch(0);
    const double l = log((double)((lane & 1 ? s1 : s0) < 1 ? 1 : (lane & 1 ? s1 : s0)));
    const double l0 = __shfl(l, 0, kWave), l1 = __shfl(l, 1, kWave);
    for (int base = 0; base < total; base += 64 * kVePieces) {
        if (base) fetch(base);
#pragma unroll
        for (int u = 0; u < kVePieces; ++u) {
            const int i = base + u * 64 + lane;
            if (i >= total) continue;
            const double ls = i < per_row ? l0 : l1;
            if constexpr (VECTOR) {
                float f[V];
                tr::unpack(p[u], f);
                T q[V];
#pragma unroll
                for (int e = 0; e < V; ++e) tr::store(&q[e], (double)f[e] + ls);
                piece_t o;
                __builtin_memcpy(&o, q, sizeof(o));
                *out_at(i) = o;
            } else {
                T q;
                tr::store(&q, (double)tr::load(&p[u]) + ls);
                *out_at(i) = q;
            }
        }
    }
}

luvc_status value_enhance_run(const void* v, const int32_t* sizes, int64_t rows, int D, int64_t v_stride, int64_t out_stride,
                              luvc_dtype dt, void* out, hipStream_t st)
{
    const size_t es = dt == LUVC_F32 ? 4 : 2;
    const bool vec = ((size_t)D * es) % 16 == 0 && ((size_t)v_stride * es) % 16 == 0 && ((size_t)out_stride * es) % 16 == 0 &&
                     (uintptr_t)v % 16 == 0 && (uintptr_t)out % 16 == 0;
    const int64_t waves = (rows + kVeRows - 1) / kVeRows;
    const unsigned g = (unsigned)((waves * 64 + 255) / 256);
#define LUVC_VE(TT, VV) LUVC_LAUNCH("value_enhance", (value_enhance<TT, VV>), dim3(g), dim3(256), 0, st, (const TT*)v, sizes, rows, D, v_stride, out_stride, (TT*)out)
    if (dt == LUVC_F32) { if (vec) LUVC_VE(float, true); else LUVC_VE(float, false); }
    else                { if (vec) LUVC_VE(bf16_t, true); else LUVC_VE(bf16_t, false); }
#undef LUVC_VE
    return check_launch("value enhancement");
}

}  // namespace luvc
