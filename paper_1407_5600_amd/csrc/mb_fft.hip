// Fluid solve on the MAC grid by a hand-written 3-D FFT for gfx950.
//
// Kernels are compiled per grid size L (all L = 2^a 3^b, 8 <= L <= 512,
// L a multiple of 8) and per precision, so every radix, stride, twiddle step
// and index division is a compile-time constant.  Spectrum layout
// A[c][z][kx][ky] (kx < L/2 + 1, ky fastest): the x passes transpose through
// LDS, the y pass reads and writes contiguous [kx][ky] blocks, and the z
// pass reads aligned ky segments.
//
//   x forward : right-hand side r = a v + b (7-point Laplacian of v) + f
//               (Crank-Nicolson explicit half; r = f in steady mode), two
//               real rows packed as one complex line, transform along x,
//               unpack the half spectra, transposed store; float64 partial
//               sums of v and f for the mean mode.
//   y         : transform along y (forward or inverse), in place.
//   z+solve   : transform along z, projection and viscous divide per
//               wavevector, mean mode, inverse transform along z.
//   x inverse : rebuild complex lines from row pairs of half spectra
//               (Hermitian extension), inverse transform, store real rows.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "mb_box.h"
#include "mb_device.h"
#include "mb_internal.h"

namespace mb {
namespace fft {

constexpr int EPT = 8;  // elements per thread in a line transform

// LDS position of element e within a line: one spare slot after every 16
// elements, so that the radix-16 stage's stores (stride 16) and the
// following stage's loads spread over the banks.
__device__ __forceinline__ constexpr int lpad(int e) { return e + (e >> 4); }
// line stride: room for the padded line (lpad(L - 1) + 1 slots), odd
constexpr int line_stride(int L) { return (L + (L - 1) / 16) | 1; }

// Radix plan: 16s, then 8, 4, 2, then 3s.
constexpr int nstages(int n) {
    int s = 0;
    while (n % 16 == 0) { n /= 16; ++s; }
    while (n % 8 == 0) { n /= 8; ++s; }
    while (n % 4 == 0) { n /= 4; ++s; }
    while (n % 2 == 0) { n /= 2; ++s; }
    while (n % 3 == 0) { n /= 3; ++s; }
    return s;
}
constexpr int radix_at(int n, int k) {
    int s = 0;
    while (n % 16 == 0) { if (s == k) return 16; n /= 16; ++s; }
    while (n % 8 == 0) { if (s == k) return 8; n /= 8; ++s; }
    while (n % 4 == 0) { if (s == k) return 4; n /= 4; ++s; }
    while (n % 2 == 0) { if (s == k) return 2; n /= 2; ++s; }
    while (n % 3 == 0) { if (s == k) return 3; n /= 3; ++s; }
    return 1;
}
constexpr int ns_at(int n, int k) {
    int p = 1;
    for (int i = 0; i < k; ++i) p *= radix_at(n, i);
    return p;
}

// One Stockham stage of radix R on NLINES lines of length N.  Butterfly j
// of a line reads elements j + r N/R through load(line, element),
// multiplies input r by W_N^{r (j mod NS) N/(NS R)}, applies the R-point
// DFT and writes output r to element (j - j mod NS) R + (j mod NS) + r NS
// through store(line, element, value).  With MIDSYNC (loads and stores on
// the same LDS lines) a barrier separates all loads from all stores, so the
// stage runs in place.  Butterflies are spread over the threads with the
// butterfly index fastest, or the line index fastest with LFAST (lanes then
// walk across lines: contiguous when lines are adjacent in memory).
template <typename T, int N, int R, int NS, bool INV, int NLINES, int NTHR, bool LFAST,
          bool MIDSYNC, typename LD, typename ST>
__device__ __forceinline__ void stage_io(const cplx<T>* tw, int tid, const LD& load,
                                         const ST& store) {
    constexpr int NB = N / R;
    constexpr int TOTAL = NB * NLINES;
    constexpr int MAXB = (TOTAL + NTHR - 1) / NTHR;
    constexpr int TSTEP = N / (NS * R);
    cplx<T> v[MAXB][R];
#pragma unroll
    for (int it = 0; it < MAXB; ++it) {
        const int w = tid + it * NTHR;
        if (TOTAL % NTHR == 0 || w < TOTAL) {
            const int line = LFAST ? w % NLINES : w / NB;
            const int j = LFAST ? w / NLINES : w - line * NB;
            const int k = j % NS;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                cplx<T> a = load(line, j + r * NB);
                if (NS > 1 && r > 0) {
                    cplx<T> t = tw[r * k * TSTEP];
                    if (INV) t.y = -t.y;
                    a = cmul(a, t);
                }
                v[it][r] = a;
            }
        }
    }
    if (MIDSYNC) __syncthreads();
#pragma unroll
    for (int it = 0; it < MAXB; ++it) {
        const int w = tid + it * NTHR;
        if (TOTAL % NTHR == 0 || w < TOTAL) {
            const int line = LFAST ? w % NLINES : w / NB;
            const int j = LFAST ? w / NLINES : w - line * NB;
            const int k = j % NS;
            dftR<T, R, INV>(v[it]);
            const int dst = (j - k) * R + k;
#pragma unroll
            for (int r = 0; r < R; ++r) store(line, dst + r * NS, v[it][r]);
        }
    }
}

template <typename T, int N, bool INV, int NLINES, int LS, int NTHR, bool LFAST, int S>
__device__ __forceinline__ void middle_stages(cplx<T>* buf, const cplx<T>* tw, int tid) {
    if constexpr (S < nstages(N) - 1) {
        auto ld = [buf](int line, int e) { return buf[line * LS + lpad(e)]; };
        auto st = [buf](int line, int e, cplx<T> x) { buf[line * LS + lpad(e)] = x; };
        stage_io<T, N, radix_at(N, S), ns_at(N, S), INV, NLINES, NTHR, LFAST, true>(tw, tid, ld,
                                                                                     st);
        __syncthreads();
        middle_stages<T, N, INV, NLINES, LS, NTHR, LFAST, S + 1>(buf, tw, tid);
    }
}

// Transform of NLINES lines of length N: the first stage reads through
// `load`, the last writes through `store`, the stages in between work in
// place on the LDS lines buf (element e of line l at buf[l * LS + lpad(e)]).
// FIRST_LDS / LAST_LDS: load / store use buf itself (the stage then needs
// its internal barrier).  A barrier follows every stage but the last; the
// caller orders what comes before the first and after the last.
template <typename T, int N, bool INV, int NLINES, int LS, int NTHR, bool LFAST,
          bool FIRST_LDS, bool LAST_LDS, typename LD, typename ST>
__device__ __forceinline__ void line_fft_io(cplx<T>* buf, const cplx<T>* tw, int tid,
                                            const LD& load, const ST& store) {
    constexpr int S = nstages(N);
    if constexpr (S == 1) {
        stage_io<T, N, N, 1, INV, NLINES, NTHR, LFAST, FIRST_LDS && LAST_LDS>(tw, tid, load,
                                                                           store);
    } else {
        auto ld = [buf](int line, int e) { return buf[line * LS + lpad(e)]; };
        auto st = [buf](int line, int e, cplx<T> x) { buf[line * LS + lpad(e)] = x; };
        stage_io<T, N, radix_at(N, 0), 1, INV, NLINES, NTHR, LFAST, FIRST_LDS>(tw, tid, load,
                                                                            st);
        __syncthreads();
        middle_stages<T, N, INV, NLINES, LS, NTHR, LFAST, 1>(buf, tw, tid);
        stage_io<T, N, radix_at(N, S - 1), ns_at(N, S - 1), INV, NLINES, NTHR, LFAST,
                 LAST_LDS>(tw, tid, ld, store);
    }
}

// In-place transform of LDS lines, ending with a barrier.
template <typename T, int N, bool INV, int NLINES, int LS, int NTHR>
__device__ __forceinline__ void line_fft(cplx<T>* buf, const cplx<T>* tw, int tid) {
    auto ld = [buf](int line, int e) { return buf[line * LS + lpad(e)]; };
    auto st = [buf](int line, int e, cplx<T> x) { buf[line * LS + lpad(e)] = x; };
    line_fft_io<T, N, INV, NLINES, LS, NTHR, false, true, true>(buf, tw, tid, ld, st);
    __syncthreads();
}

// In-place transform of NLINES lines of length N held in LDS at
// buf[idx(line, e)] (any layout), every stage in LDS; ends with a barrier.
template <typename T, int N, bool INV, int NLINES, int NTHR, bool LFAST, int S = 0,
          typename IX>
__device__ __forceinline__ void lds_fft(cplx<T>* buf, const cplx<T>* tw, int tid,
                                        const IX& idx) {
    if constexpr (S < nstages(N)) {
        auto ld = [buf, &idx](int line, int e) { return buf[idx(line, e)]; };
        auto st = [buf, &idx](int line, int e, cplx<T> x) { buf[idx(line, e)] = x; };
        stage_io<T, N, radix_at(N, S), ns_at(N, S), INV, NLINES, NTHR, LFAST, true>(tw, tid,
                                                                                   ld, st);
        __syncthreads();
        lds_fft<T, N, INV, NLINES, NTHR, LFAST, S + 1>(buf, tw, tid, idx);
    }
}

// ---------------------------------------------------------------------------
// Launch geometry per size.
constexpr int largest_even_divisor(int L, int cap) {
    int best = 2;
    for (int d = 2; d <= L && d <= cap; d += 2)
        if (L % d == 0) best = d;
    return best;
}
// rows per block of the inverse x pass (about 256 threads per block)
constexpr int rows_x(int L) { return largest_even_divisor(L, 4096 / L > 2 ? 4096 / L : 2); }
// Rows per block of the forward x pass and elements per thread (by the size, and
// by whether the force is a field and whether it is all that is transformed).  A
// block is a chain (a load round per element of a thread, the transform, the
// store), so short chains and many blocks matter most: up to L = 128, 16 rows and
// one element per thread (L <= 24), two (<= 72) or four against eight elements of
// 4096 / L rows (one 32^3 box, 48 blocks of 256 threads against 96 of 64: 10.0 ->
// 5.4 us; 64^3 float32 12.2 -> 8.0, float64 14.7 -> 12.7; 72^3 14.6 -> 9.1; 96^3
// float64 25.0 -> 21.9; 128^3 float32 21.7 -> 20.5, float64 38.2 -> 34.6).  Fewer
// rows store shorter runs of ky (a batch of 32 64^3 boxes: 69.7 us with 16 rows,
// 76 with 8).
// Above, what the loads find in the caches decides, and every size was measured
// both ways.  float32, as few elements as 512 threads allow against eight, in us:
// with boxes 192^3 85 and 88, 216^3 206 and 228, 256^3 198 and 202, 288^3 366 and
// 381, 384^3 722 and 775, 512^3 1695 and 1788, but 432^3 1195 and 1129; a field
// with a velocity 55 and 58, 107 and 116, 133 and 131, 279 and 290, 490 and 530, 1168
// and 1262, 432^3 922 and 810; a field alone 36 and 33 at 192^3, 60 and 53, 71
// and 62, 173 and 133, 307 and 253, 580 and 438, 632 and 640; boxes alone as with
// a velocity, but 288^3 290 and 250.  float64, four elements of eight rows against
// eight of 4096 / L: 192^3 with boxes 173 and 177, a field 132 and 133, 216^3 336
// and 355, 251 and 246, 256^3 404 and 413, 314 and 318; 288^3 872 and 699, 710 and
// 548, 384^3 1614 and 1455, 1299 and 1176, 432^3 a field 1922 and 1875, 512^3 2705
// and 2849; 144^3 80 and 75 (24 rows).
template <typename T>
constexpr int rows_xf(int L) {
    if (L <= 128 || (sizeof(T) == 4 && L == 144)) return largest_even_divisor(L, 16);
    if (sizeof(T) == 8 && L >= 192 && L <= 256) return 8;
    return rows_x(L);
}
template <typename T>
constexpr int elems_xf(int L, bool field, bool steady) {
    const int n = rows_xf<T>(L) / 2 * L;
    if (L <= 128) return L <= 24 ? 1 : (L <= 72 ? 2 : 4);
    if (sizeof(T) == 8) return L >= 192 && L <= 256 ? 4 : EPT;
    if (L == 432 || (steady && (field ? L >= 192 : L == 288))) return EPT;
    int e = 3;
    while (n % e != 0 || n / e > 512) ++e;
    return e;
}

// kx columns per block of the y pass (at least 128 B contiguous per row), dealt
// evenly up to 96^3, so that the last block is not left with a column or two (64^3:
// 33 = 17 + 16, not 32 + 1: 32 boxes 57 us against 84 in float64, 27 and 41 in
// float32).  Above, the uneven share changes nothing (128^3 float32 8.3 and 8.5,
// 144^3 12.5 and 12.1, 256^3 52.4 and 53.0, float64 15.2 and 15.4, 110.6 and 110.3).
template <typename T>
constexpr int cols_y(int L) {
    const int nc = L / 2 + 1;
    int w = 2048 / L;
    if (w < 1) w = 1;
    if (w >= nc) return nc;
    if (L > 96) return w;
    const int blocks = (nc + w - 1) / w;
    return (nc + blocks - 1) / blocks;
}
// Elements per thread of the z pass: four, a shorter chain, where a single box is a
// round or two of blocks and has waves to spare, else eight.  Four against eight, us,
// one box: float64 24^3 5.0 and 5.9, 32^3 5.0 and 5.5, 64^3 8.1 and 8.4, 72^3 13.8
// and 14.8 (not taken), 96^3 21.1 and 17.6, 128^3 28.0 and 22.4, 192^3 127 and 99,
// 256^3 430 and 321; float32 72^3 9.2 and 9.7, 96^3 12.2 and 13.3, 128^3 17.1 and
// 14.1, 144^3 38.8 and 28.0, 256^3 150 and 100.  (32 boxes of 48^3 in float64 take
// 44 and 35, of 64^3 74 and 72, in float32 41 and 33: the float64 ones would have
// eight, which one box would pay for.)
template <typename T>
constexpr int elems_z(int L) {
    return sizeof(T) == 8 ? (L <= 64 ? 4 : EPT) : (L == 72 || L == 96 ? 4 : EPT);
}
// ky columns per block of the z pass (a divisor of L; LDS <= 64 KB for
// float32, 100 KB for float64).  Eight float32 columns are half a 128-byte line, four
// float64 ones too: fewer split more lines, more leave fewer and larger blocks.  Four
// against eight, us: float32 64^3 (32 boxes) 38 and 33, 72^3 12.3 and 9.2, 96^3 12.3
// and 16.2 (1,176 blocks of 288 threads against 588 of 576), 128^3
// 15.5 and 14.1, 144^3 34 and 28, 216^3 106 and 83, 256^3 149 and 100, 288^3 267 and 316
// (not taken); float64 48^3 6.9 and 6.1, 64^3 7.7 and 8.3, 72^3 14.8 and 11.8 (not
// taken), 96^3 18.2 and 19.7, 128^3 22.2 and 26.5, 144^3 42 and 39, 256^3 450 and 320.
// At 128^3 float32 sixteen (520 blocks of 768 threads: two per CU, and a nearly empty
// second round) were slower, and so were sixteen of sixteen elements (18.6 against 15.1).
template <typename T>
constexpr int cols_z(int L) {
    int w = sizeof(T) == 8 ? (L <= 128 && L != 48 ? 4 : 8) : (L == 96 ? 4 : 8);
    const int cap = sizeof(T) == 8 ? 102400 : 65536;
    while (w > 1 && (L % w != 0 || 3 * L * w * 2 * (int)sizeof(T) > cap ||
                     3 * w * L / elems_z<T>(L) > 1024))
        w /= 2;
    return w;
}

template <typename T, int L>
struct Geo {
    static constexpr int NC = L / 2 + 1;
    static constexpr int R = rows_xf<T>(L);  // forward x pass: rows per block
    static constexpr int NL = R / 2;
    static constexpr int RI = rows_x(L);     // inverse x pass
    static constexpr int NLI = RI / 2;
    static constexpr int TXI = NLI * L / EPT;
    static constexpr int LS = line_stride(L); // LDS line stride (complex)
    static constexpr int WY = cols_y<T>(L);
    static constexpr int NCHY = (NC + WY - 1) / WY;
    static constexpr int TY = (WY * L + EPT - 1) / EPT;
    static constexpr int WZ = cols_z<T>(L);
    static constexpr int TZ = 3 * WZ * L / elems_z<T>(L);
    static constexpr int NBX = 3 * L * (L / R);  // blocks of an x pass
    static_assert(NBX % 8 == 0, "x-pass blocks are remapped over the 8 XCDs");
    // inverse plane pass (y and x together, one (component, z) plane per
    // block): the plane as H = L/2 complex columns, row stride PS (room for
    // the padded column H of the staged half spectrum, odd)
    static constexpr int H = L / 2;
    static constexpr int PS = (lpad(H) + 1) | 1;
    static constexpr int PLANE_BYTES = L * PS * 2 * (int)sizeof(T);
    // used when two planes fit in a CU's 160 KB of LDS (float32 L <= 128,
    // float64 L <= 72), or one plane with L <= 144 (float32 L = 144, float64
    // L = 96, 128: faster than the two passes it replaces; float32 L = 192,
    // one block per CU in 1.1 rounds, was slower)
    static constexpr int XY_LDS = PLANE_BYTES + (L + H) * 2 * (int)sizeof(T);
    static constexpr bool XY =
        PLANE_BYTES <= 72 * 1024 || (XY_LDS <= 160 * 1024 && L <= 144);
    // threads: 4 elements each, at most 1,024 (more waves hide more of the
    // latency; at 128^3 float32 18.0 against 18.9 us with 512, float64 32.9
    // against 34.5; one 32^3 box 5.8 -> 5.2 us against 8 elements, 96^3
    // float64 22.4 -> 20.8)
    static constexpr int TXY_RAW = ((L * H / 4 + WAVE - 1) / WAVE) * WAVE;
    static constexpr int TXY = TXY_RAW > 1024 ? 1024 : TXY_RAW;
    static constexpr int NBXY = 3 * L;                         // blocks per box
};

// ---------------------------------------------------------------------------
// Force of the forward x pass: the field f; the boxes (f the box array); the
// boxes plus a field; or the records of a small box.
enum : int { SRC_FIELD, SRC_BOX, SRC_BOX_ADD, SRC_REC };

// What the last two read.  add: the field added (SRC_REC: nullable).  rec,
// recf: geometry and force records of the mbox blobs of each box, from which a
// block forms the force of its rows: the spreading writes and this pass reads
// 1.67 values per node and a few blobs touch few of them (one particle in
// 32^3: spreading 6.3 us; 32 boxes of 64^3 with two particles each: spreading
// 20 us and 168 MB of mostly zero boxes).  act (SRC_REC in steady flow, where
// the force is all there is): whether each z plane of each box holds any
// force, as the binning marked it; the x and y passes pass over planes without
// one and the z pass takes them as zero (two particles in 64^3 lie in about 7
// of the 64 planes).  fexp: per box, the exponent of the fixed-point sums its
// force is formed in (add_records), as the binning left it.
template <typename T>
struct ForceSrc {
    const T* add;
    const RecG<T>* rec;
    const T* recf;
    int mbox;
    const unsigned char* act;
    int ng;  // with act: blocks that share a box's planes (active_planes)
    const int* fexp;
};

// A record as the rows of one plane see it: its first nodes along x and y
// (wrapped), the x weights, and the y weights times the z weight of the plane
// times the force, scaled by 2^e.
template <typename T>
struct RecLine {
    T wx[3], wyf[3];
    int xs, ys;
};

// The records of a box (forces recf) with nodes of component a in plane z and
// in any of the R rows from y0 into list, the forces times 2^e2; returns their
// number.  Each thread looks at one record a round (a round takes NTHR); cnt: an
// int per wave.  Called by the whole block; ends with a barrier.
template <typename T, int L, int R, int NTHR>
__device__ __forceinline__ int plane_records(const RecG<T>* __restrict__ rec,
                                             const T* __restrict__ recf, int mbox, int a, int z,
                                             int y0, int e2, RecLine<T>* list, int* cnt) {
    constexpr int NW = (NTHR + WAVE - 1) / WAVE;
    const int tid = threadIdx.x, wave = tid / WAVE;
    int n = 0;
    for (int b0 = 0; b0 < mbox; b0 += NTHR) {
        const int i = b0 + tid;
        const int ic = i < mbox ? i : 0;
        const RecG<T> r = rec[ic];
        const T F = recf[3 * ic + a];
        auto first = [&](int b) {  // first node along axis b, in [0, L)
            const int c = (int)((r.cell >> (9 * b)) & 511u) - 1;
            const int i0 = a == b ? c : c + (int)((r.cell >> (27 + b)) & 1u);
            return i0 < 0 ? i0 + L : (i0 >= L ? i0 - L : i0);
        };
        const int xs = first(0), ys = first(1);
        int dz = z - first(2);
        dz += dz < 0 ? L : 0;
        int dy = ys - y0;  // first row from y0, in [0, L); L - 2, L - 1: the rows before
        dy += dy < 0 ? L : 0;
        const bool keep = i < mbox && dz < 3 && (dy < R || dy >= L - 2);
        const unsigned long long m = __ballot(keep);
        if (NW > 1) {
            if (tid % WAVE == 0) cnt[wave] = __popcll(m);
            __syncthreads();
        }
        int before = n, total = n;
        if (NW > 1) {
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                before += w < wave ? cnt[w] : 0;
                total += cnt[w];
            }
        } else {
            total += __popcll(m);
        }
        if (keep) {
            RecLine<T>* e = list + before + __popcll(m & ((1ull << (tid % WAVE)) - 1));
#pragma unroll
            for (int b = 0; b < 3; ++b) e->wx[b] = rec_t(r, a, b);
            e->wyf[0] = F;
            e->xs = xs | dz << 16;
            e->ys = ys;
        }
        n = total;
        __syncthreads();
    }
    if (n > 0) {
        // the weights, by as few waves as the list takes
        for (int k = tid; k < n; k += NTHR) {
            RecLine<T>* e = list + k;
            const int dz = e->xs >> 16;
            T wx[3], wy[3];
            const T f = kernel_weight<T>(e->wx[2], dz) * e->wyf[0];
            kernel_weights<T>(e->wx[0], wx);
            kernel_weights<T>(e->wx[1], wy);
#pragma unroll
            for (int b = 0; b < 3; ++b) {
                e->wx[b] = wx[b];
                e->wyf[b] = ldexp(wy[b] * f, e2);
            }
            e->xs &= 0xffff;
        }
        __syncthreads();
    }
    return n;
}

// Where the x pass of a small box sums the force of node (x, y0 + y) of its rows:
// in float64 in the slot of the transform's buffer that takes the node's row pair
// (two sums are as large as two values, and the thread that reads them writes the
// slot), in float32 in an array of their own.
template <typename T, int L>
__device__ __forceinline__ int sum_slot(int y, int x) {
    constexpr int LS = line_stride(L);
    return sizeof(T) == 8 ? 2 * ((y >> 1) * LS + lpad(x)) + (y & 1) : y * L + x;
}

// The n records of a list, added to the sums acc (nacc of them, cleared here) of the
// R rows from y0 of the plane: a thread takes one of a record's nine nodes in the
// plane.  The sums are 64-bit integers, as in the spreading, so that they do not
// depend on the order; |w F| 2^e2 < 2^55 (box_exponent) for each of at most
// kSmallBlobs, so that none overflows and the quantum is below 2^-55 of the box's
// largest force.  (Sums in registers, in a loop of every wave over the records of
// its rows, took 17 us of the x pass for 247 blobs in one 16^3 box, which takes 7 so;
// 512 such boxes in steady flow 186 and 78.)  Called by the whole block, n > 0; ends
// with a barrier.
template <typename T, int L, int R, int NTHR>
__device__ __forceinline__ void add_records(const RecLine<T>* list, int n, int y0,
                                            unsigned long long* acc, int nacc) {
    for (int i = threadIdx.x; i < nacc / 2; i += NTHR)
        reinterpret_cast<ulonglong2*>(acc)[i] = ulonglong2{0ull, 0ull};
    __syncthreads();
    for (int i = threadIdx.x; i < 9 * n; i += NTHR) {
        const int k = i / 9, j = i - 9 * k;
        const int ky = j / 3, kx = j - 3 * ky;
        const RecLine<T>* e = list + k;
        int y = e->ys + ky - y0, x = e->xs + kx;  // ys - y0 in (-L, L)
        y += y < 0 ? L : 0;
        y -= y >= L ? L : 0;
        x -= x >= L ? L : 0;
        if (y < R) {
            const double c = (double)e->wx[kx] * (double)e->wyf[ky];
            atomicAdd(acc + sum_slot<T, L>(y, x), (unsigned long long)(long long)rint(c));
        }
    }
    __syncthreads();
}

// The force of a node from its sum (e2: kExpNonfinite where a force of the box is
// not finite).
template <typename T>
__device__ __forceinline__ T sum_value(unsigned long long s, int e2) {
    if (e2 == kExpNonfinite) return (T)__builtin_nan("");
    return (T)ldexp((double)(long long)s, -e2);
}

// Planes with marks act of block zi of the ng that share a box's planes (and
// one component, rows or columns): bit k of plane zi + 8 k.  ng = L (plane_blocks):
// its plane alone.  Else ng = 8: the planes eight apart, read at once (those of
// a few particles, neighbours, fall to different blocks, and few blocks find
// nothing to do).
template <int L>
__device__ __forceinline__ unsigned long long active_planes(const unsigned char* __restrict__ act,
                                                            int zi, int ng) {
    if (ng == L) return act[zi] ? 1ull : 0ull;
    unsigned long long m = 0;
#pragma unroll
    for (int k = 0; k < L / 8; ++k) m |= act[zi + 8 * k] ? 1ull << k : 0ull;
    return m;
}

// Threads of the forward x pass.
template <typename T, int L, int SRC, bool STEADY>
constexpr int threads_xf() {
    constexpr int n = Geo<T, L>::NL * L, e = elems_xf<T>(L, SRC == SRC_FIELD, STEADY);
    static_assert(n % e == 0 && n / e <= 512, "x pass");
    return n / e;
}

template <typename T, int L, int SRC, bool STEADY>
__global__ void __launch_bounds__((threads_xf<T, L, SRC, STEADY>()))
k_x_fwd(const T* __restrict__ v, const T* __restrict__ f, Tiles tl, ForceSrc<T> mk,
        const cplx<T>* __restrict__ tw, T a, T b,
        cplx<T>* __restrict__ A, double* __restrict__ psum) {
    constexpr bool BOX = SRC == SRC_BOX || SRC == SRC_BOX_ADD;
    constexpr bool REC = SRC == SRC_REC;
    constexpr bool ADD = SRC == SRC_BOX_ADD;
    using G = Geo<T, L>;
    constexpr int NC = G::NC, R = G::R, NL = G::NL, LS = G::LS;
    constexpr int NTHR = threads_xf<T, L, SRC, STEADY>(), EX = NL * L / NTHR;
    // SRC_REC: the records of a block's rows and the sums of their forces.  The sums
    // share the buffer in float64, the records (done with before it) in float32.
    constexpr bool F64 = sizeof(T) == 8;
    constexpr int LIST = (int)(kSmallBlobs * sizeof(RecLine<T>) / sizeof(cplx<T>));
    __shared__ __align__(16) cplx<T> buf[REC && !F64 && LIST > NL * LS ? LIST : NL * LS];
    __shared__ cplx<T> tws[L];
    __shared__ RecLine<T> list64[REC && F64 ? kSmallBlobs : 1];
    __shared__ __align__(16) unsigned long long acc32[REC && !F64 ? R * L : 2];
    unsigned long long* acc = F64 ? reinterpret_cast<unsigned long long*>(buf) : acc32;
    constexpr int NACC = F64 ? 2 * NL * LS : R * L;
    __shared__ double red[16];
    const int tid0 = threadIdx.x;
    // blocks of a box are consecutive (G::NBX per box, a multiple of 8);
    // within a box each XCD takes a contiguous range of (c, z, y) rows, so
    // the rows of the Laplacian's z and y neighbours, read by adjacent
    // blocks, are found in that XCD's L2
    // with act a block takes the planes of active_planes
    constexpr bool ACT = REC && STEADY;
    const bool planes = ACT && mk.act;
    const int per_box = planes ? G::NBX / L * mk.ng : G::NBX;
    const int box = blockIdx.x / per_box;
    const int lb = planes ? blockIdx.x - box * per_box : xcd_remap(blockIdx.x - box * per_box, G::NBX);
    const int yb = lb % (L / R);
    const int nz = planes ? mk.ng : L;
    const int comp = lb / (L / R) / nz;
    const int z_first = lb / (L / R) % nz;
    const int cbase = comp * L * L * L;   // component offset (elements)
    const int y0 = yb * R;
    v += (size_t)box * 3 * L * L * L;
    A += (size_t)box * 3 * L * NC * L;
    if (SRC == SRC_FIELD) f += (size_t)box * 3 * L * L * L;
    unsigned long long todo = 1;
    if (planes) {
        todo = active_planes<L>(mk.act + (size_t)box * L, z_first, mk.ng);
        if (todo == 0) return;
    }
    for (int i = tid0; i < L; i += NTHR) tws[i] = tw[i];
    do {  // (a loop only with ACT: as one of a single round, it took 10 to 20 registers more)
    // (opaque in the loop over planes: the indices formed from it are not kept
    // across it, which took up to 264 registers)
    int tid = tid0;
    if (ACT) asm volatile("" : "+v"(tid));
    const int z = z_first + (ACT ? 8 * (__ffsll(todo) - 1) : 0);
    const int cz = comp * L + z;
    double sv = 0.0, sf = 0.0;
    const int zm = (z == 0 ? L - 1 : z - 1), zp = (z == L - 1 ? 0 : z + 1);
    // boxed force: the box entries of this z plane and component
    const T* Ec = nullptr;
    AxisSrc bz{};
    if (BOX) {
        Ec = f + ((size_t)box * 3 + comp) * tl.n * box_volume(tl);
        bz = box_src_z(tl, z);
    }
    [[maybe_unused]] const T* add =
        (ADD || REC) && mk.add ? mk.add + (size_t)box * 3 * L * L * L : nullptr;
    [[maybe_unused]] int nlist = 0, e2 = 0;
    if constexpr (REC) {
        e2 = mk.fexp[box];
        const size_t b0 = (size_t)box * mk.mbox;
        RecLine<T>* list = F64 ? list64 : reinterpret_cast<RecLine<T>*>(buf);
        nlist = plane_records<T, L, R, NTHR>(mk.rec + b0, mk.recf + 3 * b0, mk.mbox, comp, z, y0,
                                             e2, list, reinterpret_cast<int*>(red));
        if (nlist > 0) add_records<T, L, R, NTHR>(list, nlist, y0, acc, NACC);
    }
    // KG iterations (2 KG nodes) per round: all loads of a round, the box
    // entries included (box_entries: loads only, in uniform branches), are
    // issued before its arithmetic.  Two where a float32 wave keeps to one row
    // pair and has them (128^3: 21.4 against 20.7 us, 256^3: 209 against 202);
    // one elsewhere (float64 128^3: 34.5 against 37.5 with two, whose registers
    // cost a wave; 96^3: 14.0 against 15.5).
    // UNI: a wave's lanes share y.
    constexpr bool UNI = L % WAVE == 0 && NTHR % L == 0;
    constexpr int KG = sizeof(T) == 4 && UNI && BOX && !STEADY && EX % 2 == 0 ? 2 : 1;
    static_assert(EX % KG == 0, "rounds of the x pass");
    // with UNI, a thread's x (and its neighbours and x box sources) is the
    // same in every round and its line differs by a constant per round, the
    // wave's rows are uniform: each load is a uniform row base plus the
    // thread's fixed x offset
    [[maybe_unused]] const int xu = tid % L;
    [[maybe_unused]] const int line0 = UNI ? __builtin_amdgcn_readfirstlane(tid / L) : 0;
    [[maybe_unused]] const unsigned ox = (unsigned)xu * (unsigned)sizeof(T);
    [[maybe_unused]] const unsigned oxm = (unsigned)(xu == 0 ? L - 1 : xu - 1) * (unsigned)sizeof(T);
    [[maybe_unused]] const unsigned oxp = (unsigned)(xu == L - 1 ? 0 : xu + 1) * (unsigned)sizeof(T);
    [[maybe_unused]] AxisSrc bxu{};
    if constexpr (UNI && BOX) bxu = box_src_x(tl, xu);
#pragma unroll
    for (int k0 = 0; k0 < EX; k0 += KG) {
        T vc[KG][2], vn[KG][2][6], fv[KG][2];
        T eb[KG][2][4][2];
        if constexpr (UNI) {
            const char* vb = reinterpret_cast<const char*>(v);
            const char* fb = reinterpret_cast<const char*>(f);
            auto at = [](const char* base, int row, unsigned o) {
                return *reinterpret_cast<const T*>(base + (size_t)row * sizeof(T) + o);
            };
#pragma unroll
            for (int g = 0; g < KG; ++g) {
            const int line = line0 + (k0 + g) * (NTHR / L);
#pragma unroll
            for (int hh = 0; hh < 2; ++hh) {
                const int y = y0 + 2 * line + hh;
                const int row = cbase + (z * L + y) * L;
                if (SRC == SRC_FIELD) fv[g][hh] = at(fb, row, ox);
                if constexpr (ADD) fv[g][hh] = at(reinterpret_cast<const char*>(add), row, ox);
                if constexpr (REC)
                    fv[g][hh] = add ? at(reinterpret_cast<const char*>(add), row, ox) : T(0);
                if (!STEADY) {
                    const int ym = y == 0 ? L - 1 : y - 1, yp = y == L - 1 ? 0 : y + 1;
                    vc[g][hh] = at(vb, row, ox);
                    vn[g][hh][0] = at(vb, row, oxm);
                    vn[g][hh][1] = at(vb, row, oxp);
                    vn[g][hh][2] = at(vb, cbase + (z * L + ym) * L, ox);
                    vn[g][hh][3] = at(vb, cbase + (z * L + yp) * L, ox);
                    vn[g][hh][4] = at(vb, cbase + (zm * L + y) * L, ox);
                    vn[g][hh][5] = at(vb, cbase + (zp * L + y) * L, ox);
                }
            }
            if constexpr (BOX) {
#pragma unroll
                for (int hh = 0; hh < 2; ++hh) {
                    const AxisSrc by = box_src_y(tl, y0 + 2 * line + hh);
                    box_entries(Ec, bxu, by, bz, eb[g][hh]);
                }
            }
            }
        } else {
#pragma unroll
        for (int g = 0; g < KG; ++g) {
            const int e = tid + (k0 + g) * NTHR;
            const int line = e / L;
            const int x = e - line * L;
            const int xm = x == 0 ? L - 1 : x - 1, xp = x == L - 1 ? 0 : x + 1;
#pragma unroll
            for (int hh = 0; hh < 2; ++hh) {
                const int y = y0 + 2 * line + hh;
                const unsigned row = (unsigned)(cbase + (z * L + y) * L);
                if (SRC == SRC_FIELD) fv[g][hh] = ld32(f, row + x);
                if constexpr (ADD) fv[g][hh] = ld32(add, row + x);
                if constexpr (REC) fv[g][hh] = add ? ld32(add, row + x) : T(0);
                if (!STEADY) {
                    const int ym = y == 0 ? L - 1 : y - 1, yp = y == L - 1 ? 0 : y + 1;
                    vc[g][hh] = ld32(v, row + x);
                    vn[g][hh][0] = ld32(v, row + xm);
                    vn[g][hh][1] = ld32(v, row + xp);
                    vn[g][hh][2] = ld32(v, (unsigned)(cbase + (z * L + ym) * L + x));
                    vn[g][hh][3] = ld32(v, (unsigned)(cbase + (z * L + yp) * L + x));
                    vn[g][hh][4] = ld32(v, (unsigned)(cbase + (zm * L + y) * L + x));
                    vn[g][hh][5] = ld32(v, (unsigned)(cbase + (zp * L + y) * L + x));
                }
            }
            if constexpr (BOX) {
                const AxisSrc bx = box_src_x(tl, x);
#pragma unroll
                for (int hh = 0; hh < 2; ++hh) {
                    const int y = y0 + 2 * line + hh;
                    box_entries(Ec, bx, box_src_y(tl, y), bz, eb[g][hh]);
                }
            }
        }
        }
#pragma unroll
        for (int g = 0; g < KG; ++g) {
            const int e = tid + (k0 + g) * NTHR;
            const int line = e / L;
            const int x = e - line * L;
            T val[2];
#pragma unroll
            for (int hh = 0; hh < 2; ++hh) {
                if (REC && (nlist > 0 || e2 == kExpNonfinite))
                    fv[g][hh] = sum_value<T>(acc[sum_slot<T, L>(2 * line + hh, x)], e2) + fv[g][hh];
                if (ADD) fv[g][hh] = box_entries_sum(eb[g][hh]) + fv[g][hh];
                else if (BOX) fv[g][hh] = box_entries_sum(eb[g][hh]);
                sf += (double)fv[g][hh];
                if (STEADY) {
                    val[hh] = fv[g][hh];
                } else {
                    sv += (double)vc[g][hh];
                    const T lap = (vn[g][hh][0] + vn[g][hh][1]) + (vn[g][hh][2] + vn[g][hh][3]) +
                                  (vn[g][hh][4] + vn[g][hh][5]) - T(6) * vc[g][hh];
                    val[hh] = a * vc[g][hh] + b * lap + fv[g][hh];
                }
            }
            buf[line * LS + lpad(x)] = cplx<T>{val[0], val[1]};
        }
    }
    __syncthreads();
    line_fft<T, L, false, NL, LS, NTHR>(buf, tws, tid);
    // unpack the two half spectra of each line; store A[c][z][kx][y]
    cplx<T>* out = A + (size_t)cz * NC * L + y0;
    for (int e = tid; e < NC * R; e += NTHR) {
        const int kx = e / R;
        const int rl = e - kx * R;
        const int line = rl >> 1;
        const cplx<T> Z = buf[line * LS + lpad(kx)];
        const cplx<T> Zc = cconj(buf[line * LS + lpad(kx == 0 ? 0 : L - kx)]);
        cplx<T> o;
        if (rl & 1) {  // (Z - Zc) / 2i
            o = cplx<T>{T(0.5) * (Z.y - Zc.y), T(-0.5) * (Z.x - Zc.x)};
        } else {       // (Z + Zc) / 2
            o = cplx<T>{T(0.5) * (Z.x + Zc.x), T(0.5) * (Z.y + Zc.y)};
        }
        st32(out, (unsigned)(kx * L + rl), o);
    }
    // the block's sums of v and f (one barrier; red holds 16 doubles, at
    // most 8 waves of two partials each)
    static_assert(2 * ((NTHR + WAVE - 1) / WAVE) <= 16, "reduction scratch");
    const double wsv = wave_sum(sv), wsf = wave_sum(sf);
    if (tid % WAVE == 0) {
        red[2 * (tid / WAVE)] = wsv;
        red[2 * (tid / WAVE) + 1] = wsf;
    }
    __syncthreads();
    if (tid == 0) {
        double ts = 0.0, tf = 0.0;
        for (int w = 0; w < (NTHR + WAVE - 1) / WAVE; ++w) {
            ts += red[2 * w];
            tf += red[2 * w + 1];
        }
        if (!planes) {
            const size_t pb = (size_t)box * G::NBX + lb;  // component-major order
            psum[2 * pb] = ts;
            psum[2 * pb + 1] = tf;
        }
    }
    } while (ACT && (todo &= todo - 1) != 0);
}

// y pass: block = (component, z plane, WY consecutive kx); the kx rows of
// length L (along ky) are contiguous in A.
template <typename T, int L, bool INV, bool ACT>
__global__ void __launch_bounds__((Geo<T, L>::TY))
k_y(cplx<T>* __restrict__ A, const cplx<T>* __restrict__ tw,
    const unsigned char* __restrict__ act, int ng) {
    using G = Geo<T, L>;
    constexpr int NC = G::NC, W = G::WY, NTHR = G::TY, LS = G::LS;
    __shared__ cplx<T> buf[W * LS];
    __shared__ cplx<T> tws[L];
    const int tid0 = threadIdx.x;
    const int ch = blockIdx.x % G::NCHY;
    // ACT: planes without a mark in act are neither read nor written; a block
    // then takes the planes of active_planes
    const int bcz = blockIdx.x / G::NCHY;  // (box * 3 + c) * L + z, or ... * ng + zi
    unsigned long long todo = 1;
    if constexpr (ACT) todo = active_planes<L>(act + (size_t)(bcz / ng / 3) * L, bcz % ng, ng);
    if (ACT && todo == 0) return;
    for (int i = tid0; i < L; i += NTHR) tws[i] = tw[i];
    do {
    int tid = tid0;
    if (ACT) asm volatile("" : "+v"(tid));  // (as in k_x_fwd)
    const int cz = ACT ? bcz / ng * L + bcz % ng + 8 * (__ffsll(todo) - 1) : bcz;
    const int kx0 = ch * W;
    const int wc = NC - kx0 < W ? NC - kx0 : W;
    cplx<T>* base = A + ((size_t)cz * NC + kx0) * L;
    // first stage straight from A, last stage straight back (a short last
    // chunk re-reads its first row and stores only its own rows)
    auto gload = [base, wc](int line, int e) {
        return ld32(base, (unsigned)((line < wc ? line : 0) * L + e));
    };
    auto gstore = [base, wc](int line, int e, cplx<T> x) {
        if (line < wc) st32(base, (unsigned)(line * L + e), x);
    };
    __syncthreads();  // twiddles; the plane before has left buf
    line_fft_io<T, L, INV, W, LS, NTHR, false, false, false>(buf, tws, tid, gload, gstore);
    } while (ACT && (todo &= todo - 1) != 0);
}

// z pass fused with the solve: block = (kx, WZ consecutive ky), all three
// components.  Per wavevector m != 0, with D the divergence symbol
// (D_b = (1 - e^{-2 pi i m_b / L}) / h, |D|^2 = sum_b 4 sin^2(pi m_b/L)/h^2):
//   v^ = (r^ - conj(D) (D . r^) / |D|^2) / ((c0 + c1 |D|^2))
// which is the solenoidal projection of eq. vf on the MAC grid followed by
// the Crank-Nicolson (c0 = N rho/dt, c1 = N eta/2) or steady (c0 = 0,
// c1 = N eta) divide, N = L^3 folding in the inverse normalisation.  The
// mean mode is set from float64 sums: mean(v) + (dt/rho) mean(f), or zero.
// ACT: planes with act[z] = 0 hold no force and are taken as zero, unread;
// with part_out they are not written either.
template <typename T, int L, bool ACT>
__global__ void __launch_bounds__((Geo<T, L>::TZ))
k_z_solve(cplx<T>* __restrict__ A, const cplx<T>* __restrict__ tw,
          const cplx<T>* __restrict__ dsym, const T* __restrict__ d2, T c0, T c1,
          int zero_mean_mode, const double* __restrict__ psum, int per_c, double mv,
          double mf, const unsigned char* __restrict__ act, int part_out) {
    using G = Geo<T, L>;
    constexpr int NC = G::NC, W = G::WZ, NTHR = G::TZ, LS = G::LS;
    constexpr int NLN = 3 * W;
    __shared__ cplx<T> buf[NLN * LS];
    __shared__ cplx<T> tws[L];
    __shared__ double red[3 * ((NTHR + WAVE - 1) / WAVE)];
    __shared__ double mean_new[3];
    const int tid = threadIdx.x;
    // blocks of a box are consecutive (NC L / W per box); when their count
    // is a multiple of 8 each XCD takes a contiguous range, so the blocks
    // sharing the cache lines of a ky segment meet in one L2
    constexpr int NZB = NC * (L / W);
    const int box = blockIdx.x / NZB;
    const int lblk = NZB % 8 == 0 ? xcd_remap(blockIdx.x - box * NZB, NZB)
                                  : blockIdx.x - box * NZB;
    const int ch = lblk % (L / W);
    const int kx = lblk / (L / W);
    const int ky0 = ch * W;
    A += (size_t)box * 3 * L * NC * L;
    psum += (size_t)box * 3 * per_c * 2;  // per_c partials per component
    for (int i = tid; i < L; i += NTHR) tws[i] = tw[i];
    __shared__ unsigned char on[ACT ? L : 1];
    if constexpr (ACT)
        for (int i = tid; i < L; i += NTHR) on[i] = act[(size_t)box * L + i];
    if (kx == 0 && ch == 0) {
        // the three components' sums together: every load of a round before
        // its adds, one reduction (each wave's sums through LDS)
        double s[3] = {0.0, 0.0, 0.0};
        if (!zero_mean_mode) {
#pragma unroll 2
            for (int i = tid; i < per_c; i += NTHR) {
                const double* p = psum + 2 * i;
#pragma unroll
                for (int c = 0; c < 3; ++c)
                    s[c] += mv * p[2 * c * per_c] + mf * p[2 * c * per_c + 1];
            }
        }
        constexpr int NW = (NTHR + WAVE - 1) / WAVE;
#pragma unroll
        for (int c = 0; c < 3; ++c) s[c] = wave_sum(s[c]);
        if (tid % WAVE == 0) {
#pragma unroll
            for (int c = 0; c < 3; ++c) red[3 * (tid / WAVE) + c] = s[c];
        }
        __syncthreads();  // (uniform over the block)
        if (tid < 3) {
            double t = 0.0;
            for (int w = 0; w < NW; ++w) t += red[3 * w + tid];
            mean_new[tid] = t;
        }
    }
    __syncthreads();  // twiddles, mean mode
    // line (c, w), w fastest: lanes read contiguous ky segments of A; the
    // forward transform reads A and leaves the spectrum in LDS, the inverse
    // reads LDS and writes A
    // unsigned 32-bit offsets from the block's column base (the spectrum of
    // one box is below 4 GiB)
    cplx<T>* Ak = A + (size_t)kx * L + ky0;
    const unsigned char* onz = on;
    auto gload = [Ak, onz](int line, int z) {
        const int c = line / W, w = line - (line / W) * W;
        if (ACT && !onz[z]) return cplx<T>{T(0), T(0)};
        return ld32(Ak, (unsigned)((c * L + z) * NC * L + w));
    };
    auto gstore = [Ak, onz, part_out](int line, int z, cplx<T> x) {
        const int c = line / W, w = line - (line / W) * W;
        if (ACT && part_out && !onz[z]) return;
        st32(Ak, (unsigned)((c * L + z) * NC * L + w), x);
    };
    cplx<T>* lb = buf;
    auto lload = [lb](int line, int e) { return lb[line * LS + lpad(e)]; };
    auto lstore = [lb](int line, int e, cplx<T> x) { lb[line * LS + lpad(e)] = x; };
    line_fft_io<T, L, false, NLN, LS, NTHR, true, false, true>(buf, tws, tid, gload, lstore);
    __syncthreads();
    const cplx<T> Dx = dsym[kx];
    const T d2x = d2[kx];
    for (int e = tid; e < L * W; e += NTHR) {
        const int w = e % W;
        const int kz = e / W;
        const int ky = ky0 + w;
        cplx<T>* X = buf + w * LS + lpad(kz);
        if (kx == 0 && ky == 0 && kz == 0) {
            X[0] = cplx<T>{(T)mean_new[0], T(0)};
            X[W * LS] = cplx<T>{(T)mean_new[1], T(0)};
            X[2 * W * LS] = cplx<T>{(T)mean_new[2], T(0)};
            continue;
        }
        const cplx<T> Dy = dsym[ky], Dz = dsym[kz];
        const T D2 = d2x + d2[ky] + d2[kz];
        const cplx<T> rx = X[0], ry = X[W * LS], rz = X[2 * W * LS];
        const cplx<T> div = cadd(cadd(cmul(Dx, rx), cmul(Dy, ry)), cmul(Dz, rz));
        const T inv_d2 = field_rcp(D2);
        const T scale = field_rcp(c0 + c1 * D2);
        const cplx<T> g = {div.x * inv_d2, div.y * inv_d2};
        const cplx<T> px = csub(rx, cmul(cconj(Dx), g));
        const cplx<T> py = csub(ry, cmul(cconj(Dy), g));
        const cplx<T> pz = csub(rz, cmul(cconj(Dz), g));
        X[0] = cplx<T>{px.x * scale, px.y * scale};
        X[W * LS] = cplx<T>{py.x * scale, py.y * scale};
        X[2 * W * LS] = cplx<T>{pz.x * scale, pz.y * scale};
    }
    __syncthreads();
    line_fft_io<T, L, true, NLN, LS, NTHR, true, true, false>(buf, tws, tid, lload, gstore);
}

// Inverse x pass: the half spectra of a row pair are staged, combined into
// one complex line Z = X_even + i X_odd (Hermitian extension for kx > L/2,
// imaginary parts of kx = 0 and L/2 dropped), transformed, and the real and
// imaginary parts stored as the two velocity rows.
template <typename T, int L, bool KEEP>
__global__ void __launch_bounds__((Geo<T, L>::TXI))
k_x_inv(const cplx<T>* __restrict__ A, const cplx<T>* __restrict__ tw,
        T* __restrict__ vout, unsigned char* __restrict__ act, int part_out) {
    using G = Geo<T, L>;
    constexpr int NC = G::NC, R = G::RI, NL = G::NLI, NTHR = G::TXI, LS = G::LS;
    // The spectrum is not read again, and before the field is, more than the
    // L2s hold passes through them: both go past the caches' replacement where
    // what a block takes of them are whole 128-byte lines (its runs of R values of
    // the spectrum, its rows of the field).  Stores: the interpolation, whose boxes
    // of nodes overlap in the caches, 206 -> 186 us at 256^3 float32, 272 -> 260 at
    // 288^3, 885 -> 874 at 512^3, float64 112 -> 103 at 192^3, 247 -> 233 at 256^3; a
    // 192^3 float64 solve's forward x pass 147 -> 133.  Loads, with the stores: this
    // pass 178 -> 153 us at 256^3 float64, 1323 -> 1294 at 512^3; of split lines 135
    // -> 155 at 288^3 float32, 755 -> 930 at 512^3.  KEEP: neither, for a solve in
    // place whose velocity, force and spectrum the last-level cache holds together,
    // so that the next one finds its input there (144^3 float64: a solve 172 us, 186
    // with the hints; into another field 193 and 171, a dense step 365 and 358).
    constexpr bool LD_ONCE = !KEEP && R * 2 * sizeof(T) % 128 == 0;
    constexpr bool ST_ONCE = !KEEP && L * sizeof(T) % 128 == 0;
    constexpr int SS = NC + 1;  // staging row stride
    __shared__ cplx<T> stg[R * SS];
    __shared__ cplx<T> buf[NL * LS];
    __shared__ cplx<T> tws[L];
    const int tid = threadIdx.x;
    const int yb = blockIdx.x % (L / R);
    const int cz = blockIdx.x / (L / R);  // (box * 3 + c) * L + z
    const int y0 = yb * R;
    if (act) {
        unsigned char* pa = act + (size_t)(cz / (3 * L)) * L + cz % L;
        if (part_out) {
            if (!*pa) return;
        } else if (tid == 0 && yb == 0 && cz / L % 3 == 0) {
            *pa = 0;  // for the next binning
        }
    }
    for (int i = tid; i < L; i += NTHR) tws[i] = tw[i];
    const cplx<T>* in = A + (size_t)cz * NC * L + y0;
    {
        // all loads first (out-of-range slots re-read the first element)
        constexpr int K = (NC * R + NTHR - 1) / NTHR;
        cplx<T> ld[K];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int e = tid + k * NTHR;
            const int kx = e / R;
            const int rl = e - kx * R;
            const unsigned i = (unsigned)(e < NC * R ? kx * L + rl : 0);
            ld[k] = LD_ONCE ? ld32_once(in, i) : ld32(in, i);
        }
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int e = tid + k * NTHR;
            if (e < NC * R) {
                const int kx = e / R;
                const int rl = e - kx * R;
                cplx<T> X = ld[k];
                if (kx == 0 || kx == L / 2) X.y = T(0);
                stg[rl * SS + kx] = X;
            }
        }
    }
    __syncthreads();
    // first stage: the combined line Z = X_even + i X_odd read from the
    // staged half spectra; last stage: real and imaginary parts stored as
    // the two velocity rows
    const cplx<T>* sg = stg;
    auto ld = [sg](int line, int k) {
        cplx<T> X1, X2;
        if (k <= L / 2) {
            X1 = sg[(2 * line) * SS + k];
            X2 = sg[(2 * line + 1) * SS + k];
        } else {
            X1 = cconj(sg[(2 * line) * SS + (L - k)]);
            X2 = cconj(sg[(2 * line + 1) * SS + (L - k)]);
        }
        return cplx<T>{X1.x - X2.y, X1.y + X2.x};
    };
    T* out = vout + ((size_t)cz * L + y0) * L;
    auto st = [out](int line, int x, cplx<T> zz) {
        const unsigned i = (unsigned)((2 * line) * L + x);
        if (ST_ONCE) {
            st32_once(out, i, zz.x);
            st32_once(out, i + L, zz.y);
        } else {
            st32(out, i, zz.x);
            st32(out, i + L, zz.y);
        }
    };
    line_fft_io<T, L, true, NL, LS, NTHR, false, false, false>(buf, tws, tid, ld, st);
}

// Inverse plane pass: y and x together for one (component, z) plane per
// block, the plane held in LDS.  The real plane v[y][x] is produced as H =
// L/2 complex columns Z[y][j] = v[y][2j] + i v[y][2j+1]: from the half
// spectrum F[kx][ky] (kx = 0..H, layout A[c][z][kx][ky] of the z pass),
//   Z'[ky][k] = E' + i O',  E' = F[ky][k] + conj F[-ky][H-k],
//   O' = (F[ky][k] - conj F[-ky][H-k]) W^-k   (W = e^{-2 pi i / L}),
// the spectra of the even and odd samples (F[ky][k + H] = conj F[-ky][H-k]
// for a real plane), then inverse transforms along y (L points) and j
// (H points); Z[y][j] is the row pair (v[y][2j], v[y][2j+1]), unnormalised
// like the rest of the solve.  Element (row, column) of the plane sits at
// row * PS + lpad(column).  PLANES: only the planes with act are
// produced (a block takes those of active_planes); else act
// (nullable) is cleared.
template <typename T, int L, bool PLANES>
__global__ void __launch_bounds__((Geo<T, L>::TXY))
k_xy_inv(const cplx<T>* __restrict__ A, const cplx<T>* __restrict__ tw,
         T* __restrict__ vout, unsigned char* __restrict__ act, int ng) {
    using G = Geo<T, L>;
    constexpr int H = G::H, PS = G::PS, NC = G::NC, NTHR = G::TXY;
    __shared__ cplx<T> buf[L * PS];
    __shared__ cplx<T> tws[L];
    __shared__ cplx<T> twh[H];
    const int tid0 = threadIdx.x;
    const int nz = PLANES ? ng : L;
    const int bc = blockIdx.x / nz, z0 = blockIdx.x % nz;  // box * 3 + c
    unsigned long long todo = 1;
    if (PLANES) {
        todo = active_planes<L>(act + (size_t)(bc / 3) * L, z0, ng);
        if (todo == 0) return;
    } else if (act && tid0 == 0 && bc % 3 == 0) {
        act[(size_t)(bc / 3) * L + z0] = 0;  // for the next binning
    }
    for (int i = tid0; i < L; i += NTHR) tws[i] = tw[i];
    for (int i = tid0; i < H; i += NTHR) twh[i] = tw[2 * i];
    do {
    const int cz = PLANES ? bc * L + z0 + 8 * (__ffsll(todo) - 1)  // (box * 3 + c) * L + z
                          : (int)blockIdx.x;
    // (opaque in the loop over planes: the indices formed from it are not kept
    // across it, which spilled)
    int tid = tid0;
    if (PLANES) asm volatile("" : "+v"(tid));
    // stage the half spectrum: F[kx][ky] at row ky, column kx (0..H)
    const cplx<T>* in = A + (size_t)cz * NC * L;
    {
        // every load of the thread issued before the LDS stores (at most 11
        // complex values per thread: K <= (L/2 + 1) L / NTHR)
        constexpr int K = (NC * L + NTHR - 1) / NTHR;
        cplx<T> ld[K];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int e = tid + k * NTHR;
            ld[k] = ld32(in, (unsigned)(e < NC * L ? e : 0));
        }
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int e = tid + k * NTHR;
            if (e < NC * L) {
                const int kx = e / L;
                const int ky = e - kx * L;
                buf[ky * PS + lpad(kx)] = ld[k];
            }
        }
    }
    __syncthreads();
    // Z'[ky][k] in place.  Slot (ky, k) and its partner (-ky, H - k) are
    // formed from each other, so each work item owns both (k = 1 .. H/2;
    // at k = H/2 only ky <= L/2); column 0 pairs with column H:
    // Z'[ky][0] = F[ky][0] + conj F[-ky][H] + i (F[ky][0] - conj F[-ky][H]).
    {
        constexpr int NPAIR = L * (H / 2);  // items (ky, k), k = 1 .. H/2 (k = H/2: ky <= L/2)
        for (int e = tid; e < NPAIR + L / 2 + 1; e += NTHR) {
            if (e < NPAIR) {
                const int k = 1 + e / L;
                const int ky = e - (k - 1) * L;
                if (k == H / 2 && ky > L / 2) continue;
                const int kyn = ky == 0 ? 0 : L - ky;
                const int kn = H - k;
                const cplx<T> F1 = buf[ky * PS + lpad(k)];
                const cplx<T> F2 = buf[kyn * PS + lpad(kn)];
                // slot (ky, k): F1 with conj F2; slot (-ky, H-k): F2 with conj F1
                const cplx<T> w1 = cconj(tws[k]);   // W^-k
                const cplx<T> w2 = cconj(tws[kn]);  // W^-(H-k)
                const cplx<T> e1 = cadd(F1, cconj(F2)), o1 = cmul(csub(F1, cconj(F2)), w1);
                const cplx<T> e2 = cadd(F2, cconj(F1)), o2 = cmul(csub(F2, cconj(F1)), w2);
                buf[ky * PS + lpad(k)] = cplx<T>{e1.x - o1.y, e1.y + o1.x};
                if (kyn != ky || kn != k)
                    buf[kyn * PS + lpad(kn)] = cplx<T>{e2.x - o2.y, e2.y + o2.x};
            } else {
                const int ky = e - NPAIR;  // 0 .. L/2
                const int kyn = ky == 0 ? 0 : L - ky;
                const cplx<T> Fa0 = buf[ky * PS + lpad(0)], FaH = buf[ky * PS + lpad(H)];
                const cplx<T> Fb0 = buf[kyn * PS + lpad(0)], FbH = buf[kyn * PS + lpad(H)];
                const cplx<T> e1 = cadd(Fa0, cconj(FbH)), o1 = csub(Fa0, cconj(FbH));
                const cplx<T> e2 = cadd(Fb0, cconj(FaH)), o2 = csub(Fb0, cconj(FaH));
                buf[ky * PS + lpad(0)] = cplx<T>{e1.x - o1.y, e1.y + o1.x};
                if (kyn != ky) buf[kyn * PS + lpad(0)] = cplx<T>{e2.x - o2.y, e2.y + o2.x};
            }
        }
    }
    __syncthreads();
    auto col = [](int line, int e) { return e * PS + lpad(line); };
    lds_fft<T, L, true, H, NTHR, true>(buf, tws, tid, col);
    // along x; the last stage stores each complex Z'[y][j] as the real pair
    // v[y][2j], v[y][2j+1]
    cplx<T>* out = reinterpret_cast<cplx<T>*>(vout + (size_t)cz * L * L);
    const cplx<T>* lb = buf;
    auto ldl = [lb](int line, int e) { return lb[line * PS + lpad(e)]; };
    auto gst = [out](int line, int e, cplx<T> x) { st32(out, (unsigned)(line * H + e), x); };
    line_fft_io<T, H, true, L, PS, NTHR, false, true, false>(buf, twh, tid, ldl, gst);
    if (PLANES) __syncthreads();  // (another plane in buf)
    } while (PLANES && (todo &= todo - 1) != 0);
}

// Blocks that share the marked planes of a box (active_planes) in a pass whose
// whole launch would be n blocks for the batch, for about `marked` planes a box.
// One plane a block while the launch fills the chip a few times at most: blocks of
// planes without a mark end at once, and a block that takes up to L / 8 planes
// runs them one after another (19 particles in one 96^3 box, float32: x pass 15 us
// against 47, y 6.3 and 25, inverse plane 12 and 54; 4 boxes 32 and 53).  Above,
// the empty blocks cost more than the chain (32 64^3 boxes of two particles: x
// pass of 24,576 blocks 32 against 25; 32 48^3, 13,824: 18.6 and 16.5), at half
// the number in the inverse plane pass, whose blocks take more LDS (32 64^3, 6,144:
// 19 and 16).  Marks of at most two a block are dealt out too, unless they are all
// the planes: the other blocks would be empty (pairs in each of 16 64^3 boxes,
// float64: y pass 5.9 us against 8.4, inverse plane 13 and 23; one particle in each
// of 8: a step 53 and 58; in 128^3: inverse plane 9.4 and 13.4).
inline int plane_blocks(int64_t n, int marked, int L) {
    return n <= 8192 && (marked > 16 || marked >= L) ? L : 8;
}

template <typename T, int L>
hipError_t solve_sized(mb_grid* g, const T* v_in, const SolveForce<T>& F, T* v_out,
                       hipStream_t s) {
    using G = Geo<T, L>;
    const bool steady = g->d.mode == MB_STEADY_STOKES;
    const bool rhs = steady || F.rhs_only;  // the force alone is transformed
    const double h = g->d.h;
    const double N = (double)g->N;
    cplx<T>* A = (cplx<T>*)g->d_spec;
    const cplx<T>* tw = (const cplx<T>*)g->d_tw;
    const T a = rhs ? T(0) : (T)(g->d.rho / g->d.dt);
    const T b = rhs ? T(0) : (T)(0.5 * g->d.eta / (h * h));
    const int nbox = g->tiles.nbox;
    ForceSrc<T> mk{};
    const T* fin = F.f;
    if (F.src != SolveForce<T>::FIELD) {
        fin = (const T*)g->d_box;
        mk.add = F.f;
    }
    if (F.src == SolveForce<T>::RECORDS) {
        mk.rec = rec_geo<T>(g);
        mk.recf = rec_force<T>(g);
        mk.mbox = F.mbox;
        mk.fexp = g->d_rank;
        if (F.planes) mk.act = g->d_act;
        mk.ng = plane_blocks((int64_t)G::NBX * nbox, F.marked, L);
    }
    if (!small_edge(L) && F.src == SolveForce<T>::RECORDS) return hipErrorInvalidValue;
    unsigned char* act = mk.act ? g->d_act : nullptr;
    const int part = F.planes && F.planes_out ? 1 : 0;
#define MB_XF(SR, ST)                                                                     \
    MB_LAUNCH(g, K_FFT_X_FWD, s, (k_x_fwd<T, L, SR, ST>),                             \
              (act ? G::NBX / L * mk.ng : G::NBX) * nbox, (threads_xf<T, L, SR, ST>()), 0, \
              v_in, fin, g->btiles, mk, tw, a, b, A, g->d_psum)
    if (F.src == SolveForce<T>::FIELD) {
        if (rhs) MB_XF(SRC_FIELD, true);
        else MB_XF(SRC_FIELD, false);
    } else if (F.src == SolveForce<T>::RECORDS) {
        if constexpr (small_edge(L)) {
            if (rhs) MB_XF(SRC_REC, true);
            else MB_XF(SRC_REC, false);
        }
    } else if (mk.add) {
        if (rhs) MB_XF(SRC_BOX_ADD, true);
        else MB_XF(SRC_BOX_ADD, false);
    } else {
        if (rhs) MB_XF(SRC_BOX, true);
        else MB_XF(SRC_BOX, false);
    }
#undef MB_XF
    const int ngy = plane_blocks((int64_t)3 * L * G::NCHY * nbox, F.marked, L);
#define MB_Y(ID, INV, AC)                                                                 \
    MB_LAUNCH(g, ID, s, (k_y<T, L, INV, AC>), 3 * (AC ? ngy : L) * G::NCHY * nbox, G::TY, 0, \
              A, tw, (const unsigned char*)act, ngy)
    if (act) {
        if constexpr (small_edge(L)) MB_Y(K_FFT_Y_FWD, false, true);
    } else {
        MB_Y(K_FFT_Y_FWD, false, false);
    }
    const T c0 = steady ? T(0) : (T)(g->d.rho / g->d.dt * N);
    const T c1 = steady ? (T)(g->d.eta * N) : (T)(0.5 * g->d.eta * N);
    const double mv = rhs ? 0.0 : 1.0 / N;
    const double mf = steady ? 0.0 : g->d.dt / g->d.rho / N;
    const int zm = (steady || g->d.zero_mean) ? 1 : 0;
#define MB_Z(AC)                                                                          \
    MB_LAUNCH(g, K_FFT_Z_SPECTRAL, s, (k_z_solve<T, L, AC>), G::NC * (L / G::WZ) * nbox,   \
              G::TZ, 0, A, tw, (const cplx<T>*)g->d_dsym, (const T*)g->d_d2, c0, c1, zm,   \
              g->d_psum, G::NBX / 3, mv, mf, (const unsigned char*)act, part)
    if (act) {
        if constexpr (small_edge(L)) MB_Z(true);
    } else {
        MB_Z(false);
    }
#undef MB_Z
    if constexpr (G::XY) {
        const int ngx = plane_blocks((int64_t)2 * G::NBXY * nbox, F.marked, L);
        if (part)
            MB_LAUNCH(g, K_FFT_XY_INV, s, (k_xy_inv<T, L, true>), 3 * ngx * nbox, G::TXY, 0,
                      A, tw, v_out, act, ngx);
        else
            MB_LAUNCH(g, K_FFT_XY_INV, s, (k_xy_inv<T, L, false>), G::NBXY * nbox, G::TXY, 0, A,
                      tw, v_out, act, L);
    } else {
        if (part) {
            if constexpr (small_edge(L)) MB_Y(K_FFT_Y_INV, true, true);
        } else {
            MB_Y(K_FFT_Y_INV, true, false);
        }
#define MB_XI(KEEP)                                                                       \
    MB_LAUNCH(g, K_FFT_X_INV, s, (k_x_inv<T, L, KEEP>), 3 * L * (L / G::RI) * nbox, G::TXI, 0, A, \
              tw, v_out, act, part)
        // v, f and the spectrum of all boxes against the 256 MB last-level cache
        constexpr int64_t three = (int64_t)9 * L * L * L * sizeof(T), room = (int64_t)224 << 20;
        const bool in_place = F.src == SolveForce<T>::FIELD && (v_out == v_in || v_out == F.f);
        if constexpr (three <= room) {
            if (in_place && three * nbox <= room) MB_XI(true);
            else MB_XI(false);
        } else {
            MB_XI(false);
        }
#undef MB_XI
    }
#undef MB_Y
    return hipGetLastError();
}

}  // namespace fft

#ifndef MB_FFT_SIZES
#define MB_FFT_SIZES(X) \
    X(8) X(16) X(24) X(32) X(48) X(64) X(72) X(96) X(128) X(144) X(192) \
    X(216) X(256) X(288) X(384) X(432) X(512)
#endif

template <typename T>
hipError_t fluid_solve(mb_grid* g, const T* v_in, const SolveForce<T>& force, T* v_out,
                       hipStream_t s) {
    switch (g->L) {
#define MB_CASE(n) \
    case n: return fft::solve_sized<T, n>(g, v_in, force, v_out, s);
        MB_FFT_SIZES(MB_CASE)
#undef MB_CASE
    }
    return hipErrorInvalidValue;
}

int fft_x_blocks(int L, int precision) {
    switch (L) {
#define MB_CASE(n) \
    case n: return precision == MB_MIXED ? fft::Geo<float, n>::NBX : fft::Geo<double, n>::NBX;
        MB_FFT_SIZES(MB_CASE)
#undef MB_CASE
    }
    return 0;
}

template hipError_t fluid_solve<float>(mb_grid*, const float*, const SolveForce<float>&, float*, hipStream_t);
template hipError_t fluid_solve<double>(mb_grid*, const double*, const SolveForce<double>&, double*, hipStream_t);

}  // namespace mb
