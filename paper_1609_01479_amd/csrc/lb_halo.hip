// Face exchange of an x-slab shard: the one-GPU part of the paper's domain
// decomposition with halo regions (Sec. 2.1.1: every stencil kernel reads a
// halo populated from the neighbouring sub-domains; Sec. 5: the decomposed
// runs).  A shard owns planes 0 .. nx-1 of a lattice split along x; its time
// levels also hold halo planes -2, -1 and nx, nx+1 (F, G) and -1, nx (phi_c),
// which the single-pass step reads in place of a periodic wrap.
//
// What the step at plane 0 reads from below: the f and g populations moving
// +x out of plane -1 (pulls into plane 0), and every population that forms
// phi at plane -1 (its stencil neighbour): g with c_x = 0 at plane -1, g with
// c_x = +1 at plane -2 and, with FP32 storage, phi_c of plane -1.  (The g
// with c_x = -1 come from plane 0, the shard's own.)  Mirror images above.
// One face buffer carries exactly that, 24 component planes of ny*nz values
// of the storage type in site order y*nz + z, then (FP32 storage) the plane
// of phi_c words:
//   slots 0..4    f_i with c_x = s of the boundary plane
//   slots 5..18   g_i with c_x in {0, s} of the boundary plane
//   slots 19..23  g_i with c_x = s of the plane behind it (one further in)
// with s = +1 for the face sent up (boundary plane nx-1, behind it nx-2;
// stored by the receiver as its planes -1 and -2) and s = -1 for the face
// sent down (planes 0 and 1; stored as the receiver's nx and nx+1).  A
// periodic lattice on one GPU is the shard that receives its own faces.
#include "lb_device.h"

namespace lbk {

using namespace dev;

namespace {

constexpr int kFaceSlots = 24;

// component of slot k for direction sign +1 and -1: the components with
// c_x = s in index order, then those with c_x in {0, s}, then c_x = s again
struct SlotTable {
    signed char c[2][kFaceSlots];
};
constexpr SlotTable slot_table()
{
    SlotTable t{};
    for (int d = 0; d < 2; d++) {
        const int s = d ? -1 : 1;
        int n = 0;
        for (int i = 0; i < NV; i++)
            if (CX[i] == s) t.c[d][n++] = i;
        for (int i = 0; i < NV; i++)
            if (CX[i] == 0 || CX[i] == s) t.c[d][n++] = i;
        for (int i = 0; i < NV; i++)
            if (CX[i] == s) t.c[d][n++] = i;
    }
    return t;
}

// One face: the direction it travels (s = +1 up, -1 down) and its boundary
// plane xb in this level, with xb - s behind it.
struct Face {
    void* buf;
    int s, xb;
};

// PACK: buffer <- level; else level <- buffer (into halo planes xb and
// xb - s).  Both faces in one launch (grid z), every slot of a site by one
// thread: the site's offset is formed once, and all its loads are in flight
// together.  32 x 256 x 256 a step with its face copies: FP32 164 us with four
// launches of a thread per value, 141 so, FP64 282 and 265; 8 x 24 x 30 22 and
// 17.
template <typename T, bool REF, bool PACK>
__global__ __launch_bounds__(kBlock) void k_faces(KParams p, T* __restrict__ F, T* __restrict__ G,
                                                  unsigned* __restrict__ phic, Face f0, Face f1)
{
    constexpr SlotTable tab = slot_table();
    const Face f = blockIdx.z ? f1 : f0;
    const int a = p.ny * p.nz;
    const int yz = blockIdx.x * int(blockDim.x) + threadIdx.x;
    if (yz >= a) return;
    const int y = yz / p.nz, z = yz - y * p.nz;
    const unsigned front = didx(p, 0, f.xb, y, z), behind = didx(p, 0, f.xb - f.s, y, z);
    T* __restrict__ b = static_cast<T*>(f.buf);
    const bool up = f.s > 0;
    auto copy = [&](int k) __attribute__((always_inline)) {
        const unsigned comp = unsigned(up ? tab.c[0][k] : tab.c[1][k]) * p.cs;
        T* q = (k < 5 ? F : G) + ((k >= 19 ? behind : front) + comp);
        if (PACK)
            return *q;
        *q = b[size_t(k) * a + yz];
        return T(0);
    };
    // a share of the slots per grid row (all of them unless the face is small)
    const int per = (kFaceSlots + gridDim.y - 1) / gridDim.y;
    const int k0 = blockIdx.y * per;
    if (gridDim.y == 1) {
        T v[kFaceSlots];
#pragma unroll
        for (int k = 0; k < kFaceSlots; k++) v[k] = copy(k);
        if (PACK)
#pragma unroll
            for (int k = 0; k < kFaceSlots; k++) b[size_t(k) * a + yz] = v[k];
    } else {
        for (int k = k0; k < k0 + per && k < kFaceSlots; k++) {
            const T v = copy(k);
            if (PACK) b[size_t(k) * a + yz] = v;
        }
    }
    if (REF && blockIdx.y == 0) {
        unsigned* pb = reinterpret_cast<unsigned*>(b + size_t(kFaceSlots) * a);
        const int c = phic_site(p, f.xb, y, z);
        if (PACK) pb[yz] = phic[c];
        else phic[c] = pb[yz];
    }
}

}  // namespace

size_t face_bytes(const KParams& p, bool fp32)
{
    const size_t a = size_t(p.ny) * p.nz;
    const size_t b = fp32 ? (kFaceSlots + 1) * a * 4 : kFaceSlots * a * 8;
    return (b + 255) / 256 * 256;
}

template <typename T>
static hipError_t faces(const KParams& p, void* state, Face f0, Face f1, int nf, bool pack,
                        hipStream_t st)
{
    constexpr bool F32 = sizeof(T) == 4;
    Lvl<T> l = level<T>(state, p, F32);
    const int a = p.ny * p.nz;
    // small faces: single waves, and the slots dealt out to more of them
    const int nt = a <= 16384 ? 64 : kBlock, rows = a <= 16384 ? kFaceSlots / 4 : 1;
    const dim3 grid((a + nt - 1) / nt, rows, nf);
    auto k = pack ? k_faces<T, F32, true> : k_faces<T, F32, false>;
    k<<<grid, nt, 0, st>>>(p, l.F, l.G, l.phic, f0, f1);
    return hipGetLastError();
}

hipError_t launch_faces(const KParams& p, bool fp32, void* state, void* lo, void* hi, bool pack,
                        hipStream_t st)
{
    // packed: the face sent down (planes 0 and 1, c_x = -1) and the one sent
    // up (planes nx-1 and nx-2, c_x = +1); unpacked: the lower neighbour's
    // upward face into planes -1 and -2, the upper one's downward face into
    // planes nx and nx+1
    const Face flo{lo, pack ? -1 : +1, pack ? 0 : -1};
    const Face fhi{hi, pack ? +1 : -1, pack ? p.nx - 1 : p.nx};
    const int nf = (lo ? 1 : 0) + (hi ? 1 : 0);
    if (nf == 0) return hipSuccess;
    const Face f0 = lo ? flo : fhi;
    return fp32 ? faces<float>(p, state, f0, fhi, nf, pack, st)
                : faces<double>(p, state, f0, fhi, nf, pack, st);
}

}  // namespace lbk
