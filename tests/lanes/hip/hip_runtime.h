// What the kernels' sources need of the HIP runtime, for a CPU build that checks every access (see lanes.cpp): lanes are
// fibres, a workgroup's run until they wait for each other, and pointers with an address space are objects that know what
// may be touched.  For the tests only; speed and memory order are not looked at.
#pragma once
#include <algorithm>
#include <cmath>
#include <cstddef>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <type_traits>
#include <vector>

#define __device__
#define __host__
#define __global__
#define __forceinline__ inline
#define __shared__ static  // (a workgroup runs to its end before the next)
#define __launch_bounds__(...)
#define __align__(n) __attribute__((aligned(n)))

struct dim3 {
    unsigned x, y, z;
    dim3(unsigned a = 1, unsigned b = 1, unsigned c = 1) : x(a), y(b), z(c) {}
};
struct uint2 { uint32_t x, y; };
struct uint4 { uint32_t x, y, z, w; };
struct float4 { float x, y, z, w; };
inline uint2 make_uint2(uint32_t a, uint32_t b) { return {a, b}; }

namespace lanes {
struct Lane {
    dim3 tid, bid, bdim, gdim;
};
extern Lane *now;
uintptr_t lds_base();
size_t lds_size();
inline unsigned char *lds() { return reinterpret_cast<unsigned char *>(lds_base()); }
inline int lane() { return (int)(now->tid.x & 63u); }
const uint64_t *wave_values(uint64_t v);  // of the wavefront's 64 lanes, once all have come here
const uint64_t *row_values(uint64_t v);   // of a row's 16 lanes, [lane of the wavefront]
void barrier();
bool inside(uintptr_t at, size_t n);      // of one allocation
void report(const char *what, uintptr_t at, size_t n);
void launch(std::function<void()> kernel, dim3 grid, dim3 block, size_t lds_bytes, const char *name);
int compute_units();

// A pointer to global memory (address space 1, 4: an address) or to LDS (3: an offset into the workgroup's).
template <int SPACE, class T>
struct Ptr {
    uintptr_t at = 0;
    using Value = typename std::remove_const<T>::type;
    using Result = typename std::conditional<std::is_const<T>::value, Value, T &>::type;  // (loads may be misaligned)
    Ptr() = default;
    Ptr(std::nullptr_t) {}
    Ptr(const Ptr &) = default;
    Ptr &operator=(const Ptr &) = default;
    explicit Ptr(uintptr_t a) : at(a) {}
    template <class U> explicit Ptr(U *p) : at(reinterpret_cast<uintptr_t>(p)) { if (SPACE == 3 && p) at -= lds_base(); }
    template <class U> explicit Ptr(const Ptr<SPACE, U> &o) : at(o.at) {}
    template <class U, class = typename std::enable_if<std::is_convertible<U *, T *>::value>::type>
    Ptr(const Ptr<SPACE, U> &o, int = 0) : at(o.at) {}
    explicit operator uintptr_t() const { return at; }
    explicit operator bool() const { return at != 0; }
    explicit operator T *() const { return &ref(at); }
    T &ref(uintptr_t a) const
    {
        static Value nothing;
        if (SPACE == 3 ? a + sizeof(T) > lds_size() : !inside(a, sizeof(T))) {
            report(SPACE == 3 ? "LDS" : "global memory", a, sizeof(T));
            return nothing;
        }
        return *reinterpret_cast<T *>(SPACE == 3 ? lds_base() + a : a);
    }
    Value get(uintptr_t a, std::true_type) const
    {
        Value v;
        memcpy((void *)&v, (const void *)&ref(a), sizeof v);
        return v;
    }
    T &get(uintptr_t a, std::false_type) const { return ref(a); }
    Result operator[](long long i) const { return get(at + (uintptr_t)(i * (long long)sizeof(T)), std::is_const<T>()); }
    Result operator*() const { return get(at, std::is_const<T>()); }
    T *operator->() const { return &ref(at); }
    Ptr operator+(long long i) const { return Ptr(at + (uintptr_t)(i * (long long)sizeof(T))); }
};
}  // namespace lanes

#define threadIdx (lanes::now->tid)
#define blockIdx (lanes::now->bid)
#define blockDim (lanes::now->bdim)
#define gridDim (lanes::now->gdim)

template <class A, class B> inline typename std::common_type<A, B>::type min(A a, B b)
{
    using C = typename std::common_type<A, B>::type;
    return (C)a < (C)b ? (C)a : (C)b;
}
template <class A, class B> inline typename std::common_type<A, B>::type max(A a, B b)
{
    using C = typename std::common_type<A, B>::type;
    return (C)a > (C)b ? (C)a : (C)b;
}
template <class To, class From> inline To bits_as(From v)
{
    To t;
    memcpy(&t, &v, sizeof t);
    return t;
}
inline float __uint_as_float(uint32_t v) { return bits_as<float>(v); }
inline uint32_t __float_as_uint(float v) { return bits_as<uint32_t>(v); }
inline float __int_as_float(int v) { return bits_as<float>(v); }
inline int __float_as_int(float v) { return bits_as<int>(v); }
inline int __popc(uint32_t v) { return __builtin_popcount(v); }
inline int __popcll(unsigned long long v) { return __builtin_popcountll(v); }
inline int __ffs(int v) { return __builtin_ffs(v); }
inline int __ffsll(unsigned long long v) { return __builtin_ffsll((long long)v); }
inline uint32_t __umul24(uint32_t a, uint32_t b) { return (a & 0xFFFFFFu) * (b & 0xFFFFFFu); }
template <class T> inline T atomicAdd(T *p, T v) { T o = *p; *p += v; return o; }
template <class T> inline T atomicOr(T *p, T v) { T o = *p; *p |= v; return o; }
template <class T> inline T atomicAnd(T *p, T v) { T o = *p; *p &= v; return o; }
template <class T> inline T atomicCAS(T *p, T expected, T v) { T o = *p; if (o == expected) *p = v; return o; }
#define __hip_atomic_store(p, v, ...) (*(p) = (v))
#define __hip_atomic_load(p, ...) (*(p))
#define __builtin_nontemporal_store(v, p) (*(p) = (v))

// ---- lanes that wait for each other
inline void __syncthreads() { lanes::barrier(); }
inline unsigned long long __ballot(bool p)
{
    const uint64_t *v = lanes::wave_values(p);
    unsigned long long r = 0;
    for (int i = 0; i < 64; i++) r |= (unsigned long long)(v[i] & 1u) << i;
    return r;
}
inline bool __any(bool p) { return __ballot(p) != 0; }
inline bool __all(bool p) { return __ballot(p) == ~0ull; }
template <class T> inline T value_of_lane(T v, int from, bool valid)
{
    uint64_t bits = 0;
    memcpy(&bits, &v, sizeof v);
    const uint64_t *all = lanes::wave_values(bits);
    if (valid) memcpy(&v, &all[from & 63], sizeof v);
    return v;
}
template <class T> inline T __shfl(T v, int from, int = 64) { return value_of_lane(v, from, true); }
template <class T> inline T __shfl_xor(T v, int d, int = 64) { return value_of_lane(v, lanes::lane() ^ d, true); }
template <class T> inline T __shfl_up(T v, int d, int = 64) { return value_of_lane(v, lanes::lane() - d, lanes::lane() >= d); }
template <class T> inline T __shfl_down(T v, int d, int = 64) { return value_of_lane(v, lanes::lane() + d, lanes::lane() + d < 64); }
inline int lanes_update_dpp(int old, int src, int ctrl, int row_mask, int, bool zero_outside)
{
    const uint64_t *all = ctrl < 0x130 ? lanes::row_values((uint32_t)src) : lanes::wave_values((uint32_t)src);
    const int l = lanes::lane(), row = l >> 4, i = l & 15, n = ctrl & 15;
    int from = -1;
    if (ctrl >= 0x111 && ctrl <= 0x11f) from = i >= n ? l - n : -1;                         // row_shr
    else if (ctrl >= 0x121 && ctrl <= 0x12f) from = (l & 48) | ((i - n) & 15);              // row_ror
    else if (ctrl == 0x142) from = row >= 1 ? 16 * row - 1 : -1;                            // row_bcast:15
    else if (ctrl == 0x143) from = row >= 2 ? 31 : -1;                                      // row_bcast:31
    else abort();
    if (!((row_mask >> row) & 1)) return old;
    return from >= 0 ? (int)(uint32_t)all[from] : (zero_outside ? 0 : old);
}
inline int lanes_readlane(int v, int from) { return (int)(uint32_t)lanes::wave_values((uint32_t)v)[from & 63]; }
#define __builtin_amdgcn_update_dpp lanes_update_dpp
#define __builtin_amdgcn_readlane lanes_readlane
#define __builtin_amdgcn_readfirstlane(v) lanes_readlane(v, 0)
#define __builtin_amdgcn_wave_barrier() ((void)lanes::wave_values(0))
#define __builtin_amdgcn_s_barrier() lanes::barrier()
#define __builtin_amdgcn_fence(...) ((void)0)
#define __builtin_amdgcn_s_setprio(x) ((void)0)
#define __builtin_amdgcn_s_sleep(x) ((void)0)
#define __builtin_amdgcn_sched_barrier(x) ((void)0)

// ---- instructions
inline uint32_t lanes_perm(uint32_t a, uint32_t b, uint32_t select)
{
    const uint64_t bytes = (uint64_t)a << 32 | b;
    uint32_t r = 0;
    for (int i = 0; i < 4; i++) {
        const uint32_t k = (select >> (8 * i)) & 255u;
        if (k > 7 && k != 12) abort();
        r |= (k == 12 ? 0u : (uint32_t)(bytes >> (8 * k)) & 255u) << (8 * i);
    }
    return r;
}
template <class V> inline float lanes_dot2(V a, V b, float c, bool)
{
    const uint32_t x = bits_as<uint32_t>(a), y = bits_as<uint32_t>(b);
    return c + __uint_as_float(x << 16) * __uint_as_float(y << 16) + __uint_as_float(x & 0xFFFF0000u) * __uint_as_float(y & 0xFFFF0000u);
}
inline uint32_t lanes_udot4(uint32_t a, uint32_t b, uint32_t c, bool)
{
    for (int i = 0; i < 32; i += 8) c += ((a >> i) & 255u) * ((b >> i) & 255u);
    return c;
}
inline uint32_t lanes_mbcnt(uint32_t mask, uint32_t c, int below) { return c + (below >= 32 ? __popc(mask) : (below > 0 ? __popc(mask & ((1u << below) - 1u)) : 0)); }
inline uint32_t lanes_ubfe(uint32_t v, uint32_t at, uint32_t n) { return n & 31u ? (v >> (at & 31u)) & ((1u << (n & 31u)) - 1u) : 0u; }
inline int lanes_sbfe(int v, uint32_t at, uint32_t n)
{
    at &= 31u, n &= 31u;
    return n ? (int)((uint32_t)v << (32 - at - n)) >> (32 - n) : 0;
}
inline uint32_t lanes_med3(uint32_t a, uint32_t b, uint32_t c) { return std::max(std::min(a, b), std::min(std::max(a, b), c)); }
#define __builtin_amdgcn_perm lanes_perm
#define __builtin_amdgcn_fdot2_f32_bf16 lanes_dot2
#define __builtin_amdgcn_udot4 lanes_udot4
#define __builtin_amdgcn_mbcnt_lo(m, c) lanes_mbcnt(m, c, lanes::lane())
#define __builtin_amdgcn_mbcnt_hi(m, c) lanes_mbcnt(m, c, lanes::lane() - 32)
#define __builtin_amdgcn_ubfe lanes_ubfe
#define __builtin_amdgcn_sbfe lanes_sbfe
#define __builtin_amdgcn_alignbit(hi, lo, s) ((uint32_t)(((uint64_t)(hi) << 32 | (lo)) >> ((s) & 31u)))

// ---- the host's side: one device, whose memory is the host's
typedef int hipError_t;
typedef void *hipStream_t, *hipEvent_t;
enum { hipSuccess, hipMemcpyHostToDevice, hipFuncAttributeMaxDynamicSharedMemorySize, hipEventDisableTiming, hipStreamNonBlocking,
       hipDeviceAttributeMultiprocessorCount, hipDeviceAttributeMaxSharedMemoryPerBlock };
struct hipFuncAttributes {
    size_t sharedSizeBytes = 0;
};
inline hipError_t hipFuncGetAttributes(hipFuncAttributes *, const void *) { return hipSuccess; }
inline hipError_t hipFuncSetAttribute(const void *, int, int) { return hipSuccess; }
inline hipError_t hipGetLastError() { return hipSuccess; }
inline hipError_t hipGetDevice(int *d) { return *d = 0, hipSuccess; }
inline hipError_t hipDeviceGetAttribute(int *v, int what, int)
{
    *v = what == hipDeviceAttributeMultiprocessorCount ? lanes::compute_units() : 160 * 1024;
    return hipSuccess;
}
inline hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, int, hipStream_t) { return memcpy(d, s, n), hipSuccess; }
inline hipError_t hipEventCreateWithFlags(hipEvent_t *, int) { return hipSuccess; }
inline hipError_t hipStreamCreateWithFlags(hipStream_t *, int) { return hipSuccess; }
inline hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
inline hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, int) { return hipSuccess; }
inline hipError_t hipGetSymbolAddress(void **p, void *s) { return *p = s, hipSuccess; }
#define HIP_SYMBOL(x) ((void *)(x))
#define hipLaunchKernelGGL(kernel, grid, block, lds_bytes, stream, ...) \
    lanes::launch([=]() { (kernel)(__VA_ARGS__); }, (grid), (block), (lds_bytes), #kernel)
