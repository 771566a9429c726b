// Internal declarations of libdwf (host and device).
//
// Internal field ("half field"): one parity, one right-hand side, Ls slices of
// 12 components (spin * 3 + colour) at the internal sites of that parity (see
// build_geometry; lex_of_site gives the lexicographic site), complex stored as
// (re, im) pairs of the storage type.  Multi-RHS fields put the RHS index
// outermost.  Sites come in tiles of 16 whose data are contiguous (precision.h);
// Vhp is Vh rounded up to whole tiles, and padding entries stay zero.
//
// Links per output parity p ("hop links"), directions d = 0..3: U_mu(x) (forward
// hop to x+mu), d = 4..7: U_mu(x-mu)^dag, with the antiperiodic time phase folded
// in.  Neighbours: internal index (other parity) of x+mu (d < 4) or x-mu (d >= 4).
// Both are tables of the same tiles, parity 0 first.
#pragma once

#include <hip/hip_runtime.h>
#include <hip/hip_bf16.h>

#include <cstdint>
#include <exception>
#include <memory>
#include <mutex>
#include <string>
#include <utility>
#include <vector>

#include "../../include/dwf.h"

namespace dwf {

// ---------------------------------------------------------------------
// error handling
// ---------------------------------------------------------------------
void set_error(const std::string& msg);
struct Error {
    int code;
    std::string msg;
};

#define DWF_HIP(call)                                                              \
    do {                                                                           \
        hipError_t e_ = (call);                                                    \
        if (e_ != hipSuccess)                                                      \
            throw ::dwf::Error{DWF_EHIP, std::string(#call) + ": " + hipGetErrorString(e_)}; \
    } while (0)

#define DWF_REQUIRE(cond, code, msg)                                               \
    do {                                                                           \
        if (!(cond)) throw ::dwf::Error{(code), (msg)};                            \
    } while (0)

// Frees the idle call scratch (scratch.cpp); false if there was none.
bool release_scratch();

// ---------------------------------------------------------------------
// device buffer (RAII)
// ---------------------------------------------------------------------
struct DevBuf {
    void* p = nullptr;
    size_t bytes = 0;
    DevBuf() = default;
    explicit DevBuf(size_t n) { alloc(n); }
    DevBuf(const DevBuf&) = delete;
    DevBuf& operator=(const DevBuf&) = delete;
    DevBuf(DevBuf&& o) noexcept : p(o.p), bytes(o.bytes) { o.p = nullptr; o.bytes = 0; }
    DevBuf& operator=(DevBuf&& o) noexcept {
        if (this != &o) { release(); p = o.p; bytes = o.bytes; o.p = nullptr; o.bytes = 0; }
        return *this;
    }
    ~DevBuf() { release(); }
    void alloc(size_t n) {
        release();
        if (n == 0) return;
        hipError_t e = hipMalloc(&p, n);
        if (e == hipErrorOutOfMemory && release_scratch()) {   // give back idle scratch first
            (void)hipGetLastError();
            e = hipMalloc(&p, n);
        }
        if (e != hipSuccess) {
            p = nullptr;
            throw Error{DWF_ENOMEM, "hipMalloc(" + std::to_string(n) + " bytes) failed"};
        }
        bytes = n;
        // fields keep zero padding past the last site (whole tiles of 16)
        e = hipMemset(p, 0, n);
        if (e != hipSuccess) throw Error{DWF_EHIP, "hipMemset failed"};
    }
    void release() {
        if (p) (void)hipFree(p);
        p = nullptr;
        bytes = 0;
    }
    template <class T> T* as() const { return static_cast<T*>(p); }
};

// Call scratch (scratch.cpp): temporaries of one operator application, kept
// between calls because their hipMalloc and hipFree cost more than the
// application (24^3x48, Ls = 16, FP32 normal operator: 2.3 ms of kernels in a
// call of 5 to 58 ms).  Idle buffers serve every operator of the same Ls and
// sites per parity on the same device (ScratchKey: one size and one layout, so
// that the zero padding of a field stays valid).  All idle buffers together are
// at most SCRATCH_IDLE_MAX, the oldest freed first: 3 % of the device's memory,
// and room for the largest call on 24^3x48, Ls = 16 (6.1 GB).  They are freed with
// the last operator of their shape, by release_scratch(), and when an allocation
// of the library finds no memory.  A call takes its own buffers, so calls from
// several threads never share one.
constexpr size_t SCRATCH_IDLE_MAX = size_t(8) << 30;
struct ScratchKey {
    // half fields by StoreKind; two-slice FP64 fields; scalars
    enum Class { F64 = 0, F32 = 1, BF16 = 2, PAIR = 3, SMALL = 4 };
    int dev, cls, Ls;
    long Vh;
    bool operator==(const ScratchKey& o) const { return dev == o.dev && cls == o.cls && Ls == o.Ls && Vh == o.Vh; }
};
DevBuf scratch_take(const ScratchKey& key, size_t bytes);
void scratch_give(const ScratchKey& key, DevBuf&& b) noexcept;

// An operator's claim to the idle buffers of its shape, on the device that is
// current when it is made.
class ScratchUser {
    ScratchKey shape_{0, 0, 0, 0};
public:
    ScratchUser() = default;
    ScratchUser(const ScratchUser&) = delete;
    ScratchUser& operator=(const ScratchUser&) = delete;
    ~ScratchUser();
    void attach(int Ls, long Vh);
    ScratchKey key(int cls) const { return {shape_.dev, cls, shape_.Ls, shape_.Vh}; }
};

// A scratch buffer for the length of one call.  It becomes idle at the end of
// the scope, when the work that uses it must have completed; a scope left by an
// exception, with work possibly in flight, frees it instead.
class Scratch {
    ScratchKey key_;
    int exc_;
    DevBuf b_;
public:
    void* p;
    Scratch(const ScratchKey& key, size_t bytes)
        : key_(key), exc_(std::uncaught_exceptions()), b_(scratch_take(key_, bytes)), p(b_.p) {}
    Scratch(const Scratch&) = delete;
    Scratch& operator=(const Scratch&) = delete;
    ~Scratch() {
        if (std::uncaught_exceptions() == exc_) scratch_give(key_, std::move(b_));
    }
    template <class T> T* as() const { return static_cast<T*>(p); }
};

// ---------------------------------------------------------------------
// fifth-dimension matrices (host FP64), built in fifth_dim.cpp
// ---------------------------------------------------------------------
constexpr int LS_MAX = 16;   // the fused hop pads s to 16 rows (one MFMA tile)

struct FifthDim {
    int Ls = 0;
    // per chirality chi (0: P+ = spins 0,1; 1: P- = spins 2,3), row-major Ls x Ls
    std::vector<double> T[2], M5[2], K[2], N[2], M[2], Minv[2], Q[2];
};
// b, c: the coefficients b_s, c_s of D_+^(s), D_-^(s), s = 0..Ls-1
FifthDim build_fifth_dim(int Ls, double M0, double m, const std::vector<double>& b, const std::vector<double>& c,
                         double alpha);

enum StoreKind { ST_F64 = 0, ST_F32 = 1, ST_BF16 = 2 };

// ---------------------------------------------------------------------
// lattice / operator objects
// ---------------------------------------------------------------------
}  // namespace dwf

struct dwf_lattice {
    int dims[4];
    int antiperiodic_t;
    long V, Vh, Vhp;   // sites, sites per parity, those rounded up to whole tiles
    int brick[3] = {0, 0, 0};       // spatial brick extents of the internal site order
    int site_order = 0;             // 0 bricks swept in t, 1 t columns (build_geometry)
    dwf::DevBuf random_site;        // even sites: place in the random fields (empty: the site itself)
    std::vector<int> lex_of_site;   // host [2][Vh]: lexicographic index of internal site
    dwf::DevBuf nbr;                // device: per parity, in tiles of 16 sites (precision.h), 8 Vhp entries
    dwf::DevBuf lex_of_site_dev;    // device [2][Vh]
    dwf::DevBuf links[3];           // per storage kind and parity, in tiles (lidx; link_elems_parity(Vhp, ..) complex)
    bool has_gauge = false;
};

// Slots of the dense per-chirality s-matrices kept on the device, each
// [2][16][16] in the compute type (zero padded beyond Ls).
enum MatSlot {
    MAT_Q = 0, MAT_QT, MAT_MQMINV, MAT_G5MIT, MAT_G5MIT_MQMINV, MAT_MQG5KT, MAT_G5MT, MAT_HALFMINV,
    MAT_MINV, MAT_M, MAT_MT, MAT_MHALFI, MAT_MHALFKTG5, MAT_IDENT, MAT_CHALF, MAT_SRCLOC, MAT_MIT, NMAT
};
// Slots of the sparse pre-mix coefficient sets, each [d0 | d1 | e0 | e1] x 16.
enum PreSlot { PRE_K = 0, PRE_G5 = 1, NPRE };
constexpr int MAT_ELEMS = 2 * 16 * 16;
constexpr int PRE_ELEMS = 4 * 16;

struct dwf_op {
    dwf_lattice* lat = nullptr;
    int Ls = 0;
    double M0 = 0, m = 0, alpha = 1;
    std::vector<double> b, c;   // b_s, c_s, s = 0..Ls-1 (Sec. 2.2; constant for s-independent (b, c))
    bool any_c() const {
        for (double v : c)
            if (v != 0.0) return true;
        return false;
    }
    dwf::FifthDim fd;
    dwf::DevBuf mats[2];   // compute kind 0: double, 1: float; NMAT * MAT_ELEMS
    dwf::DevBuf pres[2];   // NPRE * PRE_ELEMS
    std::vector<double> mats_host;   // NMAT * MAT_ELEMS, FP64
    // solve workspace kept between solves on this operator (solver.cpp owns
    // the type); solves on one operator run one at a time
    mutable std::shared_ptr<void> solve_ws;
    mutable std::mutex solve_mu;
    dwf::ScratchUser scratch;
    const void* mat(int store_kind, int slot) const {
        const int ck = store_kind == dwf::ST_F64 ? 0 : 1;
        const size_t esz = ck == 0 ? 8 : 4;
        return static_cast<const char*>(mats[ck].p) + (size_t)slot * MAT_ELEMS * esz;
    }
    // one half field of storage kind `kind` (ops.h: complex_bytes_of) as call scratch
    size_t field_bytes(int kind) const { return (size_t)Ls * 12 * lat->Vhp * (kind == 0 ? 16 : (kind == 1 ? 8 : 4)); }
    const void* pre(int store_kind, int slot) const {
        const int ck = store_kind == dwf::ST_F64 ? 0 : 1;
        const size_t esz = ck == 0 ? 8 : 4;
        return static_cast<const char*>(pres[ck].p) + (size_t)slot * PRE_ELEMS * esz;
    }
};

namespace dwf {
// Sites per parity by which entry points limit the size of a field: an odd
// multiple of 32, never less than Vhp.  (Fields were padded to it once; what a
// caller may rely on being refused is not moved with the padding.)
inline long limit_sites(long Vh) {
    const long n = (Vh + 31) / 32;
    return 32 * (n % 2 ? n : n + 1);
}

// Call scratch of an operator: a half field, a two-slice FP64 half field
// (4D sources), and room for reduction partials and scalars.
struct FieldScratch : Scratch {
    FieldScratch(const dwf_op* op, int kind) : Scratch(op->scratch.key(kind), op->field_bytes(kind)) {}
};
struct PairScratch : Scratch {
    explicit PairScratch(const dwf_op* op)
        : Scratch(op->scratch.key(ScratchKey::PAIR), (size_t)2 * 12 * op->lat->Vhp * 16) {}
};
struct SmallScratch : Scratch {
    SmallScratch(const dwf_op* op, size_t bytes) : Scratch(op->scratch.key(ScratchKey::SMALL), bytes) {}
};
}  // namespace dwf
