// Idle call scratch (ScratchKey, Scratch in dwf_internal.h).
#include <algorithm>
#include <new>
#include <utility>

#include "dwf_internal.h"

namespace dwf {

namespace {
struct Idle {
    ScratchKey key;
    DevBuf buf;
};
struct Pool {
    std::mutex mu;
    std::vector<Idle> idle;   // oldest first
    size_t bytes = 0;         // of idle
    std::vector<std::pair<ScratchKey, int>> users;   // operators by shape (class 0)
    int* users_of(ScratchKey key) {
        key.cls = 0;
        for (auto& u : users)
            if (u.first == key) return &u.second;
        return nullptr;
    }
};
// never destroyed, so that an operator destroyed at process exit still finds it
Pool& pool() {
    static Pool* p = new Pool;
    return *p;
}

// Moves the idle buffers that `drop` accepts, oldest first, to `out` (to be
// freed without the lock); nothing is moved if memory for that is missing.
template <class F> void take_out(Pool& p, std::vector<DevBuf>& out, F drop) {
    out.reserve(p.idle.size());
    for (Idle& i : p.idle)
        if (drop(i)) {
            p.bytes -= i.buf.bytes;
            out.push_back(std::move(i.buf));
        }
    p.idle.erase(std::remove_if(p.idle.begin(), p.idle.end(), [](const Idle& i) { return !i.buf.p; }), p.idle.end());
}
}  // namespace

DevBuf scratch_take(const ScratchKey& key, size_t bytes) {
    {
        Pool& p = pool();
        std::lock_guard<std::mutex> lock(p.mu);
        // the one idle longest: a call's first kernel then writes what its last ones
        // used (FP64 5D operator on 6x10x6x14, Ls = 10: 54.1 us, with the newest 57.1)
        for (size_t k = 0; k < p.idle.size(); ++k)
            if (p.idle[k].key == key && p.idle[k].buf.bytes == bytes) {
                DevBuf b = std::move(p.idle[k].buf);
                p.idle.erase(p.idle.begin() + (long)k);
                p.bytes -= bytes;
                return b;
            }
    }
    return DevBuf(bytes);
}

void scratch_give(const ScratchKey& key, DevBuf&& b) noexcept {
    DevBuf mine(std::move(b));   // freed here unless it is kept
    std::vector<DevBuf> out;
    try {
        Pool& p = pool();
        std::lock_guard<std::mutex> lock(p.mu);
        if (mine.bytes > SCRATCH_IDLE_MAX || !p.users_of(key)) return;
        size_t over = p.bytes + mine.bytes > SCRATCH_IDLE_MAX ? p.bytes + mine.bytes - SCRATCH_IDLE_MAX : 0;
        p.idle.reserve(p.idle.size() + 1);
        if (over)
            take_out(p, out, [&](const Idle& i) {
                if (!over) return false;
                over -= std::min(over, i.buf.bytes);
                return true;
            });
        p.bytes += mine.bytes;
        p.idle.push_back({key, std::move(mine)});
    } catch (const std::bad_alloc&) {
    }
}

bool release_scratch() {
    std::vector<Idle> out;
    Pool& p = pool();
    std::lock_guard<std::mutex> lock(p.mu);
    out.swap(p.idle);
    p.bytes = 0;
    return !out.empty();
}

void ScratchUser::attach(int Ls, long Vh) {
    ScratchKey shape{0, 0, Ls, Vh};
    DWF_HIP(hipGetDevice(&shape.dev));
    Pool& p = pool();
    std::lock_guard<std::mutex> lock(p.mu);
    if (int* n = p.users_of(shape)) ++*n;
    else p.users.push_back({shape, 1});
    shape_ = shape;
}

ScratchUser::~ScratchUser() {
    if (!shape_.Ls) return;   // not attached
    std::vector<DevBuf> out;
    Pool& p = pool();
    std::lock_guard<std::mutex> lock(p.mu);
    if (--*p.users_of(shape_) > 0) return;
    p.users.erase(std::find_if(p.users.begin(), p.users.end(), [](const auto& u) { return u.second == 0; }));
    try {
        take_out(p, out, [&](const Idle& i) { return i.key.dev == shape_.dev && i.key.Ls == shape_.Ls && i.key.Vh == shape_.Vh; });
    } catch (const std::bad_alloc&) {   // they stay within the bound, and go first
    }
}

}  // namespace dwf
