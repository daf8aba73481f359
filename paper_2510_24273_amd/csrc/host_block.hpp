// Host memory that a blocking call reads back into (host code; the allocator is a parameter, so that a test can refuse).
#pragma once
#include <mutex>
#include <new>

namespace sals {

// A block of BYTES, for one call at a time.  Pinned, as a wait for the device and 8 KB from it take 11 us, into other memory 22; making
// and freeing it takes 25 us and waits for every stream of the process, so up to KEEP blocks, all alike, are kept from call to call.  Where pinned
// memory is refused it is ordinary memory, freed behind the call; p is null if there is neither.
template <typename ALLOC, size_t BYTES, int KEEP> struct HostBlock {
    void* p = nullptr;
    bool idle = false;   // set behind the last wait: no copy into the block is under way
    HostBlock()
    {
        {
            const std::lock_guard<std::mutex> hold(lock());
            for (void*& k : kept())
                if (k) { p = k; k = nullptr; pinned = true; return; }
        }
        p = ALLOC::pin(BYTES);
        pinned = p != nullptr;
        if (!pinned) p = ::operator new(BYTES, std::nothrow);
    }
    ~HostBlock()
    {
        if (!pinned) { ::operator delete(p); return; }
        if (idle) {
            const std::lock_guard<std::mutex> hold(lock());
            for (void*& k : kept())
                if (!k) { k = p; return; }
        }
        ALLOC::unpin(p);
    }
    HostBlock(const HostBlock&) = delete;
    HostBlock& operator=(const HostBlock&) = delete;

private:
    typedef void* Blocks[KEEP];
    static std::mutex& lock() { static std::mutex m; return m; }
    static Blocks& kept() { static Blocks b = {}; return b; }
    bool pinned = false;
};

}  // namespace sals
