// Compute units of one XCD as the scenes of this process share them.
//
// The blocks of a colouring, and those of a cluster of a solve, wait for each
// other, so all of them must be on the chip at once; a block takes a CU (its
// LDS or its threads fill one).  Two launches that dispatch together and do not
// fit side by side could each hold a part of the CUs and wait for the rest.  So
// a step enters with the CUs per XCD that its waiting blocks take and leaves
// when the GPU has finished it: steps that fit run together, the others one
// after the other, in the order in which they came (a large one is not kept
// out by small ones).  Blocks that wait for no other block need no place here:
// they end, and their CUs become free.  Host waits only.
#pragma once
#include <condition_variable>
#include <cstdint>
#include <mutex>

namespace trk {

class CuGate {
public:
    // waits until need of the capacity's units are free, and takes them
    void enter(int need, int capacity)
    {
        std::unique_lock<std::mutex> lock(m_);
        const uint64_t mine = next_++;
        cv_.wait(lock, [&] { return mine == serving_ && (used_ == 0 || used_ + need <= capacity); });
        used_ += need;
        ++serving_;
        cv_.notify_all();
    }
    void leave(int need)
    {
        std::lock_guard<std::mutex> lock(m_);
        used_ -= need;
        cv_.notify_all();
    }

private:
    std::mutex m_;
    std::condition_variable cv_;
    uint64_t next_ = 0, serving_ = 0;
    int used_ = 0;
};

}  // namespace trk
