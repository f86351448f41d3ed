// Device memory of one handle: everything it keeps is gathered on the host while the handle is built and goes to the
// device as ONE allocation with ONE copy.
#pragma once
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <memory>
#include <utility>
#include <vector>

namespace mixaq {

class Arena {
public:
    void reserve(size_t bytes) { grow(bytes); }
    // room for n values, to be filled before the next call; *field becomes its device address in commit()
    template <typename T, typename F>
    T* take(size_t n, F** field)
    {
        const size_t at = (used_ + 255) & ~(size_t)255, bytes = std::max<size_t>(n * sizeof(T), 16);
        if (at + bytes > cap_) grow(std::max(2 * cap_, at + bytes));
        used_ = at + bytes;
        fields_.emplace_back((void*)field, at);
        return (T*)(host_.get() + at);
    }
    template <typename T, typename F>
    void add(const std::vector<T>& data, F** field)
    {
        T* p = take<T>(data.size(), field);
        if (!data.empty()) memcpy(p, data.data(), data.size() * sizeof(T));
    }
    hipError_t commit()
    {
        hipError_t e = hipMalloc(&dev_, used_ + 256);
        if (e == hipSuccess) e = hipMemcpy(dev_, host_.get(), used_, hipMemcpyHostToDevice);
        if (e != hipSuccess) return e;
        for (auto& f : fields_) {
            void* p = (char*)dev_ + f.second;
            memcpy(f.first, &p, sizeof(p));
        }
        host_.reset();
        fields_ = {};
        return hipSuccess;
    }
    void release()
    {
        if (dev_) (void)hipFree(dev_);
        dev_ = nullptr;
    }

private:
    void grow(size_t cap)
    {
        if (cap <= cap_) return;
        std::unique_ptr<char[]> h(new char[cap]);
        if (used_) memcpy(h.get(), host_.get(), used_);
        host_ = std::move(h);
        cap_ = cap;
    }
    std::unique_ptr<char[]> host_;
    size_t used_ = 0, cap_ = 0;
    std::vector<std::pair<void*, size_t>> fields_;
    void* dev_ = nullptr;
};

}  // namespace mixaq
