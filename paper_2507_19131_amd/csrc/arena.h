// Device memory of one handle: everything it keeps is gathered on the host while the handle is built and goes to the
// device as ONE allocation with ONE copy.  (Forty small allocations cost more to make, and lie on pages of their own: the
// kernels of a wide block walk through all of them.)
#pragma once
#include <hip/hip_runtime.h>

#include <cstring>
#include <utility>
#include <vector>

namespace mixaq {

class Arena {
public:
    // copies `data`; *field becomes its device address in commit()
    template <typename T, typename F>
    void add(const std::vector<T>& data, F** field)
    {
        const size_t at = (host_.size() + 255) & ~(size_t)255, bytes = data.size() * sizeof(T);
        host_.resize(at + (bytes ? bytes : 16));
        if (bytes) memcpy(host_.data() + at, data.data(), bytes);
        fields_.emplace_back((void*)field, at);
    }
    hipError_t commit()
    {
        hipError_t e = hipMalloc(&dev_, host_.size() + 256);
        if (e == hipSuccess) e = hipMemcpy(dev_, host_.data(), host_.size(), hipMemcpyHostToDevice);
        if (e != hipSuccess) return e;
        for (auto& f : fields_) {
            void* p = (char*)dev_ + f.second;
            memcpy(f.first, &p, sizeof(p));
        }
        host_ = {};
        fields_ = {};
        return hipSuccess;
    }
    void release()
    {
        if (dev_) (void)hipFree(dev_);
        dev_ = nullptr;
    }

private:
    std::vector<char> host_;
    std::vector<std::pair<void*, size_t>> fields_;
    void* dev_ = nullptr;
};

}  // namespace mixaq
