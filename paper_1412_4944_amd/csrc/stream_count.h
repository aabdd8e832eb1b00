// How many streams of a GPU carry live contexts of one kind (host code without HIP).  Streams of different
// devices are different streams, also where their handles are equal (the null stream).
#pragma once

#include <algorithm>
#include <mutex>
#include <vector>

namespace sbo {

class StreamCount {
public:
    void add(int device, const void* stream) {
        std::lock_guard<std::mutex> lock(mutex_);
        live_.push_back({device, stream});
    }
    void remove(int device, const void* stream) {
        std::lock_guard<std::mutex> lock(mutex_);
        auto it = std::find(live_.begin(), live_.end(), Entry{device, stream});
        if (it != live_.end()) live_.erase(it);
    }
    int streams(int device) {
        std::lock_guard<std::mutex> lock(mutex_);
        int n = 0;
        for (size_t i = 0; i < live_.size(); ++i)
            n += live_[i].device == device && std::find(live_.begin(), live_.begin() + i, live_[i]) == live_.begin() + i;
        return n;
    }

private:
    struct Entry {
        int device;
        const void* stream;
        bool operator==(const Entry& o) const { return device == o.device && stream == o.stream; }
    };
    std::mutex mutex_;
    std::vector<Entry> live_;
};

}  // namespace sbo
