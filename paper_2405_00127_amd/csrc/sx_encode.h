// Host path encoder (Section 8.2).
#pragma once
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

#include <new>
#include <string>
#include <vector>

#include "strokex.h"

namespace sx {

// Where a Buf's memory comes from (the library puts small scenes' streams in
// pinned memory, which the GPU reads by itself).
struct HostAlloc {
    void* (*get)(size_t);
    void (*put)(void*);
};
// A growing array of plain values.  Unlike a vector's, its memory is not
// zeroed before it is written.
template <class T>
class Buf {
   public:
    explicit Buf(HostAlloc a = {malloc, free}) : a_(a) {}
    Buf(const Buf&) = delete;
    Buf& operator=(const Buf&) = delete;
    ~Buf() { reset(); }
    T* data() { return p_; }
    const T* data() const { return p_; }
    size_t size() const { return n_; }
    size_t capacity() const { return cap_; }
    bool empty() const { return n_ == 0; }
    T& operator[](size_t i) { return p_[i]; }
    const T& operator[](size_t i) const { return p_[i]; }
    T& back() { return p_[n_ - 1]; }
    void clear() { n_ = 0; }
    void reset() {
        if (p_) a_.put(p_);
        p_ = nullptr;
        n_ = cap_ = 0;
    }
    // room for `more` values past the size, which put() then needs no check for
    void room(size_t more) {
        if (n_ + more <= cap_) return;
        const size_t cap = n_ + more + cap_ / 2;
        T* q = static_cast<T*>(a_.get(cap * sizeof(T)));
        if (!q) throw std::bad_alloc();
        if (n_) memcpy(q, p_, n_ * sizeof(T));
        if (p_) a_.put(p_);
        p_ = q;
        cap_ = cap;
    }
    void put(T v) { p_[n_++] = v; }
    // the next `n` values are written at end() by the caller
    T* end() { return p_ + n_; }
    void add(size_t n) { n_ += n; }

   private:
    HostAlloc a_;
    T* p_ = nullptr;
    size_t n_ = 0, cap_ = 0;
};

struct HostEncoding {
    explicit HostEncoding(HostAlloc a = {malloc, free}) : tags(a), data(a) {}
    Buf<uint8_t> tags;
    Buf<float> data;                     // x, y pairs
    std::vector<uint32_t> style_stream;  // caller style index per style entry
    std::vector<uint32_t> xform_stream;  // caller transform index per transform entry
    std::vector<uint32_t> path_map;      // encoded path -> input path
    void clear() {
        tags.clear();
        data.clear();
        style_stream.clear();
        xform_stream.clear();
        path_map.clear();
    }
};

// Replaces the contents of `out` (its memory is reused).
// styles: the caller's style table (n_styles entries); a path whose style
// has SX_STYLE_FILL gets every subpath closed.
bool encode_paths(const sx_paths& in, const sx_style* styles, uint32_t n_styles, uint32_t n_xforms,
                  HostEncoding& out, std::string& err);

}  // namespace sx
