// devbuf.h -- device buffers of a context, and how long they live.
//
// A launch that a stream capture records holds the addresses of the buffers it
// read, and its replays come at any time.  So a buffer that a recording holds
// is never freed and its tables are never written again while the context
// lives: where a later run needs a larger one, or a load other tables, it is
// put aside and a new one allocated.
#pragma once
#include <stddef.h>

#include <vector>

namespace soft {

template <typename T> struct DevBuf {
    T *p = nullptr;
    size_t n = 0;           // elements allocated
    bool recorded = false;  // a captured launch holds its address
};

// Mem: `static int alloc(void **p, size_t bytes)` and `static int free(void *p)`,
// 0 on success.
template <typename Mem> class Buffers {
  public:
    // At least n elements; the contents are kept only if the buffer is.
    template <typename T> int ensure(DevBuf<T> &b, size_t n) {
        if (n == 0) n = 1;
        if (b.n >= n) return 0;
        if (int e = drop(b)) return e;
        void *p = nullptr;
        if (int e = Mem::alloc(&p, n * sizeof(T))) return e;
        b.p = static_cast<T *>(p);
        b.n = n;
        return 0;
    }
    // The same, for contents that are about to be replaced.
    template <typename T> int renew(DevBuf<T> &b, size_t n) {
        if (b.recorded)
            if (int e = drop(b)) return e;
        return ensure(b, n);
    }
    // Give the buffer up: freed, or put aside if a recording holds it.
    template <typename T> int drop(DevBuf<T> &b) {
        int e = 0;
        if (b.p && b.recorded) aside_.push_back(b.p);
        else if (b.p) e = Mem::free(b.p);
        if (!e) b = DevBuf<T>();
        return e;
    }
    // Free a buffer, and at the end those put aside: no replay comes any more.
    template <typename T> void release(DevBuf<T> &b) {
        if (b.p) (void)Mem::free(b.p);
        b = DevBuf<T>();
    }
    void release_aside() {
        for (void *p : aside_) (void)Mem::free(p);
        aside_.clear();
    }

  private:
    std::vector<void *> aside_;
};

}  // namespace soft
