// A fork of a stream: launches on a second stream that follow what the first one holds when they are made and that the first one waits
// for at close(), or where the fork goes out of scope, so that to the caller all of it is work on the first stream.
#pragma once

namespace agzo {

// Api: stream_t, event_t, error_t (0: success), record(event, stream), wait(stream, event), synchronize(stream)
template <typename Api>
class Fork {
  public:
    typedef typename Api::stream_t stream_t;
    typedef typename Api::event_t event_t;
    typedef typename Api::error_t error_t;

    Fork(stream_t main, stream_t side, event_t fork, event_t join) : main_(main), side_(side), fork_(fork), join_(join) {}
    Fork(const Fork&) = delete;
    Fork& operator=(const Fork&) = delete;
    ~Fork() { (void)close(); }

    // once per fork
    template <typename F>
    error_t run(F launches) {
        error_t e = Api::record(fork_, main_);
        if (e == error_t(0)) e = Api::wait(side_, fork_);
        if (e != error_t(0)) return e;
        open_ = true;            // whatever follows, also an exception: something may be under way on the second stream
        return launches(side_);
    }
    // Where the first stream cannot be made to wait, the host does (an event that was not recorded stands for an older fork).  Still
    // open behind a close() that failed at that too: another one tries again
    error_t close() {
        if (!open_) return error_t(0);
        error_t e = Api::record(join_, side_);
        if (e == error_t(0)) e = Api::wait(main_, join_);
        if (e != error_t(0) && Api::synchronize(side_) != error_t(0)) return e;
        open_ = false;
        return e;
    }
    bool open() const { return open_; }

  private:
    stream_t main_, side_;
    event_t fork_, join_;
    bool open_ = false;
};

}  // namespace agzo
