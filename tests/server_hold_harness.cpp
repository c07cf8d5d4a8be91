// Host harness for the scheduler's waiting rule (Core::hold in
// paper_2607_06731_amd/csrc/server_core.h), built by tests/test_server_hold.py.
//
// TEST INFRASTRUCTURE.  A simulated device on a fake clock, whose launches take
// what the scenario says; the scheduler is stepped every 10 us.  Prints one line
// per scenario: its name and, per request, the launch it went into and the time it
// waited for that launch (us).
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <map>
#include <string>
#include <vector>

#include "server_core.h"

using namespace gpsrv;

struct MockDev {
    double now = 0.0, launch_ms = 1.0;
    int64_t launches = 0;
    std::vector<double> done;
    std::map<int64_t, std::pair<int64_t, double>> launched;     // ticket -> (launch, time)
    double now_ms() const { return now; }
    int upload(Request& R)
    {
        R.upload = &R;
        return 0;
    }
    void release_upload(Request&) {}
    size_t workspace_bytes(int64_t, int64_t, int32_t, int32_t, int32_t, int64_t) const { return 4096; }
    int launch(int si, const Batch& B)
    {
        for (const Entry& e : B.ent)
            if (!launched.count(e.R->ticket)) launched[e.R->ticket] = {launches, now};
        done[(size_t)si] = now + launch_ms;
        ++launches;
        return 0;
    }
    int poll(int si) { return now >= done[(size_t)si] ? 1 : 0; }
    void deliver(Request&) {}
};

struct Sim {
    MockDev dev;
    Core<MockDev> core;
    std::vector<std::vector<uint32_t>> nodes;
    std::vector<std::vector<int64_t>> offsets;
    std::vector<std::vector<double>> out;
    std::map<int64_t, double> submitted;
    static Config config(bool one_each)
    {
        Config c;
        c.ws_cap = size_t(1) << 30;
        c.one_launch_per_request = one_each;
        return c;
    }
    explicit Sim(bool one_each = false) : core(dev, config(one_each), size_t(1) << 30, size_t(1) << 30)
    {
        dev.done.assign(core.slots.size(), 0.0);
        for (int64_t n : {1000ll, 1ll << 20}) {
            Dataset D;
            D.live = true;
            D.n_vars = 1;
            D.n_cases = n;
            core.datasets.push_back(D);
        }
    }
    void submit(int ds, int64_t programs, int64_t len)
    {
        offsets.emplace_back();
        for (int64_t p = 0; p <= programs; ++p) offsets.back().push_back(p * len);
        nodes.emplace_back((size_t)(programs * len), 0u);
        out.emplace_back((size_t)programs, 0.0);
        auto R = std::make_shared<Request>();
        R->nodes = nodes.back().data();
        R->n_nodes = (int64_t)nodes.back().size();
        R->offsets = offsets.back().data();
        R->P = programs;
        R->out_f = out.back().data();
        R->ds = ds;
        int64_t t = 0;
        if (core.submit(R, &t) == 0) submitted[t] = dev.now;
    }
    void run(double ms)
    {
        for (const double end = dev.now + ms; dev.now < end; dev.now += 0.01)
            while (core.step()) {}
    }
    void print(const char* name)
    {
        std::printf("%s", name);
        for (const auto& kv : submitted) {
            const auto it = dev.launched.find(kv.first);
            if (it == dev.launched.end()) std::printf(" none");
            else std::printf(" %lld:%.0f", (long long)it->second.first, (it->second.second - kv.second) * 1e3);
        }
        std::printf("\n");
    }
};

int main()
{
    {
        // a launch of few node evaluations that takes long; a small request after it
        Sim s;
        s.dev.launch_ms = 10.0;
        s.submit(1, 8, 128);
        s.run(0.05);
        s.submit(0, 50, 30);
        s.run(2.0);
        s.print("long_launch");
    }
    {
        // small launches: requests that arrive meanwhile share the next one
        Sim s;
        s.dev.launch_ms = 0.1;
        s.submit(0, 50, 30);
        s.run(0.02);
        for (int k = 0; k < 4; ++k) {
            s.submit(0, 50, 30);
            s.run(0.01);
        }
        s.run(1.0);
        s.print("small_launches");
    }
    {
        // more work than the limit waits for nothing
        Sim s;
        s.dev.launch_ms = 10.0;
        s.submit(0, 50, 30);
        s.run(0.05);
        s.submit(1, 100, 64);
        s.run(1.0);
        s.print("large_request");
    }
    {
        Sim s(true);
        s.dev.launch_ms = 0.1;
        for (int k = 0; k < 3; ++k) s.submit(0, 50, 30);
        s.run(2.0);
        s.print("one_each");
    }
    return 0;
}
