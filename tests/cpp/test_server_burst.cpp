// CPU unit test of the kind of launch that the request server gives a request
// (pso_server.hip against the stub HIP runtime and the stand-ins of
// test_server_host.cpp, whose device has 16 places of each on-chip kind).
// Prints "ok" and exits 0 on success.
#define main test_server_host_main
#include "test_server_host.cpp"
#undef main

static int kind_of(pso_server *srv, double at_ms, int64_t N, int D)
{
    set_fake_ms(at_ms);
    static uint64_t seed = 1;
    const pso_desc d = desc_of(seed++, N, D, 3, 0.0f);
    uint64_t t = 0;
    CHECK(pso_server_submit(srv, &d, &t) == PSO_OK);
    std::lock_guard<std::mutex> g(srv->mu);
    return srv->reqs.at(t)->kind;
}

int main()
{
    set_fake_ms(1000.0);
    pso_server *srv = nullptr;
    CHECK(pso_server_create(size_t(1) << 26, 0, &srv) == PSO_OK);
    srv->clock.store(&fake_now);
    set_gate(false); // what is submitted stays in flight
    // the first of a burst by its size, those within 0.05 ms of the last one like it
    CHECK(kind_of(srv, 1001.0, 1000, 10) == REGISTERS);
    CHECK(kind_of(srv, 1001.04, 100, 10) == REGISTERS);
    CHECK(kind_of(srv, 1002.0, 100, 10) == STAGED);
    CHECK(kind_of(srv, 1002.04, 1000, 10) == STAGED);
    // where the requests fill the device, by size again
    CHECK(kind_of(srv, 1002.05, 1000, 10) == REGISTERS);
    CHECK(kind_of(srv, 1002.06, 100, 10) == REGISTERS);
    // a streamed request (too wide) starts no burst of its kind
    CHECK(kind_of(srv, 1003.0, 100, 100) == STREAMED);
    CHECK(kind_of(srv, 1003.01, 1000, 10) == REGISTERS);
    set_gate(true);
    CHECK(pso_server_destroy(srv) == PSO_OK);
    std::printf("ok\n");
    return 0;
}
