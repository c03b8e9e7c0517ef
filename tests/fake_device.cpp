// The host side of libdn on a device that does not exist: this program defines the HIP runtime functions that the library calls,
// with as many compute units as the first argument says, so that the choice of kernels can be tested without a GPU.  Device
// memory is host memory; launched kernels do nothing but leave their name and grid in the log.
//
//   fake_device UNITS COMMAND...
//     net:784-128-10:ce:1     a net (widths; ce: softmax and cross-entropy, mse: sigmoid and squared error; largest batch), tanh
//                             below the last layer
//     option:online_mode=2
//     train:96:1:0.9          one epoch: samples, batch, momentum
//     forward:64              rows
//     convback:128:32:32:32:64:3:1:1   dn_conv_backward: batch, channels, height, width, output channels, filter edge, stride, padding
// One line per command: its status, the schedule of the last epoch and its kernel, and the launches it made (name/workgroups/template arguments/what
// fake_plans.cpp reads in the kernel's parameters).
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

#include <cxxabi.h>
#include <unistd.h>

#include "dn.h"

std::string plan_of(const std::string &kernel, void **parameters);   // fake_plans.cpp

namespace {

int units = 0;
std::string launches;
struct Dim3 { uint32_t x, y, z; };
struct Call { Dim3 grid, block; size_t shared; void *stream; } call;
char somewhere[4096];

std::map<const void *, std::string> &names()   // (the library registers its kernels before this file's objects exist)
{
    static std::map<const void *, std::string> m;
    return m;
}

int log_launch(const void *f, Dim3 grid, void **parameters)
{
    int status;
    char *full = abi::__cxa_demangle(names()[f].c_str(), nullptr, nullptr, &status);
    std::string name = full ? full : names()[f];
    free(full);
    const size_t end = name.find("_kernel"), begin = name.find_last_of(": ", end);   // without namespaces, template arguments and parameters
    std::string arguments = end == std::string::npos ? "" : name.substr(end + 7, name.rfind('(') - end - 7);
    name = end == std::string::npos ? name : name.substr(begin + 1, end + 7 - begin - 1);
    launches += " " + name + "/" + std::to_string(grid.x * grid.y * grid.z) + "/";
    for (char c : arguments)
        if (c != ' ') launches += c;
    launches += "/" + plan_of(name, parameters);
    return 0;
}

std::vector<std::string> split(const std::string &text, char by)
{
    std::vector<std::string> parts(1);
    for (char c : text) {
        if (c == by) parts.emplace_back();
        else parts.back() += c;
    }
    return parts;
}

}  // namespace

extern "C" {

void **__hipRegisterFatBinary(const void *) { static void *module; return &module; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *f, char *, const char *name, unsigned, void *, void *, void *, void *, int *) { names()[f] = name; }
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t shared, void *stream) { call = Call{grid, block, shared, stream}; return 0; }
int __hipPopCallConfiguration(Dim3 *grid, Dim3 *block, size_t *shared, void **stream)
{
    *grid = call.grid; *block = call.block; *shared = call.shared; *stream = call.stream;
    return 0;
}
int hipLaunchKernel(const void *f, Dim3 grid, Dim3, void **parameters, size_t, void *) { return log_launch(f, grid, parameters); }
int hipExtLaunchKernel(const void *f, Dim3 grid, Dim3, void **parameters, size_t, void *, void *, void *, int) { return log_launch(f, grid, parameters); }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int, size_t) { *n = 1; return 0; }
int hipFuncSetAttribute(const void *, int, int) { return 0; }
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipDeviceGetAttribute(int *v, int, int) { *v = units; return 0; }
int hipGetLastError() { return 0; }
int hipGetSymbolAddress(void **p, const void *) { *p = somewhere; return 0; }
int hipHostMalloc(void **p, size_t n, unsigned) { *p = calloc(1, n); return 0; }
int hipThreadExchangeStreamCaptureMode(int *) { return 0; }
int hipEventCreate(void **e) { *e = somewhere; return 0; }
int hipEventDestroy(void *) { return 0; }
int hipEventRecord(void *, void *) { return 0; }
int hipEventElapsedTime(float *ms, void *, void *) { *ms = 0.f; return 0; }
int hipStreamSynchronize(void *) { return 0; }
int hipMemset(void *p, int v, size_t n) { memset(p, v, n); return 0; }
int hipMemsetAsync(void *p, int v, size_t n, void *) { memset(p, v, n); return 0; }
int hipMemcpy(void *to, const void *from, size_t n, int) { memcpy(to, from, n); return 0; }
int hipMemcpyAsync(void *to, const void *from, size_t n, int, void *) { memcpy(to, from, n); return 0; }

}  // extern "C"

int main(int argc, char **argv)
{
    if (argc < 3) return 2;
    units = atoi(argv[1]);
    dn_net *net = nullptr;
    const float *X = (const float *)somewhere;   // nothing reads the samples
    for (int i = 2; i < argc; ++i) {
        launches.clear();
        const std::vector<std::string> c = split(argv[i], ':');
        int status = -1;
        if (c[0] == "net") {
            std::vector<int32_t> widths;
            for (const std::string &w : split(c[1], '-')) widths.push_back(atoi(w.c_str()));
            const bool ce = c[2] == "ce";
            std::vector<dn_act> acts(widths.size() - 1, DN_ACT_TANH);
            acts.back() = ce ? DN_ACT_SOFTMAX : DN_ACT_SIGMOID;
            const size_t bytes = dn_net_arena_bytes(widths.data(), (int32_t)widths.size(), atoi(c[3].c_str()));
            void *arena = bytes ? aligned_alloc(256, bytes) : nullptr;
            if (net) dn_net_destroy(net);
            net = nullptr;
            status = dn_net_create(widths.data(), (int32_t)widths.size(), acts.data(), ce ? DN_LOSS_CROSS_ENTROPY : DN_LOSS_MSE,
                                   atoi(c[3].c_str()), arena, bytes, nullptr, &net);
        } else if (c[0] == "option") {
            const std::vector<std::string> o = split(c[1], '=');
            status = dn_set_option(net, o[0].c_str(), atoi(o[1].c_str()));
        } else if (c[0] == "train") {
            float loss;
            status = dn_train_epoch(net, X, (const int32_t *)X, atoi(c[1].c_str()), atoi(c[2].c_str()), 0.01f, (float)atof(c[3].c_str()), &loss);
        } else if (c[0] == "forward") {
            status = dn_forward(net, X, atoi(c[1].c_str()), (float *)somewhere);
        } else if (c[0] == "convback") {
            int32_t v[8];
            for (int k = 0; k < 8; ++k) v[k] = atoi(c[k + 1].c_str());
            const size_t bytes = dn_conv_backward_workspace_bytes(v[0], v[1], v[2], v[3], v[4], v[5], v[5], v[6], v[7]);
            float *Y = (float *)somewhere;
            status = dn_conv_backward(X, X, Y, Y, Y, nullptr, Y, Y, somewhere, bytes, v[0], v[1], v[2], v[3], v[4], v[5], v[5], v[6], v[7], DN_ACT_TANH, nullptr);
        }
        int32_t schedule = -1;
        const char *kernel = "";
        if (net) dn_last_schedule(net, &schedule);
        if (net) dn_last_kernel(net, &kernel);
        printf("%d %d=%s%s\n", status, schedule, kernel, launches.c_str());
        fflush(stdout);
    }
    _exit(0);
}
