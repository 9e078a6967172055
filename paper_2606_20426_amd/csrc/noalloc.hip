// Extraction that allocates nothing: the variant of tc_extract for callers
// that cannot allocate device memory (code under stream capture, tight
// serving loops, harnesses that forbid it).  Its launch descriptor, step
// state, indenter poses, tile lists and partial sums live in one file-scope
// device array of fixed size instead of the context's step scratch, plan and
// state pool; the kernels are the ones tc_extract launches.
#include <cstring>
#include <mutex>

#include "runtime.h"

namespace tc {
namespace {

constexpr size_t NOALLOC_BYTES = size_t(4) << 20;   // TC_NOALLOC_SCRATCH_BYTES
constexpr int MAX_DEVICES = 64;
static_assert(NOALLOC_BYTES == TC_NOALLOC_SCRATCH_BYTES, "header and library agree on the size");

// One copy per device.  Host code never passes this name to a kernel or a
// copy: it takes the device address from hipGetSymbolAddress below.
static __device__ __align__(256) unsigned char scratch[NOALLOC_BYTES];

std::mutex g_mu;
void* g_ptr[MAX_DEVICES] = {};

size_t up256(size_t b) { return (b + 255) & ~size_t(255); }
int cdiv(int64_t a, int64_t b) { return (int)((a + b - 1) / b); }

// Everything the call's kernels read, passed by value: the descriptor, state
// and poses go to the scratch array, and the three tile lists {pad 0, tile i} of
// n[c] tiles are written behind one another.  One launch (2.3 us of the host)
// instead of three copies from unpinned memory (4 us each) and three fills.
struct NoallocArgs {
  EnvDesc desc;
  EnvState state;
  EnvPose pose;
  int n[3];
};
static_assert(sizeof(NoallocArgs) <= 4000 && sizeof(EnvDesc) % 4 == 0 && sizeof(EnvState) % 4 == 0 &&
              sizeof(EnvPose) % 4 == 0, "kernel argument limit");

__global__ void k_noalloc_setup(NoallocArgs a, uint32_t* desc, uint32_t* state, uint32_t* pose, Tile* tiles) {
  if (blockIdx.x == 0) {
    auto put = [](uint32_t* to, const void* from, int words) {
      for (int i = threadIdx.x; i < words; i += blockDim.x) to[i] = static_cast<const uint32_t*>(from)[i];
    };
    put(desc, &a.desc, sizeof a.desc / 4);
    put(state, &a.state, sizeof a.state / 4);
    put(pose, &a.pose, sizeof a.pose / 4);
  }
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < a.n[0] + a.n[1] + a.n[2])
    tiles[i] = Tile{0, i < a.n[0] ? i : i < a.n[0] + a.n[1] ? i - a.n[0] : i - a.n[0] - a.n[1]};
}

}  // namespace

// Device address of this device's scratch array, looked up once per device
// with that device current (context creation).
tc_status noalloc_init(int device) {
  if (device < 0 || device >= MAX_DEVICES) return set_error(TC_E_INVALID_ARG, "device ordinal beyond 63");
  std::lock_guard<std::mutex> lk(g_mu);
  if (g_ptr[device]) return TC_OK;
  void* p = nullptr;
  const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
  if (e != hipSuccess) return hip_fail(e, "hipGetSymbolAddress(no-alloc scratch)");
  if (!p) return set_error(TC_E_HIP, "no-alloc scratch has no device address");
  g_ptr[device] = p;
  return TC_OK;
}

}  // namespace tc

using namespace tc;

tc_status tc_extract_noalloc(tc_pad* pad, int32_t n_ind, const tc_indenter* ind, double* reaction) {
  if (!pad) return set_error(TC_E_INVALID_ARG, "pad is null");
  tc_context* ctx = pad->ctx;
  std::string err;
  tc_status s = validate_indenters(n_ind, ind, err);
  if (s) return set_error(s, err);
  if ((s = check_meshes(ctx, n_ind, ind))) return s;
  if (pad->busy.load()) return set_error(TC_E_BUSY, "pad has a request in flight on a server");
  std::lock_guard<std::recursive_mutex> lk(ctx->mu);
  TC_HIP(hipSetDevice(ctx->device));
  char* base;
  {
    std::lock_guard<std::mutex> g(g_mu);
    base = ctx->device < MAX_DEVICES ? static_cast<char*>(g_ptr[ctx->device]) : nullptr;
  }
  if (!base) return set_error(TC_E_HIP, "no-alloc scratch not initialised on this device");
  // layout: descriptor, state, poses, tiles (tet, surface, contact vertex),
  // contact and traction partial sums
  const int n_tt = cdiv(pad->T, ctx->el_block);
  const int n_st = cdiv(pad->S, ctx->cg_block);
  const int n_ct = pad->C > 0 ? cdiv(pad->C, ctx->cg_block) : 0;
  size_t off = 0;
  auto take = [&](size_t b) { const size_t o = off; off += up256(b); return o; };
  const size_t o_desc = take(sizeof(EnvDesc));
  const size_t o_state = take(sizeof(EnvState));
  const size_t o_pose = take(sizeof(EnvPose));
  const size_t o_tiles = take(sizeof(Tile) * ((size_t)n_tt + n_st + n_ct));
  const size_t o_c3 = take(24 * (size_t)std::max(n_ct, 1));
  const size_t o_s3 = take(24 * (size_t)std::max(n_st, 1));
  if (off > NOALLOC_BYTES)
    return set_error(TC_E_INVALID_ARG, "pad needs " + std::to_string(off) + " bytes of no-alloc scratch, more than " +
                                           std::to_string(NOALLOC_BYTES));
  NoallocArgs args;
  EnvDesc& E = args.desc;
  E = pad->desc;
  E.n_tt = n_tt;
  E.n_st = n_st;
  E.n_ct = n_ct;
  E.part_c3 = reinterpret_cast<double*>(base + o_c3);
  E.part_s3 = reinterpret_cast<double*>(base + o_s3);
  E.st = reinterpret_cast<EnvState*>(base + o_state);
  E.pose = reinterpret_cast<const EnvPose*>(base + o_pose);
  EnvPose& Q = args.pose;
  init_state(args.state, Q, 1, n_ind, ind, pad);
  if (Q.pairs)
    return set_error(TC_E_INVALID_ARG,
                     "vertex-face / edge-edge pairs (mesh_contact 2 with a mesh indenter) need the pad's step "
                     "scratch: use tc_extract");
  hipStream_t st = ctx->stream;
  Tile* tiles = reinterpret_cast<Tile*>(base + o_tiles);
  Tile* t_tet = tiles;
  Tile* t_surf = tiles + n_tt;
  Tile* t_cand = tiles + n_tt + n_st;
  args.n[0] = n_tt;
  args.n[1] = n_st;
  args.n[2] = n_ct;
  hipLaunchKernelGGL(k_noalloc_setup, dim3(cdiv((int64_t)n_tt + n_st + n_ct, 256)), dim3(256), 0, st, args,
                     reinterpret_cast<uint32_t*>(base + o_desc), reinterpret_cast<uint32_t*>(base + o_state),
                     reinterpret_cast<uint32_t*>(base + o_pose), tiles);
  const EnvDesc* d_desc = reinterpret_cast<const EnvDesc*>(base + o_desc);
  auto go = [&](KernelId k, const Tile* t, int nt, int block) {
    LaunchArgs a;
    a.envs = d_desc;
    a.n_env = 1;
    a.stream = st;
    a.tiles = t;
    a.ntiles = nt;
    a.block = block;
    return launch_kernel(k, pad->fp64, a);
  };
  (void)go(KernelId::sigma, t_tet, n_tt, ctx->el_block);
  (void)go(KernelId::traction, t_surf, n_st, ctx->cg_block);
  (void)go(KernelId::contact, t_cand, n_ct, ctx->cg_block);
  (void)go(KernelId::env_extract, nullptr, 0, 256);
  TC_HIP(hipGetLastError());
  if ((s = ctx->sig.publish(base + o_state, ctx->sig.buf(), sizeof(EnvState), st))) return s;
  EnvState S;
  std::memcpy(&S, ctx->sig.buf(), sizeof S);
  if (S.status != TC_OK) return set_error(S.status, "extraction failed");
  if (reaction)
    for (int c = 0; c < 3; ++c) reaction[c] = S.reaction[c];
  return TC_OK;
}
