// Host run of the client's two loops (csrc/host_keys.cpp, included whole to reach its internals): every instruction set
// that this processor has against a plain loop, at dimensions around the vector widths; the sharing out over
// threads; and whole calls on counts that use several threads against samples formed one by one.
#include <cstdio>
#include <cstdlib>

#include "../../paper_1806_03461_amd/csrc/host_keys.cpp"

#define CHECK(cond) do { if (!(cond)) { std::fprintf(stderr, "%s:%d: %s\n", __FILE__, __LINE__, #cond); std::exit(1); } } while (0)

namespace {

struct Variant { const char *name; FillFn fill; DotFn dot; };

std::vector<Variant> variants() {
    std::vector<Variant> v{{"base", fill_base, dot_base}};
#if defined(__x86_64__)
    __builtin_cpu_init();
    if (__builtin_cpu_supports("avx2")) v.push_back({"avx2", fill_avx2, dot_avx2});
    if (__builtin_cpu_supports("avx512f") && __builtin_cpu_supports("avx512dq")) v.push_back({"avx512", fill_avx512, dot_avx512});
#endif
    return v;
}

void check_variants() {
    Stream keys(11, Stream::kLweKey), words(12, Stream::kEncMask);
    for (int n : {1, 2, 3, 7, 8, 9, 15, 16, 17, 31, 32, 33, 63, 65, 500, 501, 1023, 1024, 4097}) {
        std::vector<uint32_t> select((size_t)n);
        for (int j = 0; j < n; ++j) select[(size_t)j] = 0u - keys.bit((uint64_t)j);
        for (uint64_t first : {(uint64_t)0, (uint64_t)1, (uint64_t)500 * 12345, (uint64_t)0xFFFFFFF0u}) {
            std::vector<uint32_t> want((size_t)n);
            uint32_t sum = 0;
            for (int j = 0; j < n; ++j) {
                want[(size_t)j] = words.word32(first + (uint64_t)j);
                if (select[(size_t)j]) sum += want[(size_t)j];
            }
            for (const Variant &v : variants()) {
                std::vector<uint32_t> c((size_t)n + 1, 0xA5A5A5A5u);
                CHECK(v.fill(words.origin() + kGolden * (first + 1), select.data(), c.data(), n) == sum);
                CHECK(std::memcmp(c.data(), want.data(), (size_t)n * 4) == 0 && c[(size_t)n] == 0xA5A5A5A5u);
                CHECK(v.dot(select.data(), want.data(), n) == sum);
            }
        }
    }
    std::printf("instruction sets:");
    for (const Variant &v : variants()) std::printf(" %s", v.name);
    std::printf("\n");
}

void check_ranges() {
    for (size_t count : {0, 1, 2, 15, 16, 17, 199, 200, 399, 400, 401, 3333, 12544})
        for (size_t grain : {1, 7, 200, 800, 100000}) {
            std::vector<uint8_t> seen(count, 0);
            parallel_ranges(count, grain, [&](size_t begin, size_t end) { for (size_t k = begin; k < end; ++k) ++seen[k]; });
            for (uint8_t s : seen) CHECK(s == 1);
        }
}

// several threads: n = 500 shares out from 400 samples (encryption) and 1,600 (decryption), n = 3 later
void check_calls() {
    for (int n : {3, 500}) {
        const tfhe_params P{n, 2, 1, 2, 10, 1, 1, -15, -25};
        tfhe_secret_key *sk = nullptr;
        CHECK(tfhe_keygen(&P, 77, &sk, nullptr) == TFHE_OK);
        const size_t counts[] = {1, 399, 401, n == 3 ? (size_t)200001 : (size_t)3333};
        for (size_t count : counts) {
            std::vector<uint8_t> bits(count), back(count, 9);
            std::vector<uint32_t> ct(count * (size_t)(n + 1) + 1, 0xA5A5A5A5u), want((size_t)n + 1);
            const Stream mask(5, Stream::kEncMask), err(5, Stream::kEncNoise), coin(6, Stream::kKsMask);
            for (size_t s = 0; s < count; ++s) bits[s] = (uint8_t)(coin.word32(s) & 1);
            CHECK(tfhe_encrypt(sk, 5, bits.data(), count, ct.data()) == TFHE_OK);
            CHECK(ct.back() == 0xA5A5A5A5u);
            for (size_t s = 0; s < count; ++s) {
                uint32_t body = (bits[s] ? kEighth : 0u - kEighth) + err.noise(s, P.lwe_noise_log2);
                for (int j = 0; j < n; ++j) {
                    want[(size_t)j] = mask.word32(s * (uint64_t)n + (uint64_t)j);
                    if (sk->lwe[(size_t)j]) body += want[(size_t)j];
                }
                want[(size_t)n] = body;
                CHECK(std::memcmp(want.data(), &ct[s * (size_t)(n + 1)], want.size() * 4) == 0);
            }
            for (size_t s = 0; s < count; ++s) ct[s * (size_t)(n + 1) + (size_t)n] += coin.word32(s + count);      // any phase
            CHECK(tfhe_decrypt(sk, ct.data(), count, back.data()) == TFHE_OK);
            for (size_t s = 0; s < count; ++s) {
                uint32_t phase = (bits[s] ? kEighth : 0u - kEighth) + err.noise(s, P.lwe_noise_log2) + coin.word32(s + count);
                CHECK(back[s] == ((int32_t)phase > 0));
            }
        }
        tfhe_free_secret_key(sk);
    }
}

}  // namespace

int main() {
    check_variants();
    check_ranges();
    check_calls();
    std::puts("client: ok");
    return 0;
}
